// Block metadata (Section 2.2; built when a block fills, Section 3.1): the
// bounding cuboid (channel-wise min and max) of the keys of each KV block,
// or, as the mean-key variant, the mean of the block's keys.
//
// HBM bounds it: each key is read once, and little is written.  A wave owns
// up to 8 consecutive blocks and issues all of its loads (16 KiB for cuboids)
// before it reduces anything.  Keys that cannot still lie in the
// 256 MB last-level cache (more than kLargeBytes of them) are read with the
// non-temporal policy, and with the heads' waves side by side where the
// heads' rows are interleaved (place(), below).  A layer of a 128k-token
// prompt (token-major, 8 heads, 302 MB moved): cuboids 77.5 us before, 61.2
// with the default policy, 53.4 with both (5.66 TB/s); mean keys 67.7, 53.5
// and 47.6 us.  128k tokens as block records: 61.3 and 50.9 us, mean keys
// 49.5 and 45.9.  Within the cache both cost time: 33 MB of keys in blocks of
// 8 took 15.0 us without them and 16.2 to 18.6 with the non-temporal policy,
// and the mean keys of 67 MB in blocks of 32 took 12.0 us unit by unit and
// 13.0 with the heads side by side.
#include "internal.hpp"

namespace {

constexpr int D = ss::kHeadDim;
constexpr int WAVES = 4;
constexpr int64_t kLargeBytes = 160LL << 20;  // slower at 128 MiB of keys, faster at 192

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef short i16x2_t __attribute__((ext_vector_type(2)));

// two bf16 values -> two 16-bit keys whose signed order is IEEE totalOrder
// (-0 < +0): negative values flip their magnitude bits.  Its own inverse.
__device__ __forceinline__ uint32_t key2(uint32_t w)
{
    const i16x2_t sign = __builtin_bit_cast(i16x2_t, w) >> 15;
    return w ^ (__builtin_bit_cast(uint32_t, sign) & 0x7FFF7FFFu);
}

__device__ __forceinline__ uint32_t min2(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(i16x2_t, a),
                                                                  __builtin_bit_cast(i16x2_t, b)));
}

// lanes 0..31: the minimum of a over its two halves, lanes 32..63: that of b
__device__ __forceinline__ uint32_t min_halves(uint32_t a, uint32_t b)
{
    const auto x = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return min2(x[0], x[1]);
}

// per 32 lanes: the first 16 hold the minimum of a over its two 16-lane rows, the others that of b
__device__ __forceinline__ uint32_t min_rows(uint32_t a, uint32_t b)
{
    const auto x = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    return min2(x[0], x[1]);
}

template <bool STREAM, class T>
__device__ __forceinline__ T load(const T *p)
{
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}

struct place_t {
    uint32_t u;  // unit
    int j0, n;   // first block of the wave, blocks of the unit
};

// Wave -> `per` consecutive blocks of a unit.  Where a unit's keys lie on
// their own the waves walk unit after unit; where the heads' rows are
// interleaved (token-major KV) and come from HBM, neighbouring waves take the
// heads of the same blocks, so that together they read whole tokens: one head
// at a time, all reads in flight fall on the same 256 bytes of every token,
// which are few of the memory channels.
// A launch has fewer than 2^26 waves, so I may be 32 bits wide (the cuboid of
// one block of 16 takes 2.45 us with them and 2.56 with 64; but the mean keys
// of a large token-major prompt in blocks of 8 53.0 us with them, 50.9 with 64).
template <class I>
__device__ __forceinline__ place_t place(I wave, int per, const int32_t *nblk, int Hkv, int nblk_max, int heads_inner)
{
    const int groups = (nblk_max + per - 1) / per;
    place_t p;
    I grp;
    if (heads_inner) {
        const I x = wave / Hkv;
        const I b = x / groups;
        p.u = (uint32_t)(b * Hkv + (wave - x * Hkv));
        grp = x - b * groups;
    } else {
        const I u = wave / groups;
        p.u = (uint32_t)u;
        grp = wave - u * groups;
    }
    p.j0 = (int)grp * per;
    const int n = nblk[(I)p.u / Hkv];
    p.n = n < 0 ? 0 : (n > nblk_max ? nblk_max : n);
    return p;
}

// Cuboids.  A lane loads 16 B (8 channels) of one row per step, so a
// wave-wide load covers 4 rows, and reduces its rows of each block; the four
// 16-lane rows then exchange halves instead of all reducing everything: with
// four blocks, lane row r ends with block r of them.  The largest key is
// found as the complement of the smallest complement, so every step is one
// packed minimum.
// The wave's blocks from their loaded rows to m; live(b): block b is stored.
template <int BPW, int LPB, class Live>
__device__ __forceinline__ void reduce_blocks(const u32x4_t (&v)[BPW][LPB], uint16_t *m, int row, const Live &live)
{
    uint32_t lo[BPW][4], nhi[BPW][4];  // nhi: complements of the largest keys
#pragma unroll
    for (int b = 0; b < BPW; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo[b][i] = key2(v[b][0][i]);
            nhi[b][i] = ~lo[b][i];
#pragma unroll
            for (int r = 1; r < LPB; ++r) {
                const uint32_t k = key2(v[b][r][i]);
                lo[b][i] = min2(lo[b][i], k);
                nhi[b][i] = min2(nhi[b][i], ~k);
            }
        }
    if constexpr (BPW == 2) {
        // lane rows 0, 1: lo and hi of the first block, rows 2, 3: of the second
        uint4 x;
        uint32_t *xs = &x.x;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t k = min_rows(min_halves(lo[0][i], lo[1][i]), min_halves(nhi[0][i], nhi[1][i]));
            xs[i] = key2(row & 1 ? ~k : k);
        }
        if (live(row >> 1)) *reinterpret_cast<uint4 *>(m + row * D) = x;
    } else {
#pragma unroll
        for (int b = 0; b < BPW; b += 4) {
            uint4 x, y;
            uint32_t *xs = &x.x, *ys = &y.x;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                xs[i] = key2(min_rows(min_halves(lo[b][i], lo[b + 2][i]), min_halves(lo[b + 1][i], lo[b + 3][i])));
                ys[i] = key2(~min_rows(min_halves(nhi[b][i], nhi[b + 2][i]),
                                       min_halves(nhi[b + 1][i], nhi[b + 3][i])));
            }
            if (live(b + row)) {
                *reinterpret_cast<uint4 *>(m + (b + row) * (2 * D)) = x;
                *reinterpret_cast<uint4 *>(m + (b + row) * (2 * D) + D) = y;
            }
        }
    }
}

template <int BLK, bool STREAM>
__global__ __launch_bounds__(WAVES * 64) void meta_kernel(const uint8_t *__restrict__ kv_base,
                                                          const int64_t *__restrict__ unit_off,
                                                          const int32_t *__restrict__ nblk, int Hkv, int nblk_max,
                                                          uint32_t waves, int heads_inner, int64_t block_stride,
                                                          int64_t row_stride, uint16_t *__restrict__ meta)
{
    constexpr int BPW = 64 / BLK;  // blocks per wave: 16 loads of 16 B per lane in flight
    constexpr int LPB = BLK / 4;   // wave-wide loads per K tile (4 rows each)
    const int lane = threadIdx.x & 63;
    const uint32_t w = blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= waves) return;
    const place_t p = place(w, BPW, nblk, Hkv, nblk_max, heads_inner);
    if (p.j0 >= p.n) return;
    const int row = lane >> 4, c16 = lane & 15;
    const uint8_t *src = kv_base + unit_off[p.u] + row * row_stride + c16 * 16;

    u32x4_t v[BPW][LPB];
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
        const int j = min(p.j0 + b, p.n - 1);  // past the end: the last block again, not stored
#pragma unroll
        for (int r = 0; r < LPB; ++r)
            v[b][r] = load<STREAM>(reinterpret_cast<const u32x4_t *>(src + j * block_stride + 4 * r * row_stride));
    }
    reduce_blocks(v, meta + ((int64_t)p.u * nblk_max + p.j0) * (2 * D) + c16 * 8, row,
                  [&](int b) { return p.j0 + b < p.n; });
}

// The same with a wave's blocks consecutive ones of all units (a unit's last
// and the next one's first share a wave), whose metadata is consecutive too;
// missing ones are not read.  Short rows leave no part of a wave idle that way,
// and more of a large launch's loads are in flight; where a launch is small the
// look-up of each block's unit costs 0.3 to 1 us.  us, units of n blocks: a wave
// per unit's blocks before and now, and this (keys read once, four sets in turn):
// 16384 x 1 in blocks of 8 17.7, 17.7, 9.7; 65536 x 1 in blocks of 32 172, 172,
// 98; 8192 x 33 of 8 146, 146, 128; 512 x 9 of 8 4.4, 4.4, 5.0.
template <int BLK, bool STREAM>
__global__ __launch_bounds__(WAVES * 64) void meta_flat_kernel(const uint8_t *__restrict__ kv_base,
                                                               const int64_t *__restrict__ unit_off,
                                                               const int32_t *__restrict__ nblk, uint32_t units,
                                                               int Hkv, int nblk_max, uint32_t waves,
                                                               int64_t block_stride, int64_t row_stride,
                                                               uint16_t *__restrict__ meta)
{
    constexpr int BPW = 64 / BLK;
    constexpr int LPB = BLK / 4;
    const int lane = threadIdx.x & 63;
    const uint32_t w = blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= waves) return;
    const int row = lane >> 4, c16 = lane & 15;
    // where the blocks lie, then all units' counts and offsets side by side
    uint32_t u = w * BPW / (uint32_t)nblk_max, seq = u / (uint32_t)Hkv;
    int j = (int)(w * BPW - u * nblk_max), g = (int)(u - seq * Hkv);
    const uint32_t last = units - 1, last_seq = last / (uint32_t)Hkv;
    int n[BPW], at[BPW];
    int64_t off[BPW];
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
        at[b] = u < units ? j : nblk_max;
        n[b] = nblk[min(seq, last_seq)];
        off[b] = unit_off[min(u, last)];
        if (++j == nblk_max) {
            j = 0;
            ++u;
            if (++g == Hkv) {
                g = 0;
                ++seq;
            }
        }
    }
    uint32_t live = 0;
    u32x4_t v[BPW][LPB];
    const uint8_t *base = kv_base + row * row_stride + c16 * 16;
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
        if (at[b] < min(n[b], nblk_max)) {
            live |= 1u << b;
            const uint8_t *src = base + off[b] + at[b] * block_stride;
#pragma unroll
            for (int r = 0; r < LPB; ++r)
                v[b][r] = load<STREAM>(reinterpret_cast<const u32x4_t *>(src + 4 * r * row_stride));
        } else {
#pragma unroll
            for (int r = 0; r < LPB; ++r) v[b][r] = u32x4_t{0, 0, 0, 0};
        }
    }
    if (!live) return;
    reduce_blocks(v, meta + (int64_t)w * BPW * (2 * D) + c16 * 8, row, [&](int b) { return (live >> b & 1u) != 0; });
}

// Mean key of each block: one wave per block, each lane two channels (with
// two blocks per wave and four channels per lane the mean keys of 128k tokens
// in blocks of 16 took 48.2 to 49.7 us against 47.6 and 45.9); the rows are
// summed in fp64 in token order (the sum of blk bf16 keys is exact unless
// their magnitudes span more than about 2^40), scaled by 1/blk (exact) and
// rounded once to bf16, ties to even.
template <int BLK, bool STREAM>
__global__ __launch_bounds__(WAVES * 64) void meta_mean_kernel(const uint8_t *__restrict__ kv_base,
                                                               const int64_t *__restrict__ unit_off,
                                                               const int32_t *__restrict__ nblk, int Hkv,
                                                               int nblk_max, uint32_t waves, int heads_inner,
                                                               int64_t block_stride, int64_t row_stride,
                                                               uint16_t *__restrict__ meta)
{
    const int lane = threadIdx.x & 63;
    const uint32_t w = blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= waves) return;
    const place_t p = place((int64_t)w, 1, nblk, Hkv, nblk_max, heads_inner);
    if (p.j0 >= p.n) return;
    const uint8_t *src = kv_base + unit_off[p.u] + p.j0 * block_stride + lane * 4;

    uint32_t v[BLK];
#pragma unroll
    for (int t = 0; t < BLK; ++t) v[t] = load<STREAM>(reinterpret_cast<const uint32_t *>(src + t * row_stride));
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int t = 0; t < BLK; ++t) {
        s0 += (double)__uint_as_float(v[t] << 16);
        s1 += (double)__uint_as_float(v[t] & 0xFFFF0000u);
    }
    reinterpret_cast<uint32_t *>(meta + ((int64_t)p.u * nblk_max + p.j0) * D)[lane] =
        ss::pack_bf16_rne_f64(s0 * (1.0 / BLK), s1 * (1.0 / BLK));
}

// the kernel for a kind, a block size and a cache policy; flat: cuboids in meta_flat_kernel
template <int BLK, bool STREAM>
void launch_blk(int meta_kind, bool flat, dim3 gr, hipStream_t s, const uint8_t *kv, const int64_t *unit_off,
                const int32_t *nblk, int64_t units, int Hkv, int nblk_max, int64_t waves, int inner, int64_t bs,
                int64_t rs, uint16_t *m)
{
    const dim3 bl(WAVES * 64);
    if (flat)
        ss::launch(meta_flat_kernel<BLK, STREAM>, gr, bl, s, kv, unit_off, nblk, units, Hkv, nblk_max, waves, bs, rs, m);
    else if (meta_kind == SS_META_CUBOID)
        ss::launch(meta_kernel<BLK, STREAM>, gr, bl, s, kv, unit_off, nblk, Hkv, nblk_max, waves, inner, bs, rs, m);
    else
        ss::launch(meta_mean_kernel<BLK, STREAM>, gr, bl, s, kv, unit_off, nblk, Hkv, nblk_max, waves, inner, bs, rs, m);
}

}  // namespace

extern "C" ss_status ss_build_metadata_strided(const void *kv_base, const int64_t *unit_off, const int32_t *nblk,
                                               int B, int Hkv, int nblk_max, int blk, int d, int64_t block_stride,
                                               int64_t row_stride, int meta_kind, void *meta, void *stream)
{
    SS_CHECK_ARG(B >= 0 && Hkv > 0 && nblk_max >= 0, "ss_build_metadata: bad shape B=%d Hkv=%d nblk_max=%d", B,
                 Hkv, nblk_max);
    SS_CHECK_ARG(meta_kind == SS_META_CUBOID || meta_kind == SS_META_MEAN, "ss_build_metadata: metadata kind %d",
                 meta_kind);
    SS_CHECK_SUPPORTED(d == ss::kHeadDim, "ss_build_metadata: d=%d (only 128)", d);
    SS_CHECK_SUPPORTED(ss::supported_blk(blk), "ss_build_metadata: blk=%d (8, 16 or 32)", blk);
    SS_CHECK_SUPPORTED(nblk_max <= ss::kMaxBlocks, "ss_build_metadata: nblk_max=%d > %d", nblk_max, ss::kMaxBlocks);
    SS_CHECK_ARG(block_stride > 0 && row_stride > 0 && block_stride % 16 == 0 && row_stride % 16 == 0,
                 "ss_build_metadata: strides %lld, %lld must be positive multiples of 16", (long long)block_stride,
                 (long long)row_stride);
    if ((int64_t)B * nblk_max == 0) return SS_OK;
    SS_CHECK_ARG(kv_base && unit_off && nblk && meta, "ss_build_metadata: null pointer");
    SS_CHECK_ARG(((uintptr_t)kv_base & 15) == 0 && ((uintptr_t)meta & 15) == 0,
                 "ss_build_metadata: kv_base and meta must be 16-byte aligned");
    const int per = meta_kind == SS_META_CUBOID ? 64 / blk : 1;  // blocks per wave
    const int64_t units = (int64_t)B * Hkv, rows = units * nblk_max * blk;
    const int64_t flat_waves = (units * nblk_max + per - 1) / per;
    const int64_t grid_least = (flat_waves + WAVES - 1) / WAVES;
    SS_CHECK_SUPPORTED(grid_least * WAVES * 64 <= 0xFFFFFFFFll, "ss_build_metadata: too many blocks");
    const bool large = rows * (d * 2) > kLargeBytes;
    const int64_t unit_waves = units * ((nblk_max + per - 1) / per);
    // Other heads' rows lie between a head's rows: the stride spans the keys of
    // all heads (with two heads it may span their own values instead, which
    // costs nothing).  Heads that lie one after another, each with its values,
    // are slower side by side: mean keys of 4 x 16384 blocks of 16 46.4 us, 50.2
    // that way, cuboids 52.9 and 55.2.  In rows of 16 waves or more the last one
    // of each, which may hold one block, is lost among them.
    const int inner = large && Hkv > 1 && row_stride >= (int64_t)Hkv * d * 2 && nblk_max >= 16 * per && unit_waves * 64 <= 0xFFFFFFFFll;
    // From 64 MiB of keys on the blocks go to waves across the units (64 MiB in
    // blocks of 8, 2048 units: 16.6 us both ways, 128 MiB 40.3 and 37.6, 256 MiB
    // 73.1 and 64.6; 8 MiB, 256 units, 6.1 and 7.7); so do many units that would
    // fill half a wave each (4096 of one block of 8: 6.4 and 4.9 us, of 16 7.1 and
    // 5.7; 2048: 3.9 and 4.6, 4.4 and 4.2).
    // Rows with others between them gain nothing before they come from HBM
    // (1024 blocks of 32, 8 heads, token-major: 36.8 and 38.8 us).
    const bool flat = meta_kind == SS_META_CUBOID && !inner &&
                      ((row_stride > d * 2 ? large : rows > (1 << 18)) || (units >= 4096 && 2 * nblk_max <= per));
    const int64_t waves = flat ? flat_waves : unit_waves;
    hipStream_t s = ss::as_stream(stream);
    const uint8_t *kv = static_cast<const uint8_t *>(kv_base);
    const dim3 gr((unsigned)((waves + WAVES - 1) / WAVES));
    auto *go = large ? launch_blk<32, true> : launch_blk<32, false>;
    if (blk == 8) go = large ? launch_blk<8, true> : launch_blk<8, false>;
    else if (blk == 16) go = large ? launch_blk<16, true> : launch_blk<16, false>;
    go(meta_kind, flat, gr, s, kv, unit_off, nblk, units, Hkv, nblk_max, waves, inner, block_stride, row_stride,
       static_cast<uint16_t *>(meta));
    return ss::check_launch("ss_build_metadata");
}

extern "C" ss_status ss_build_metadata(const void *kv_base, const int64_t *unit_off, const int32_t *nblk, int B,
                                       int Hkv, int nblk_max, int blk, int d, void *meta, void *stream)
{
    const int64_t rec = 2LL * blk * d * 2;  // block records: K rows of d bf16 each
    return ss_build_metadata_strided(kv_base, unit_off, nblk, B, Hkv, nblk_max, blk, d, rec, (int64_t)d * 2,
                                     SS_META_CUBOID, meta, stream);
}

extern "C" ss_status ss_build_metadata_mean(const void *kv_base, const int64_t *unit_off, const int32_t *nblk,
                                            int B, int Hkv, int nblk_max, int blk, int d, void *meta, void *stream)
{
    const int64_t rec = 2LL * blk * d * 2;
    return ss_build_metadata_strided(kv_base, unit_off, nblk, B, Hkv, nblk_max, blk, d, rec, (int64_t)d * 2,
                                     SS_META_MEAN, meta, stream);
}
