// Top-k block selection per (sequence, KV head) (Section 2.2), ties to the
// lower block index, output in ascending block order.
//
// One workgroup per unit, the unit's scores in registers as 32-bit keys whose
// unsigned order is the float order (-0 folded onto +0; key 0, below every
// score, for padding).  Wave w owns R*64 consecutive scores, lane l of it the
// scores i*64 + l of those: the loads are coalesced, are issued before the
// unit's block count arrives (loads past the row's nblk_max scores read as
// zero, by the bounds of its buffer), and ranks in block order are ballots.
//
// The selection is every key above a bound and the first `quota` keys equal
// to it.  To find the bound (m = min(k, n) keys wanted):
//   - one wave: bit by bit from the highest bit in which the keys differ,
//     counting the keys at or above the trial value with ballots, until
//     exactly the wanted number is;
//   - several waves: the range of the keys is cut into 256 equal intervals
//     (a shift of key - lowest key) and counted into them in LDS; the interval
//     of the m-th largest key holds few of them (about ten of 8192 Gaussian
//     scores with k = 128).  They are collected in LDS, and every wave finds
//     the bound among them by itself, bit by bit, one key a lane.  An interval
//     with more keys than lanes is cut again: searched in place, up to 512 of
//     them eight a lane, few distinct values cost every wave all their bits
//     (1024 units of 1025 whole numbers below 200: 15.9 us, cut again 9.8).
// LDS atomics of one instruction to one address are done one lane at a time,
// so the counts go to 8 copies (lane l to copy l mod 8), laid out so that the
// copies of an interval lie in different banks and four intervals of a copy
// are one 16-byte read (16 copies: up to 4% slower on Gaussian scores).
//
// What bounds it is latency: the chain of loads, exchanges between the waves
// (LDS and a barrier) and the kernel's own launch.  Reductions and scans
// within a wave are DPP and lane swaps, not LDS shuffles, and the loops over
// a lane's keys are free of branches (a taken branch per key was a quarter of
// the kernel).  Dispatch events, us, Gaussian scores, with the 8-bit radix
// passes over consecutive scores handed out through LDS, shuffle reductions
// and scans that this replaces, and now (an empty kernel reads about 4):
// 8 units of 8192 blocks 9.4, 5.7; 512 units 12.1, 7.9; 256 of 2048 6.0, 4.4;
// 192 of 16384 (k = 512) 13.0, 10.6; 8 of 65536 55.8, 21.7.  Outliers above a
// tight band, 512 units of 8192: 19.9, 12.6; one value but for one: 52.5,
// 14.4.  In graphs: whole numbers below 200, 1024 units of 1025 10.9, 9.7; N(0,1),
// 512 of 1025 7.4, 6.1.
#include <climits>

#include "score_tile.hpp"

namespace {

constexpr int kCopies = 8;            // copies of the interval counts
constexpr int kPitch = 256 + 4;        // words per copy: one interval's copies lie in different banks
constexpr int kCand = 64;              // most keys of the last search, one per lane
constexpr int kBufferFlags = 0x00020000;  // raw buffer descriptor word 3 for gfx9 (32-bit data)

// order-preserving key of a score's bits; at least 1 (0 is padding)
__device__ __forceinline__ uint32_t score_key(uint32_t x)
{
    const uint32_t b = __float_as_uint(__uint_as_float(x) + 0.0f);  // -0 -> +0
    return max(b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u), 1u);
}

// a value that is the same in every lane, as a scalar
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// minimum over the wave, in every lane
__device__ __forceinline__ uint32_t wave_min(uint32_t x)
{
    x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false));   // lane ^ 1
    x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false));   // lane ^ 2
    x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, false));  // mirrored in 8 lanes
    x = min(x, (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x140, 0xF, 0xF, false));  // mirrored in 16 lanes
    const auto h = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = min(h[0], h[1]);
    const auto w = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return min(w[0], w[1]);
}

// inclusive prefix sum over the wave
__device__ __forceinline__ int wave_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);  // from 1, 2, 4, 8 lanes below in the row
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // the row below's total, rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // the lower half's total, rows 2 and 3
    return x;
}

// bits of R keys
template <int R>
struct bits_of {
    typedef uint32_t type;
};
template <>
struct bits_of<64> {
    typedef unsigned long long type;
};
__device__ __forceinline__ int popcount(uint32_t x) { return __popc(x); }
__device__ __forceinline__ int popcount(unsigned long long x) { return __popcll(x); }
__device__ __forceinline__ int lowest(uint32_t x) { return __ffs(x) - 1; }
__device__ __forceinline__ int lowest(unsigned long long x) { return __ffsll(x) - 1; }

// The selection: keys above `above`, and the first `quota` keys equal to it.
struct bound_t {
    uint32_t above;
    int quota;
};

// The bound of the `want` largest of the wave's keys lo + off[*] (offsets of
// 0, padding among them, only win if nothing else is left), 0 < want <= the
// keys there.  span: no offset is larger.
template <int N>
__device__ __forceinline__ bound_t search(const uint32_t (&off)[N], uint32_t lo, uint32_t span, int want)
{
    uint32_t t = 0;
    int at_least = INT_MAX;  // keys at or above t: the whole set at t = 0
    for (int bit = span ? 31 - __clz(span) : -1; bit >= 0; --bit) {
        const uint32_t trial = t | 1u << bit;
        int c = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) c += __popcll(__ballot(off[i] >= trial));
        if (c >= want) {
            t = trial;
            at_least = c;
            if (c == want) break;
        }
    }
    if (at_least == want) return {lo + t - 1, 0};
    int c = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) c += __popcll(__ballot(off[i] > t));
    return {lo + t, want - c};
}

// The bound of the m largest of one wave's keys, m below their number; lo, hi:
// the smallest key - 1 and the complement of the largest.
template <int R>
__device__ __forceinline__ bound_t bound_of_wave(const uint32_t (&key)[R], uint32_t lo, uint32_t hi, int m)
{
    lo = uniform(lo) + 1u;
    uint32_t off[R];
#pragma unroll
    for (int i = 0; i < R; ++i) off[i] = key[i] ? key[i] - lo : 0u;
    return search(off, lo, ~uniform(hi) - lo, m);
}

// smallest key - 1 and complement of the largest key over the wave (padding wraps to the largest)
template <int R>
__device__ __forceinline__ void key_range(const uint32_t (&key)[R], uint32_t &lo, uint32_t &hi)
{
    lo = 0xFFFFFFFFu;
    hi = 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        lo = min(lo, key[i] - 1u);
        hi = min(hi, ~key[i]);
    }
    lo = wave_min(lo);
    hi = wave_min(hi);
}

template <int NW, int R>
struct place_t {
    alignas(8) uint32_t map[2][NW][2 * R];  // a bit per score
    int tot[2][NW];
};

// Writes the unit's selection (and its copy) in block order.  The lanes hand
// the selected scores' bits to the lane that owns R consecutive ones (all of
// them this wave's own, so the waves exchange only their totals); a scan of
// the lanes' bit counts places each lane's first output.  A key equal to the
// bound is taken if fewer than `quota` of them come before it.
template <int NW, int R>
__device__ __forceinline__ void place(const uint32_t (&key)[R], bound_t bound, int m, int wave, int lane, int32_t *out,
                                      int32_t *out2, place_t<NW, R> &sm)
{
    typedef typename bits_of<R>::type bits_t;
    auto hand_over = [&](int which, auto taken) -> bits_t {
        uint32_t lo = 0, hi = 0;
        int c = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const unsigned long long mask = __ballot(taken(key[i]));
            lo = lane == i ? (uint32_t)mask : lo;
            hi = lane == i ? (uint32_t)(mask >> 32) : hi;
            c += __popcll(mask);
        }
        uint32_t *map = sm.map[which][wave];
        if (lane < R) {
            map[2 * lane] = lo;
            map[2 * lane + 1] = hi;
        }
        if (lane == 0) sm.tot[which][wave] = c;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if constexpr (R == 64) {
            return (unsigned long long)map[2 * lane + 1] << 32 | map[2 * lane];
        } else {
            return (map[lane * R / 32] >> (lane * R % 32)) & ((1u << R) - 1u);
        }
    };
    bits_t bits = hand_over(0, [&](uint32_t x) { return x > bound.above; }), eq_bits = 0;
    if (bound.quota) eq_bits = hand_over(1, [&](uint32_t x) { return x == bound.above; });
    int pos = wave_scan(popcount(bits)) - popcount(bits);
    if constexpr (NW > 1) {
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) pos += w < wave ? sm.tot[0][w] : 0;
    }
    if (bound.quota) {
        int before = wave_scan(popcount(eq_bits)) - popcount(eq_bits);
        if constexpr (NW > 1) {
#pragma unroll
            for (int w = 0; w < NW; ++w) before += w < wave ? sm.tot[1][w] : 0;
        }
        pos += min(before, bound.quota);
        int left = max(bound.quota - before, 0);
        for (bits_t e = eq_bits; e && left > 0; e &= e - 1, --left) bits |= e & (~e + 1);
    }
    const int first = (wave * 64 + lane) * R;
    for (; bits; bits &= bits - 1, ++pos)
        if (pos < m) {  // always holds; the guard keeps writes in range
            const int j = first + lowest(bits);
            out[pos] = j;
            if (out2) out2[pos] = j;
        }
}

// R = 16 is held to the 64 registers at which two workgroups of 1024 threads share a CU
template <int NT, int R>
__global__ __launch_bounds__(NT, R == 16 ? 8 : 1) void topk_kernel(const float *__restrict__ scores,
                                                                   const int32_t *__restrict__ nblk, int Hkv,
                                                                   int nblk_max, int k, int32_t *__restrict__ sel,
                                                                   int32_t *__restrict__ mirror)
{
    constexpr int NW = NT / 64;
    const int u = blockIdx.x;
    const int b = u / Hkv;
    const float *s = scores + (int64_t)u * nblk_max;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int e0 = wave * (64 * R) + lane;  // the lane's first score

    // the whole row's loads first; the block count masks them afterwards
    // (buffer loads: those past nblk_max read as zero)
    const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc((void *)s, (short)0, nblk_max * 4, kBufferFlags);
    uint32_t key[R];
#pragma unroll
    for (int i = 0; i < R; ++i) key[i] = __builtin_amdgcn_raw_buffer_load_b32(row, (e0 + i * 64) * 4, 0, 0);
    __shared__ __align__(16) int count[NW > 1 ? kCopies * kPitch : 4];
    auto clear = [&] {
        int4 *z = reinterpret_cast<int4 *>(count);
#pragma unroll
        for (int i = 0; i < kCopies * kPitch / 4; i += NT)  // no counter a lane, for which R = 16 had no register left
            if (i + t < kCopies * kPitch / 4) z[i + t] = make_int4(0, 0, 0, 0);
    };
    if constexpr (NW > 1) clear();
    int n = nblk[b];
    n = n < 0 ? 0 : (n > nblk_max ? nblk_max : n);
    const int m = k < n ? k : n;
    int32_t *out = sel + (int64_t)u * k;
    int32_t *out2 = mirror ? mirror + (int64_t)u * k : nullptr;  // copy in mapped host memory
    for (int i = m + t; i < k; i += NT) {
        out[i] = -1;
        if (out2) out2[i] = -1;
    }
    if (m == 0) return;
#pragma unroll
    for (int i = 0; i < R; ++i) key[i] = e0 + i * 64 < n ? score_key(key[i]) : 0u;

    bound_t bound = {0u, 0};  // every key, where all are selected
    if (m < n) {
        uint32_t lo, hi;
        key_range(key, lo, hi);
        if constexpr (NW == 1) {
            bound = bound_of_wave(key, lo, hi, m);
        } else {
            __shared__ uint32_t cand[kCand];
            __shared__ uint32_t red_lo[NW], red_hi[NW];
            __shared__ int pick[3], n_cand;
            if (lane == 0) {
                red_lo[wave] = lo;
                red_hi[wave] = hi;
            }
            if (t == 0) n_cand = 0;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                lo = min(lo, red_lo[w]);
                hi = min(hi, red_hi[w]);
            }
            lo = uniform(lo) + 1u;
            const uint32_t top = ~uniform(hi);
            uint32_t span = top - lo;  // the bound lies in [lo, lo + span]
            int want = m;              // keys wanted from there
            for (;;) {
                if (span == 0) {
                    bound = {lo, want};
                    break;
                }
                const int bits = 32 - __clz(span);
                const int shift = bits > 8 ? bits - 8 : 0;
                const int c = (lane & (kCopies - 1)) * kPitch;
#pragma unroll
                for (int i = 0; i < R; ++i)
                    if (key[i] - lo <= span) atomicAdd(&count[c + ((key[i] - lo) >> shift)], 1);
                __syncthreads();
                if (wave == 0) {
                    // lane l holds intervals 255-4l .. 252-4l (descending order)
                    int4 v = make_int4(0, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < kCopies; ++i) {
                        const int4 y = *reinterpret_cast<const int4 *>(count + i * kPitch + 252 - 4 * lane);
                        v.x += y.x;
                        v.y += y.y;
                        v.z += y.z;
                        v.w += y.w;
                    }
                    const int sum = (v.x + v.y) + (v.z + v.w);
                    const int incl = wave_scan(sum);
                    const int above = incl - sum;  // keys in higher intervals than this lane's
                    if (above < want && want <= incl) {
                        const int in[4] = {v.w, v.z, v.y, v.x};
                        int acc = above;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if (acc < want && want <= acc + in[i]) {
                                pick[0] = 255 - 4 * lane - i;
                                pick[1] = want - acc;
                                pick[2] = in[i];
                            }
                            acc += in[i];
                        }
                    }
                }
                __syncthreads();
                lo += uniform((uint32_t)pick[0]) << shift;
                span = min((1u << shift) - 1u, top - lo);  // an interval past `top` could wrap to the padding
                want = uniform(pick[1]);
                const int held = uniform(pick[2]);
                if (want == held) {  // the whole interval
                    bound = {lo - 1u, 0};
                    break;
                }
                if (span && held <= kCand) {
#pragma unroll
                    for (int h = 0; h < R; h += 32) {
                        // per lane the bits of its keys there; branches only for the few waves that have any
                        uint32_t bits = 0;
#pragma unroll
                        for (int i = h; i < R && i < h + 32; ++i) bits |= (key[i] - lo <= span ? 1u : 0u) << (i - h);
                        if (!__ballot(bits != 0)) continue;
                        const int incl = wave_scan(__popc(bits));
                        int at = 0;
                        if (lane == 63) at = atomicAdd(&n_cand, incl);
                        at = __builtin_amdgcn_readlane(at, 63) + incl - __popc(bits);
                        while (__ballot(bits != 0)) {
                            const int low = __ffs(bits) - 1;
                            uint32_t v = 0;
#pragma unroll
                            for (int i = h; i < R && i < h + 32; ++i) v = low == i - h ? key[i] : v;
                            if (bits) cand[at] = v - lo;
                            ++at;
                            bits &= bits - 1;
                        }
                    }
                    __syncthreads();
                    const uint32_t off[1] = {lane < held ? cand[lane] : 0u};
                    bound = search(off, lo, span, want);
                    break;
                }
                if (span) {
                    clear();
                    __syncthreads();
                }
            }
        }
    }

    __shared__ place_t<NW, R> sm;
    place<NW, R>(key, bound, m, wave, lane, out, out2, sm);
}

// Scores and selects rows of at most 16*W blocks in one launch: one workgroup
// per unit, one wave per tile (all of the unit's metadata is in flight at
// once), then wave 0 selects from the scores in LDS.
template <int W>
__global__ __launch_bounds__(W * 64) void score_topk_kernel(const uint16_t *__restrict__ q,
                                                            const uint8_t *__restrict__ meta,
                                                            const int32_t *__restrict__ nblk, int Hq, int Hkv, int G,
                                                            int nblk_max, int k, float *__restrict__ scores,
                                                            int32_t *__restrict__ sel)
{
    constexpr int R = W * ss::kTile / 64;
    __shared__ uint4 stage[W][ss::tile_shape<SS_META_CUBOID>::STAGE];
    __shared__ uint32_t row[W * ss::kTile];
    __shared__ place_t<1, R> sm;
    const int u = blockIdx.x;
    const int b = u / Hkv, g = u - b * Hkv;
    int n = nblk[b];
    n = n < 0 ? 0 : (n > nblk_max ? nblk_max : n);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = wave * ss::kTile;
    if (j0 < n) {
        const float v = ss::score_tile<SS_META_CUBOID, SS_AGG_MAX>(q, meta, b, g, u, n, j0, Hq, G, nblk_max,
                                                                   stage[wave]);
        if (lane < ss::kTile) {
            row[j0 + lane] = __float_as_uint(v);
            if (j0 + lane < n) scores[(int64_t)u * nblk_max + j0 + lane] = v;
        }
    }
    __syncthreads();
    if (wave > 0) return;
    const int m = k < n ? k : n;
    int32_t *out = sel + (int64_t)u * k;
    for (int i = m + lane; i < k; i += 64) out[i] = -1;
    if (m == 0) return;
    uint32_t key[R];
#pragma unroll
    for (int i = 0; i < R; ++i) key[i] = i * 64 + lane < n ? score_key(row[i * 64 + lane]) : 0u;
    bound_t bound = {0u, 0};  // every key, where all are selected
    if (m < n) {
        uint32_t lo, hi;
        key_range(key, lo, hi);
        bound = bound_of_wave(key, lo, hi, m);
    }
    place<1, R>(key, bound, m, 0, lane, out, nullptr, sm);
}

template <int NT, int R>
void launch_variant(const float *scores, const int32_t *nblk, int units, int Hkv, int nblk_max, int k, int32_t *sel,
            int32_t *mirror, hipStream_t s)
{
    ss::launch(topk_kernel<NT, R>, dim3(units), dim3(NT), s, scores, nblk, Hkv, nblk_max, k, sel, mirror);
}

}  // namespace

namespace ss {

// `mirror` (nullable): a second copy of the selection, e.g. in mapped host memory
ss_status launch_topk(const float *scores, const int32_t *nblk, int B, int Hkv, int nblk_max, int k, int32_t *sel,
                      int32_t *mirror, hipStream_t s)
{
    const int units = B * Hkv;
    if (units == 0) return SS_OK;
    // Threads x scores per thread.  A wave alone finds the bound without an
    // exchange, but pays for every key in every bit: it is level with 256
    // threads up to 256 blocks (4.1 us) and slower beyond (512: 4.4 against
    // 4.2; 1024: 5.5 against 4.1).  From 2048 blocks, 512 threads of 4 to 16
    // keys against 1024 of half as many: 4.5 and 5.6 us for 256 units of 2048
    // blocks, 6.1 and 8.0 for 512 of 4096, 8.0 and 9.6 for 512 of 8192.
    if (nblk_max <= 64 * 4) launch_variant<64, 4>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 256 * 2) launch_variant<256, 2>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 256 * 4) launch_variant<256, 4>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 512 * 4) launch_variant<512, 4>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 512 * 8) launch_variant<512, 8>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 512 * 16) launch_variant<512, 16>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else if (nblk_max <= 1024 * 16) launch_variant<1024, 16>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    else launch_variant<1024, 64>(scores, nblk, units, Hkv, nblk_max, k, sel, mirror, s);
    return check_launch("ss_select_topk");
}

}  // namespace ss

extern "C" ss_status ss_select_topk(const float *scores, const int32_t *nblk, int B, int Hkv, int nblk_max, int k,
                                    int32_t *sel, void *stream)
{
    SS_CHECK_ARG(B >= 0 && Hkv > 0 && nblk_max >= 0 && k > 0, "ss_select_topk: bad shape B=%d Hkv=%d nblk_max=%d k=%d",
                 B, Hkv, nblk_max, k);
    SS_CHECK_SUPPORTED(nblk_max <= ss::kMaxBlocks, "ss_select_topk: nblk_max=%d > %d", nblk_max, ss::kMaxBlocks);
    if (B == 0) return SS_OK;
    SS_CHECK_ARG(nblk && sel && (scores || nblk_max == 0), "ss_select_topk: null pointer");
    return ss::launch_topk(scores, nblk, B, Hkv, nblk_max, k, sel, nullptr, ss::as_stream(stream));
}

extern "C" size_t ss_score_topk_workspace(int B, int Hq, int Hkv, int nblk_max, int d, int k)
{
    if (B < 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv || d != ss::kHeadDim || nblk_max < 0 || k <= 0) return 0;
    return (size_t)B * Hkv * nblk_max * sizeof(float);
}

extern "C" ss_status ss_score_topk(const void *q, const void *meta, const int32_t *nblk, int B, int Hq, int Hkv,
                                   int nblk_max, int d, int k, float *scores, int32_t *sel, void *stream)
{
    ss_status st = ss::check_score_args(q, meta, nblk, B, Hq, Hkv, nblk_max, d, scores, "ss_score_topk",
                                        SS_META_CUBOID, SS_AGG_MAX);
    if (st != SS_OK) return st;
    SS_CHECK_ARG(k > 0, "ss_score_topk: k=%d", k);
    if (B == 0) return SS_OK;
    SS_CHECK_ARG(sel, "ss_score_topk: null sel");
    hipStream_t s = ss::as_stream(stream);
    // One launch where a workgroup per unit holds its whole row in flight: a
    // launch and the scores' way through memory less.  us a call, two launches
    // and one: 4 units of 256 blocks 7.5, 5.5; 256 units of 256 10.9, 9.0; 512
    // of 100 10.2, 7.2; 512 of 64 8.6, 5.7.  16 waves fill a CU, so beyond one
    // unit a CU the selections no longer hide under other units' loads (512
    // units of 256 blocks 15.8, 16.7).  Units that do not fit a launch are left
    // to the two, which know how far they go.
    const int64_t units = (int64_t)B * Hkv;
    auto *kernel = score_topk_kernel<16>;
    int waves = 16;
    if (nblk_max <= 4 * ss::kTile) kernel = score_topk_kernel<4>, waves = 4;
    else if (nblk_max <= 8 * ss::kTile) kernel = score_topk_kernel<8>, waves = 8;
    if (nblk_max >= 1 && nblk_max <= waves * ss::kTile && (waves < 16 || units <= 256) &&
        units * waves * 64 <= 0xFFFFFFFFll) {
        ss::launch(kernel, dim3((unsigned)units), dim3(waves * 64), s, static_cast<const uint16_t *>(q),
                   static_cast<const uint8_t *>(meta), nblk, Hq, Hkv, Hq / Hkv, nblk_max, k, scores, sel);
        return ss::check_launch("ss_score_topk");
    }
    st = ss::launch_score(q, meta, SS_META_CUBOID, SS_AGG_MAX, nblk, B, Hq, Hkv, nblk_max, scores, s);
    if (st != SS_OK) return st;
    return ss::launch_topk(scores, nblk, B, Hkv, nblk_max, k, sel, nullptr, s);
}
