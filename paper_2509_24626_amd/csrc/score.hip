// Block criticality scores (Section 2.2): for block j of KV head g and each
// query head h of the group, the largest q_h.k over the block's key cuboid
// [lo, hi], then the maximum over the group's heads.
//
// Since hi >= lo channel-wise,
//     max(q*lo, q*hi) = max(q,0)*hi + min(q,0)*lo     (exactly, per channel),
// so with the metadata row m_j = [lo_j, hi_j] (256 bf16) and the query
// weights w_h = [min(q_h,0), max(q_h,0)] the per-head bound is the plain dot
// product w_h . m_j.  For one unit this is the small dense contraction
//     S^T[heads x blocks] = W^T[G x 256] * M^T[256 x nblk],
// done with v_mfma_f32_16x16x32_bf16: bf16 x bf16 products are exact in
// fp32 and accumulate in fp32.  The GQA heads fill the MFMA rows (padded to
// 16 with zero weights); each column is one block.
//
// HBM bounds it.  Each wave reads one tile of 16 consecutive metadata rows as
// whole contiguous 1 KiB pieces with the non-temporal cache policy, stages it
// in LDS and reads its MFMA B fragments from there; there is no cross-lane
// reduction, the head maximum is taken over accumulator registers.  Fragments
// loaded straight from HBM (each instruction covering 64-byte pieces of 16
// rows) reached 0.765 of the 8 TB/s peak on the 128k-token batch and got
// slower with the non-temporal policy, since a 128-byte line was then
// requested by two instructions; staged with the default policy 0.765 too.
//
// Workgroups are two waves of one tile each, so the last workgroups of a
// launch are short and a ragged batch leaves no CU with a long rest; seven of
// them a CU keep as many bytes in flight as the eight waves of double-buffered
// tiles, four tiles a wave, that this replaces.  Dispatch events, us, before
// and now: 64 sequences x 8 heads x 8192 blocks 330, 317 (6.8 TB/s); the same
// with 1024 to 8192 blocks 225, 176; 32 x 8 x 2048 blocks 41, 38.7; 11 x 4 x
// 1024 to 8192 24.2, 20.0; mean keys of 16 x 8 x 256 to 2048 11.0, 8.6; 2 x 2 x
// 256 5.0, 4.1.  Workgroups of one, four and eight such waves: 330, 330 and 341
// us for the first, 31.9, 32.4 and 41.4 against 31.4 for 20 x 8 x 512 to 4096.
// Giving each XCD runs of 512 KiB left the first at 317 and slowed the ragged
// ones to 205 and 42.
//
// Workgroups go to the XCDs in turn, so with the chunks of a row in their own
// order and a power of two of them a row, one chunk of every row meets one XCD,
// and what ragged rows leave out is left out on the same XCDs.  Rows of up to
// 512 KiB of metadata therefore take their chunks in an order that differs from
// row to row (spread(), a multiplicative hash), for cuboids from one run of 32
// rows to the next.  Plain order and this, us: 512 sequences x 8 heads x 64 to
// 512 blocks 118, 93; 128 x 8 x 128 to 1024 55.5, 47.6; mean keys of 512 x 8 x
// 128 to 1024 129, 96.5.  Equal rows are best read with each XCD in a part of
// memory of its own, which a run keeps: 1024 x 8 x 512 319, 321, but 337 with an
// order a row, and 163 against 160 for 256 x 8 x 1024.  Mean keys pay 0 to 5%
// with an order a row and up to 7% with runs (2048 rows of 128), which also even
// out their ragged rows less.  In longer rows the XCDs even out by themselves
// (0 to 8% gained) and equal ones pay 3 to 6%; rows of an odd number of chunks
// never meet the XCDs in step.
//
// Short rows by the hundred are bound by the workgroups that start, not by
// HBM: one workgroup of four waves takes a whole row of up to 256 blocks, a
// tile a wave at a time (wide()).  Rows of 33 to 64 blocks gain from 192 rows
// on (two waves a workgroup and this, us: 32 x 8 x 48 3.5, 3.1; 128 rows 2.8,
// 2.9), mean keys, whose rows take half the bytes, from 6144 rows on up to 256
// blocks (6 to 8% at 8192 rows of 65, 0 to 6% at 192, 3% lost to 1% gained at
// 250; with 2048 rows 0 to 16% lost).  Cuboid rows of 65 blocks and more are
// bound by HBM and up to 30% slower so.
#include "score_tile.hpp"

namespace {

constexpr int TILE = ss::kTile;
constexpr int WAVES = 2, WIDE_WAVES = 4;  // waves of a workgroup
constexpr int WIDE_TILES = 4;             // tiles of a wave in a wide workgroup, one otherwise
constexpr int BLOCKS_PER_WG = TILE * WAVES, BLOCKS_PER_WIDE = TILE * WIDE_WAVES * WIDE_TILES;
constexpr int kSpreadBytes = 512 * 1024;
// runs of 16 rows: equal rows up to 6% slower; of 64: ragged ones lose up to half the gain
constexpr int kRunLog2 = 5;
// Cuboid workgroups take 16.5 KiB of LDS, nine to a CU.  A launch that does
// not fit at once reserves 22 KiB for each, seven to a CU: 64 x 8 x 8192 blocks
// 317 us against 322, 32 x 8 x 8192 155 against 159 (six: 314 and 153, but 7.2
// us against 6.5 for one sequence and 32.5 against 31.7 for 20 ragged ones).
// Mean-key rows are half as long and launch with no reservation.
constexpr size_t kResidencyLds = 22 * 1024;
constexpr int kResident = 9 * 256;
constexpr size_t kStageBytes = (size_t)WAVES * ss::tile_shape<0>::STAGE * 16;

// Whether a workgroup of four waves takes a row.
bool wide(int meta_kind, int64_t units, int nblk_max)
{
    if (nblk_max <= BLOCKS_PER_WG) return false;
    return units >= 192 && nblk_max <= 2 * BLOCKS_PER_WG ||
           meta_kind == SS_META_MEAN && units >= 6144 && nblk_max <= BLOCKS_PER_WIDE;
}

// The bits of a chunk's number that differ from row to row: a permutation of
// the row's chunks, since they come in whole groups of that many.
int spread(int meta_kind, int chunks)
{
    const int bytes = BLOCKS_PER_WG * (meta_kind == SS_META_CUBOID ? ss::tile_shape<0>::ROW : ss::tile_shape<1>::ROW);
    return chunks <= kSpreadBytes / bytes ? (chunks & -chunks) - 1 : 0;
}

// Division of 0 <= x < 2^31 by d, as a multiplication: with 2^(s-1) < d <= 2^s
// and d*mul = 2^(31+s) + e, 0 <= e < 2^s, x*mul / 2^(31+s) exceeds x/d by less
// than 1/d.  There is no instruction for it, and two divisions at the head of
// every workgroup cost small calls up to 6% (mean keys of 64 to 128 rows of 48).
struct Divisor {
    uint32_t mul, shift;
    explicit Divisor(int d) : shift(0)
    {
        while ((1ll << shift) < d) ++shift;
        mul = (uint32_t)(((1ull << (31 + shift)) + d - 1) / d);
    }
    __device__ int divide(int x) const { return __umulhi(2u * x, mul) >> shift; }
};

template <int KIND, int AGG, int NW, int NT>
__global__ __launch_bounds__(NW * 64) void score_kernel(const uint16_t *__restrict__ q,
                                                        const uint8_t *__restrict__ meta,
                                                        const int32_t *__restrict__ nblk, int u0, int Hq, int Hkv,
                                                        Divisor by_hkv, int G, int nblk_max, int chunks_per_unit,
                                                        Divisor by_chunks, int spread, float *__restrict__ scores)
{
    __shared__ uint4 stage[NW][ss::tile_shape<KIND>::STAGE];
    const int uc = by_chunks.divide(blockIdx.x);
    const int u = u0 + uc;
    const uint32_t run = (uint32_t)uc >> (KIND == 0 ? kRunLog2 : 0);  // rows that share an order
    const int chunk = (blockIdx.x - uc * chunks_per_unit) ^ ((run * 0x9E3779B1u >> 16) & spread);
    const int b = by_hkv.divide(u), g = u - b * Hkv;
    int n = nblk[b];
    n = n < 0 ? 0 : (n > nblk_max ? nblk_max : n);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int j0 = chunk * (TILE * NW * NT) + wave * TILE;
#pragma unroll
    for (int t = 0; t < NT; ++t, j0 += TILE * NW) {
        if (j0 >= n) return;
        const float v = ss::score_tile<KIND, AGG>(q, meta, b, g, u, n, j0, Hq, G, nblk_max, stage[wave]);
        if (lane < TILE && j0 + lane < n) scores[(int64_t)u * nblk_max + j0 + lane] = v;
    }
}

template <int NW, int NT>
auto pick(int meta_kind, int agg)
{
    if (meta_kind == SS_META_CUBOID) return agg == SS_AGG_MAX ? score_kernel<0, 0, NW, NT> : score_kernel<0, 1, NW, NT>;
    return agg == SS_AGG_MAX ? score_kernel<1, 0, NW, NT> : score_kernel<1, 1, NW, NT>;
}

}  // namespace

namespace ss {

ss_status launch_score(const void *q, const void *meta, int meta_kind, int agg, const int32_t *nblk, int B, int Hq,
                       int Hkv, int nblk_max, float *scores, hipStream_t s)
{
    const int64_t units = (int64_t)B * Hkv;
    const bool w = wide(meta_kind, units, nblk_max);
    const int blocks = w ? BLOCKS_PER_WIDE : BLOCKS_PER_WG, threads = (w ? WIDE_WAVES : WAVES) * 64;
    const int chunks = (nblk_max + blocks - 1) / blocks;
    if (units * chunks == 0) return SS_OK;
    // what one launch of 256 threads per 256 blocks holds is taken; these
    // shorter workgroups may need several launches for it
    SS_CHECK_SUPPORTED(units * ((nblk_max + 255) / 256) <= 0xFFFFFFFFll / 256, "score: grid too large");
    const int64_t per = 0xFFFFFFFFll / threads / chunks;  // units per launch
    const auto *qq = static_cast<const uint16_t *>(q);
    const auto *mm = static_cast<const uint8_t *>(meta);
    const int G = Hq / Hkv;
    auto *kernel = w ? pick<WIDE_WAVES, WIDE_TILES>(meta_kind, agg) : pick<WAVES, 1>(meta_kind, agg);
    for (int64_t u0 = 0; u0 < units; u0 += per) {
        const int64_t grid = (units - u0 < per ? units - u0 : per) * chunks;
        const bool cap = !w && meta_kind == SS_META_CUBOID && grid > kResident;
        ss::launch_lds(kernel, dim3((unsigned)grid), dim3(threads), cap ? kResidencyLds - kStageBytes : 0, s, qq, mm,
                       nblk, (int)u0, Hq, Hkv, Divisor(Hkv), G, nblk_max, chunks, Divisor(chunks),
                       spread(meta_kind, chunks), scores);
    }
    return check_launch("ss_score_blocks");
}

ss_status check_score_args(const void *q, const void *meta, const int32_t *nblk, int B, int Hq, int Hkv,
                           int nblk_max, int d, const void *scores, const char *who, int meta_kind, int agg)
{
    SS_CHECK_ARG(meta_kind == SS_META_CUBOID || meta_kind == SS_META_MEAN, "%s: metadata kind %d", who, meta_kind);
    SS_CHECK_ARG(agg == SS_AGG_MAX || agg == SS_AGG_SUM, "%s: aggregation %d", who, agg);
    SS_CHECK_ARG(B >= 0 && Hq > 0 && Hkv > 0 && nblk_max >= 0, "%s: bad shape B=%d Hq=%d Hkv=%d nblk_max=%d", who, B,
                 Hq, Hkv, nblk_max);
    SS_CHECK_ARG(Hq % Hkv == 0, "%s: Hq=%d not a multiple of Hkv=%d", who, Hq, Hkv);
    SS_CHECK_SUPPORTED(Hq / Hkv <= kMaxGroup, "%s: group size %d > %d", who, Hq / Hkv, kMaxGroup);
    SS_CHECK_SUPPORTED(d == kHeadDim, "%s: d=%d (only 128)", who, d);
    SS_CHECK_SUPPORTED(nblk_max <= kMaxBlocks, "%s: nblk_max=%d > %d", who, nblk_max, kMaxBlocks);
    if ((int64_t)B * nblk_max > 0) SS_CHECK_ARG(q && meta && nblk && scores, "%s: null pointer", who);
    return SS_OK;
}

}  // namespace ss

extern "C" ss_status ss_score_blocks(const void *q, const void *meta, const int32_t *nblk, int B, int Hq, int Hkv,
                                     int nblk_max, int d, float *scores, void *stream)
{
    return ss_score_blocks_variant(q, meta, SS_META_CUBOID, SS_AGG_MAX, nblk, B, Hq, Hkv, nblk_max, d, scores,
                                   stream);
}

extern "C" ss_status ss_score_blocks_variant(const void *q, const void *meta, int meta_kind, int agg,
                                             const int32_t *nblk, int B, int Hq, int Hkv, int nblk_max, int d,
                                             float *scores, void *stream)
{
    ss_status st = ss::check_score_args(q, meta, nblk, B, Hq, Hkv, nblk_max, d, scores, "ss_score_blocks", meta_kind,
                                        agg);
    if (st != SS_OK) return st;
    return ss::launch_score(q, meta, meta_kind, agg, nblk, B, Hq, Hkv, nblk_max, scores, ss::as_stream(stream));
}
