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
#include "score_tile.hpp"

namespace {

constexpr int TILE = ss::kTile;  // one tile per wave
constexpr int WAVES = 2;
constexpr int BLOCKS_PER_WG = TILE * WAVES;
// Cuboid workgroups take 16.5 KiB of LDS, nine to a CU.  A launch that does
// not fit at once reserves 22 KiB for each, seven to a CU: 64 x 8 x 8192 blocks
// 317 us against 322, 32 x 8 x 8192 155 against 159 (six: 314 and 153, but 7.2
// us against 6.5 for one sequence and 32.5 against 31.7 for 20 ragged ones).
// Mean-key rows are half as long and launch with no reservation.
constexpr size_t kResidencyLds = 22 * 1024;
constexpr int kResident = 9 * 256;
constexpr size_t kStageBytes = (size_t)WAVES * ss::tile_shape<0>::STAGE * 16;

template <int KIND, int AGG>
__global__ __launch_bounds__(WAVES * 64) void score_kernel(const uint16_t *__restrict__ q,
                                                           const uint8_t *__restrict__ meta,
                                                           const int32_t *__restrict__ nblk, int u0, int Hq, int Hkv,
                                                           int G, int nblk_max, int chunks_per_unit,
                                                           float *__restrict__ scores)
{
    __shared__ uint4 stage[WAVES][ss::tile_shape<KIND>::STAGE];
    const int uc = blockIdx.x / chunks_per_unit;
    const int u = u0 + uc, chunk = blockIdx.x - uc * chunks_per_unit;
    const int b = u / Hkv, g = u - b * Hkv;
    int n = nblk[b];
    n = n < 0 ? 0 : (n > nblk_max ? nblk_max : n);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = chunk * BLOCKS_PER_WG + wave * TILE;
    if (j0 >= n) return;

    const int lane = threadIdx.x & 63;
    const float v = ss::score_tile<KIND, AGG>(q, meta, b, g, u, n, j0, Hq, G, nblk_max, stage[wave]);
    if (lane < TILE && j0 + lane < n) scores[(int64_t)u * nblk_max + j0 + lane] = v;
}

}  // namespace

namespace ss {

ss_status launch_score(const void *q, const void *meta, int meta_kind, int agg, const int32_t *nblk, int B, int Hq,
                       int Hkv, int nblk_max, float *scores, hipStream_t s)
{
    const int chunks = (nblk_max + BLOCKS_PER_WG - 1) / BLOCKS_PER_WG;
    const int64_t units = (int64_t)B * Hkv;
    if (units * chunks == 0) return SS_OK;
    // what one launch of 256 threads per 256 blocks holds is taken; these
    // shorter workgroups may need several launches for it
    SS_CHECK_SUPPORTED(units * ((nblk_max + 255) / 256) <= 0xFFFFFFFFll / 256, "score: grid too large");
    const int64_t per = 0xFFFFFFFFll / (WAVES * 64) / chunks;  // units per launch
    const auto *qq = static_cast<const uint16_t *>(q);
    const auto *mm = static_cast<const uint8_t *>(meta);
    const dim3 bl(WAVES * 64);
    const int G = Hq / Hkv;
    auto *kernel = score_kernel<0, 0>;
    if (meta_kind == SS_META_CUBOID) kernel = agg == SS_AGG_MAX ? score_kernel<0, 0> : score_kernel<0, 1>;
    else kernel = agg == SS_AGG_MAX ? score_kernel<1, 0> : score_kernel<1, 1>;
    for (int64_t u0 = 0; u0 < units; u0 += per) {
        const int64_t grid = (units - u0 < per ? units - u0 : per) * chunks;
        const bool cap = meta_kind == SS_META_CUBOID && grid > kResident;
        ss::launch_lds(kernel, dim3((unsigned)grid), bl, cap ? kResidencyLds - kStageBytes : 0, s, qq, mm, nblk, (int)u0,
                       Hq, Hkv, G, nblk_max, chunks, scores);
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
