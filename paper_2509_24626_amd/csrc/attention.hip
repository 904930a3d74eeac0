// Sparse decode attention over the selected KV blocks (Section 2.1's
// softmax(q K^T / sqrt(d)) V, restricted to the tokens of the top-k blocks
// chosen in Section 2.2).
//
// The G query heads that share a KV head make both products small dense
// contractions, run on MFMA with heads as the 16-wide N dimension (padded
// with zero queries).  A wave consumes 16 tokens (8 KiB of K and V) per
// step:
//   S^T[16 tok x 16 heads]  = K[16 tok x 128] * Q^T     4 x v_mfma_f32_16x16x32_bf16
//   O^T[128 ch x 16 heads] += V^T[128 x 16 tok] * P^T   8 x v_mfma_f32_16x16x16_bf16 (x2, hi/lo)
// The S^T accumulator leaves lane (L = lane/16, col = lane%16) holding head
// `col` for tokens 4L .. 4L+3, which is exactly the lane's B fragment of the
// 16x16x16 PV product, so P never moves between lanes.  The step's K rows
// are read as four contiguous 1 KiB loads and staged in the wave's LDS tile,
// from which the A fragments (channels m*32 + 8L .. +7 of row `col`) are
// read; loading the fragments directly (each instruction a 64-byte piece of
// 16 rows) measured 0.805 of the HBM peak on the 128k batch against 0.825.
// The V tile of a block record is stored channel-major, so each V^T
// fragment is one 8-byte load and each V load instruction reads 512
// contiguous bytes.
// Each wave keeps two steps in flight (the next step's loads are issued
// before the current step is computed).  K and V are read with raw buffer
// loads over the unit's cache region: a skipped entry gets an offset past
// the region's end, which the hardware answers with zeros, so the loads
// are unconditional and the compiler can wait for exactly one step's loads
// (a conditional load forces a wait for all outstanding loads).
//
// Softmax runs online in the exp2 domain with fp32 state per head; the
// accumulator rescale is skipped while no head's running maximum changes.
// P enters the PV product as a bf16 hi + lo pair, which keeps about 16
// significant bits of every probability.
//
// Work split: grid (unit, split); a workgroup of 4 or 8 waves owns a
// contiguous range of 16-token steps, waves take steps round-robin, the wave
// partials are merged in LDS in wave order (a wave's partial output takes the
// place of its K tile), and with several splits a second kernel merges the
// split partials in split order.  All merges run in a fixed order, so results
// do not depend on scheduling.  plan() says how waves and splits are chosen.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <unordered_map>

#include "internal.hpp"

namespace {

constexpr int D = ss::kHeadDim;
constexpr int TOK = 16;  // tokens per wave step
constexpr int CUS = 256;
constexpr int KPITCH = D * 2 / 16 + 1;  // LDS row pitch of a staged K tile, in 16-byte units

typedef short s16x4_t __attribute__((ext_vector_type(4)));
constexpr int kBufferFlags = 0x00020000;  // raw buffer descriptor word 3 for gfx9 (32-bit data)
// cache policy of the K/V loads: non-temporal (each record is read once per
// launch); measured 0.81 of the HBM peak for the 128k batch against 0.72
// with the default policy
constexpr int kStream = 2;

union frag8_t {  // 8 x bf16: A/B fragment of the 16x16x32 MFMA
    bf16x8_t v;
    uint4 u;
};

union frag4_t {  // 4 x bf16: A/B fragment of the 16x16x16 MFMA
    s16x4_t v;
    uint2 u;
    uint16_t h[4];
};

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

constexpr int kMaxSplits = 32;  // splits of a unit's steps

struct split_plan {
    int waves, splits, steps_per_split;
};

template <int BLK, int WAVES>
__global__ __launch_bounds__(WAVES * 64, WAVES == 4 ? 3 : WAVES / 4) void attn_kernel(const uint16_t *__restrict__ q, const uint8_t *__restrict__ kv,
                                                      const int64_t *__restrict__ region_off,
                                                      const int32_t *__restrict__ slots,
                                                      const int32_t *__restrict__ capacity, int slot_limit, int Hq,
                                                      int Hkv, int G, int k, float scale_log2, int steps_per_split,
                                                      float *__restrict__ out, float *__restrict__ ws)
{
    constexpr int64_t REC = 2LL * BLK * D * 2;
    __shared__ float sm_m[WAVES][16], sm_l[WAVES][16];
    // per wave: the K tile of its current step, then its partial output [16][D + 4]
    __shared__ __align__(16) unsigned char sm_wave[WAVES][16 * (D + 4) * 4];
    static_assert(TOK * KPITCH * 16 <= 16 * (D + 4) * 4, "the K tile fits the partial output's place");

    const int u = blockIdx.x, split = blockIdx.y, splits = gridDim.y;
    const int b = u / Hkv, g = u - b * Hkv;
    const int lane = threadIdx.x & 63;
    // wave-uniform, so per-step slot indices are scalar loads: a vector load
    // would make every step wait for the previous step's K/V loads (the
    // vector-memory counter completes in order)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int L = lane >> 4, col = lane & 15;
    const int nsteps = (int)(((int64_t)k * BLK + TOK - 1) / TOK);
    const int s_begin = split * steps_per_split;
    const int s_end = min(s_begin + steps_per_split, nsteps);

    // B fragments of S^T = K Q^T: head `col`, channels m*32 + 8L .. +7
    frag8_t qf[4];
    {
        const bool live = col < G;
        const uint16_t *qh = q + ((int64_t)b * Hq + g * G + (live ? col : 0)) * D + L * 8;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            uint4 x = *reinterpret_cast<const uint4 *>(qh + m * 32);
            qf[m].u = live ? x : make_uint4(0, 0, 0, 0);
        }
    }

    const uint8_t *ubase = kv + region_off[u];
    const int32_t *us = slots + (int64_t)u * k;
    // the unit's own slot count bounds its entries, so a slot past it can
    // never reach into the next unit's region (or past the cache)
    int nslot = slot_limit;
    if (capacity) {
        const int c = capacity[u];
        nslot = c < 0 ? 0 : (c < slot_limit ? c : slot_limit);
    }
    const uint32_t lim = (uint32_t)nslot * (uint32_t)REC;  // bytes of the region (< 2^31, host-checked)
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)ubase, (short)0, (int)lim,
                                                                          kBufferFlags);

    float mrun = -INFINITY, lrun = 0.f;
    f32x4_t o[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    struct step_t {
        uint4 kr[4];  // K rows 4i + L, channels 8col .. 8col+7
        frag4_t vf[8];
        bool vz;  // the lane's accumulator tokens 4L .. 4L+3 are selected
    };
    // token t of the unit's selected-token sequence -> (entry t / BLK, position t % BLK)
    auto load_step = [&](int st, step_t &x) {
        const int tv = st * TOK + L * 4;  // this lane's V^T / accumulator tokens
        // entries of the step (uniform): one, or two when BLK = 8
        const int e0 = (st * TOK) / BLK;
        const int s0 = e0 < k ? us[e0] : -1;
        const int s1 = (BLK == 8 && e0 + 1 < k) ? us[e0 + 1] : -1;
        const int sv = (BLK == 8 && L >= 2) ? s1 : s0;
        const bool live = st < s_end;  // steps past the range load zeros
        const bool vv = live && sv >= 0 && sv < nslot;
        // skipped entries read at `lim`, past the region: the loads return zeros.
        // K: load i reads token rows 4i .. 4i+3 of the step, 1 KiB contiguous
        // (whole 128-byte lines, so the non-temporal policy pays)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + L;
            const int sr = (BLK == 8 && r >= 8) ? s1 : s0;
            const bool vr = live && sr >= 0 && sr < nslot;
            const uint32_t ko = vr ? (uint32_t)sr * (uint32_t)REC + ((st * TOK + r) % BLK) * (D * 2) + col * 16 : lim;
            x.kr[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, ko, 0, kStream));
        }
        const uint32_t vo = vv ? (uint32_t)sv * (uint32_t)REC + BLK * D * 2 + (col * BLK + tv % BLK) * 2 : lim;
#pragma unroll
        for (int t = 0; t < 8; ++t)
            x.vf[t].v = __builtin_bit_cast(s16x4_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo + t * 16 * BLK * 2, 0, kStream));
        x.vz = vv;
    };
    auto compute_step = [&](const step_t &x) {
        // K rows through the wave's LDS tile into A fragments: row `col`,
        // channels m*32 + 8L .. +7 (the padded pitch keeps each 16-lane group
        // of a fragment read on 64 distinct banks)
        uint4 *kt = reinterpret_cast<uint4 *>(sm_wave[wave]);
#pragma unroll
        for (int i = 0; i < 4; ++i) kt[(4 * i + L) * KPITCH + col] = x.kr[i];
        f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int m = 0; m < 4; ++m)
            sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kt[col * KPITCH + 4 * m + L]),
                                                           qf[m].v, sacc, 0, 0, 0);
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = x.vz ? sacc[i] * scale_log2 : -INFINITY;
        float cm = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
        cm = fmaxf(cm, __shfl_xor(cm, 16));
        cm = fmaxf(cm, __shfl_xor(cm, 32));
        const float mnew = fmaxf(mrun, cm);
        float p[4], alpha = 1.f;
        if (mnew == -INFINITY) {
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = 0.f;
        } else {
            alpha = __builtin_amdgcn_exp2f(mrun - mnew);
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(z[i] - mnew);
        }
        if (__any(mnew != mrun)) {
#pragma unroll
            for (int t = 0; t < 8; ++t) o[t] *= alpha;
        }
        mrun = mnew;
        frag4_t ph, pl;
        float psum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            psum += p[i];
            const uint16_t hi = f32_to_bf16_rne(p[i]);
            ph.h[i] = hi;
            pl.h[i] = f32_to_bf16_rne(p[i] - bf16_to_f32(hi));
        }
        lrun = lrun * alpha + psum;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            o[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.vf[t].v, ph.v, o[t], 0, 0, 0);
            o[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.vf[t].v, pl.v, o[t], 0, 0, 0);
        }
    };

    // the prefetches are unconditional (a step past the end loads zeros) so
    // that every path has the same loads in flight and each compute waits
    // only for its own step
    step_t bufA, bufB;
    int st = s_begin + wave;
    load_step(st, bufA);
    for (; st < s_end; st += 2 * WAVES) {
        load_step(st + WAVES, bufB);
        compute_step(bufA);
        if (st + WAVES >= s_end) break;
        load_step(st + 2 * WAVES, bufA);
        compute_step(bufB);
    }
    lrun += __shfl_xor(lrun, 16);
    lrun += __shfl_xor(lrun, 32);

    // wave partials -> LDS; lane holds O^T[16t + 4L + i][col]
    if (L == 0) {
        sm_m[wave][col] = mrun;
        sm_l[wave][col] = lrun;
    }
    if (col < G) {
        float *o_row = reinterpret_cast<float *>(sm_wave[wave]) + col * (D + 4);
#pragma unroll
        for (int t = 0; t < 8; ++t) *reinterpret_cast<f32x4_t *>(o_row + 16 * t + L * 4) = o[t];
    }
    __syncthreads();

    for (int idx = threadIdx.x; idx < G * D; idx += blockDim.x) {
        const int h = idx / D, ch = idx - h * D;
        float M = sm_m[0][h];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sm_m[w][h]);
        float lsum = 0.f, osum = 0.f;
        if (M != -INFINITY) {
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const float sc = __builtin_amdgcn_exp2f(sm_m[w][h] - M);
                lsum += sc * sm_l[w][h];
                osum += sc * reinterpret_cast<const float *>(sm_wave[w])[h * (D + 4) + ch];
            }
        }
        if (splits == 1) {
            out[((int64_t)b * Hq + g * G + h) * D + ch] = lsum > 0.f ? osum / lsum : 0.f;
        } else {
            float *pp = ws + (((int64_t)u * splits + split) * G + h) * (D + 2);
            if (ch == 0) {
                pp[0] = M;
                pp[1] = lsum;
            }
            pp[2 + ch] = osum;
        }
    }
}

// two floats, aligned as one is (the workspace is the caller's)
typedef float f32x2_t __attribute__((ext_vector_type(2), aligned(4)));

// maximum over the wave, in every lane
__device__ __forceinline__ float wave_max(float x)
{
    auto step = [](float v, int y) { return fmaxf(v, __int_as_float(y)); };
    x = step(x, __builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));   // lane ^ 1
    x = step(x, __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xF, 0xF, false));   // lane ^ 2
    x = step(x, __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x141, 0xF, 0xF, false));  // mirrored in 8 lanes
    x = step(x, __builtin_amdgcn_mov_dpp(__float_as_int(x), 0x140, 0xF, 0xF, false));  // mirrored in 16 lanes
    const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]));
}

// One wave per (unit, head), two channels per lane, at most N splits.  The
// splits' maxima and sums are read side by side, one split per lane, together
// with the partials (none of the loads waits for another), and the weights go
// round as scalars.  Latency bounds it: 8 splits of 32 heads took 3.3 us with
// each thread walking the splits twice, 2.5 now; 12 splits of 308 heads 6.4
// and 4.6 (of which about 2 are the launch).
template <int N>
__global__ __launch_bounds__(64) void combine_kernel(const float *__restrict__ ws, int Hq, int Hkv, int G, int splits,
                                                     float *__restrict__ out)
{
    static_assert(kMaxSplits <= 64, "one split per lane");
    const int u = blockIdx.x, h = blockIdx.y, lane = threadIdx.x;
    const int b = u / Hkv, g = u - b * Hkv;
    const float *p = ws + ((int64_t)u * splits * G + h) * (D + 2);
    const int stride = G * (D + 2);
    // partials past the last split read as zero (buffer bounds): a clamped one,
    // weighted by 0, may be infinite, and selecting costs 0.2 us
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0,
                                                                          ((splits - 1) * stride + D + 2) * 4, kBufferFlags);
    f32x2_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        x[i] = __builtin_bit_cast(f32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (i * stride + 2 + 2 * lane) * 4, 0, 0));
    f32x2_t ml = {-INFINITY, 0.f};
    if (lane < splits) ml = *reinterpret_cast<const f32x2_t *>(p + lane * stride);
    const float M = wave_max(ml.x);
    // 0 past the last split, and everywhere if nothing is selected; no branch,
    // behind which the partials' loads would move and wait for M (0.35 us)
    const float w = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - M);
    const float wl = w * ml.y;
    float lsum = 0.f;
    f32x2_t osum = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float sc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), i));
        lsum += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wl), i));
        osum.x += sc * x[i].x;
        osum.y += sc * x[i].y;
    }
    f32x2_t y = {0.f, 0.f};
    if (lsum > 0.f) y = f32x2_t{osum.x / lsum, osum.y / lsum};
    *reinterpret_cast<f32x2_t *>(out + ((int64_t)b * Hq + g * G + h) * D + 2 * lane) = y;
}

// Waves of the workgroup that takes a whole unit: 8 where that is faster than
// 4, us with 4 and with 8.  More waves share a unit's steps, but each brings a
// partial to merge, and where the units fill the chip the steps share its
// bandwidth anyway.
//   - Below 8 steps the many heads' larger merge is shared by more threads: 1
//     step of 256 units, G = 16, blocks of 32 4.7, 4.4; but G = 1 3.6, 3.8.  5 and 6
//     steps are one round of 8 waves, two of 4 (1 unit, G = 1, blocks of 8 3.8, 3.6).
//   - From 8 steps on blocks of 8 and 16 tokens, whose loads are shorter, gain
//     with many heads (1 unit of 20 steps, G = 7, blocks of 8 6.3, 5.6; 160 units
//     equal), with few heads only for few units (G = 1, blocks of 8: 1 unit of 20
//     steps 6.2, 5.0; 16 7.0, 6.6; 128 equal, 256 9.5, 10.1); blocks of 32 lose 1 to 8%.
//   - From 384 to 511 units, two rounds of the CUs, long selections gain with
//     blocks of 32 (511 of 384 steps, G = 1 299, 288) and are equal otherwise;
//     short ones lose (448 of 32 steps, G = 4 20.4, 21.7).
int waves_of_one(int units, int steps, int G, int blk)
{
    if (units >= 384) return units < 512 && steps >= 96 ? 8 : 4;
    if (units > 256) return 4;
    if (steps < 8) {
        if (G >= 3) return G >= 7 || steps < 7 || blk == 32 ? 8 : 4;
        return steps >= 5 && steps <= 6 && blk < 32 && units <= 16 ? 8 : 4;
    }
    if (blk == 32 || steps == 8) return 4;  // 8 steps: two full rounds of 4 waves
    if (G >= 7) return 8;
    const int few = blk == 8 ? 128 : 64;
    return units <= (G >= 3 ? few : few / 8) ? 8 : 4;
}

// Splits per unit: those that take least time by this model.  Its constants
// (us, but for a common factor) are fitted so that the choices lose least
// against the best of all plans over 6126 shapes (1 to 1024 units, 1 to 512
// steps, G 1 to 16, every block size): 0.5% on average.  Two 4-wave workgroups
// per CU lose 9%, up to a factor of 2.5 (few units of long selections); the
// plan that gave units whole to 8 waves wherever it had won at 128 steps lost
// 3%, up to a factor of 1.6 (us, then and now: 320 units of 64 steps 33.3,
// 30.6; 112 of 64 15.1, 13.4; 448 of 32 21.9, 20.4).
//   - The chip's bandwidth: kStepHbm per step and workgroup in flight.
//   - The fullest CU: alone on it, a workgroup's 4 waves take a step each per
//     round, of kRound (kLoad more for every other workgroup in flight);
//     together, workgroups take kStep2 (two) or kStep3 per step each.
//   - The second launch, with the partials' way through memory.
// 24 steps at least, 4 a split; units * splits stays below 1024, which bounds
// the partials, and no more than `most` splits are taken, for which there is
// room.
split_plan plan(int units, int k, int blk, int G, int most)
{
    constexpr float kStepHbm = 0.000945f, kRound = 0.197f, kLoad = 0.00018f, kStep2 = 0.2835f, kStep3 = 0.3245f;
    constexpr float kMerge = 2.3f, kMergeSplit = 0.0077f, kMergeGroup = 0.00032f, kMergeHead = 0.00024f;
    const int steps = (int)(((int64_t)k * blk + TOK - 1) / TOK);
    int best = 1;
    float least = 0.f;
    for (int n = 1; n <= most && (n == 1 || (steps >= 24 && units * n < 1024 && 4 * n <= steps)); ++n) {
        const int sps = (steps + n - 1) / n;
        const float groups = (float)units * ((steps + sps - 1) / sps);  // workgroups: rounding may need fewer splits
        const float rounds = std::ceil(groups / CUS);
        const float cu = rounds == 1.f ? (float)((sps + 3) / 4 * 4) * (kRound + kLoad * groups)
                                       : sps * rounds * (rounds == 2.f ? kStep2 : kStep3);
        float cost = std::max(sps * groups * kStepHbm, cu);
        if (n > 1) cost += kMerge + kMergeSplit * (groups / units) + (kMergeGroup + kMergeHead * G) * groups;
        if (n == 1 || cost < least) {
            best = n;
            least = cost;
        }
    }
    const int sps = (steps + best - 1) / best;
    const int splits = (steps + sps - 1) / sps;
    return {splits == 1 ? waves_of_one(units, steps, G, blk) : 4, splits, sps};
}

// The splits a workspace must have room for: two 4-wave workgroups per CU of
// 16 steps or more each.  Callers bring that much whichever plan serves the
// shape; what is refused does not move with the plans.  A plan that wants more
// is cut to what the workspace holds, and the query asks for the larger of the
// two.  units * splits stays below 1024 (fewer than units + 512, with more
// than one split only below 512 units).
int least_splits(int units, int k, int blk)
{
    const int steps = (int)(((int64_t)k * blk + TOK - 1) / TOK);
    const int want = std::max(1, std::min((512 + units - 1) / units, steps / 16));
    const int sps = (steps + want - 1) / want;
    return (steps + sps - 1) / sps;
}

bool has_plan(int B, int Hq, int Hkv, int d, int blk, int k)
{
    return B > 0 && Hkv > 0 && Hq > 0 && Hq % Hkv == 0 && d == D && ss::supported_blk(blk) && k > 0;
}

// bytes of the partials of one split of every unit
size_t split_bytes(int B, int Hq) { return (size_t)B * Hq * (D + 2) * sizeof(float); }

}  // namespace

size_t ss::attention_workspace_least(int B, int Hq, int Hkv, int d, int blk, int k)
{
    if (!has_plan(B, Hq, Hkv, d, blk, k)) return 0;
    const int splits = least_splits(B * Hkv, k, blk);
    return splits > 1 ? splits * split_bytes(B, Hq) : 0;
}

extern "C" size_t ss_sparse_attention_workspace(int B, int Hq, int Hkv, int d, int blk, int k)
{
    if (!has_plan(B, Hq, Hkv, d, blk, k)) return 0;
    const int units = B * Hkv;
    const int splits = std::max(least_splits(units, k, blk), plan(units, k, blk, Hq / Hkv, kMaxSplits).splits);
    return splits > 1 ? splits * split_bytes(B, Hq) : 0;
}

extern "C" ss_status ss_sparse_attention(const void *q, const void *kv_base, const int64_t *region_off,
                                         const int32_t *slots, const int32_t *capacity, int32_t slot_limit, int B,
                                         int Hq, int Hkv, int d,
                                         int blk, int k, float scale, float *out, void *workspace, size_t ws_bytes,
                                         void *stream)
{
    SS_CHECK_ARG(B >= 0 && Hq > 0 && Hkv > 0 && k > 0, "ss_sparse_attention: bad shape B=%d Hq=%d Hkv=%d k=%d", B, Hq,
                 Hkv, k);
    SS_CHECK_ARG(Hq % Hkv == 0, "ss_sparse_attention: Hq=%d not a multiple of Hkv=%d", Hq, Hkv);
    SS_CHECK_SUPPORTED(Hq / Hkv <= ss::kMaxGroup, "ss_sparse_attention: group size %d > %d", Hq / Hkv, ss::kMaxGroup);
    SS_CHECK_SUPPORTED(d == D, "ss_sparse_attention: d=%d (only 128)", d);
    SS_CHECK_SUPPORTED(ss::supported_blk(blk), "ss_sparse_attention: blk=%d (8, 16 or 32)", blk);
    SS_CHECK_ARG(std::isfinite(scale), "ss_sparse_attention: scale not finite");
    if (B == 0) return SS_OK;
    SS_CHECK_ARG(q && kv_base && region_off && slots && out, "ss_sparse_attention: null pointer");
    SS_CHECK_SUPPORTED(slot_limit >= 0 && (int64_t)slot_limit * 2 * blk * D * 2 <= 0x7FFFFFFF,
                       "ss_sparse_attention: slot_limit=%d records exceed a 2 GiB region", slot_limit);
    const int units = B * Hkv;
    const size_t need = ss::attention_workspace_least(B, Hq, Hkv, d, blk, k);
    if (ws_bytes < need || (need && !workspace))
        return ss::fail(SS_ERR_OOM, "ss_sparse_attention: workspace %zu bytes < %zu", ws_bytes, need);
    const size_t room = workspace ? ws_bytes / split_bytes(B, Hq) : 0;
    const int G = Hq / Hkv;
    const split_plan sp = plan(units, k, blk, G, (int)std::min(room, (size_t)kMaxSplits));
    hipStream_t s = ss::as_stream(stream);
    const float scale_log2 = scale * 1.4426950408889634f;
    const dim3 grid(units, sp.splits);
    const uint16_t *qq = static_cast<const uint16_t *>(q);
    const uint8_t *kv = static_cast<const uint8_t *>(kv_base);
    float *ws = static_cast<float *>(workspace);
    const bool wide = sp.waves == 8;
    auto *kernel = wide ? attn_kernel<32, 8> : attn_kernel<32, 4>;
    if (blk == 8) kernel = wide ? attn_kernel<8, 8> : attn_kernel<8, 4>;
    else if (blk == 16) kernel = wide ? attn_kernel<16, 8> : attn_kernel<16, 4>;
    ss::launch(kernel, grid, dim3(sp.waves * 64), s, qq, kv, region_off, slots, capacity, slot_limit, Hq, Hkv, G, k,
               scale_log2, sp.steps_per_split, out, ws);
    ss_status st = ss::check_launch("ss_sparse_attention");
    if (st != SS_OK || sp.splits == 1) return st;
    // reads as many partials as there may be splits: 16 of them cost 2 splits of 88 units 0.6 us of 9.4
    auto *combine = combine_kernel<kMaxSplits>;
    if (sp.splits <= 4) combine = combine_kernel<4>;
    else if (sp.splits <= 8) combine = combine_kernel<8>;
    else if (sp.splits <= 16) combine = combine_kernel<16>;
    combine<<<dim3(units, G), dim3(64), 0, s>>>(ws, Hq, Hkv, G, sp.splits, out);
    return ss::check_launch("ss_sparse_attention(combine)");
}

// ------------------------------------------------- allocation-free variant
// The split partials of ss_sparse_attention_static live in this file-scope
// device array instead of a caller workspace.  Every supported shape fits:
// with more than one split, units * splits <= 1023 and G <= 16, so the partials
// take at most 1023 * 16 * (128 + 2) * 4 bytes.
// Host code never uses the array's name as an address: each device's copy
// is looked up once with hipGetSymbolAddress and that pointer is passed on.
namespace {
constexpr size_t kStaticScratchBytes = 9u << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::mutex g_scratch_mu;
std::unordered_map<int, void *> g_scratch_addr;  // by device

ss_status scratch_address(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return ss::fail(SS_ERR_HIP, "ss_sparse_attention_static: hipGetDevice: %s", hipGetErrorString(e));
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    auto it = g_scratch_addr.find(dev);
    if (it != g_scratch_addr.end()) {
        *out = it->second;
        return SS_OK;
    }
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        return ss::fail(SS_ERR_HIP, "ss_sparse_attention_static: hipGetSymbolAddress of the scratch array: %s",
                        hipGetErrorString(e));
    g_scratch_addr[dev] = p;
    *out = p;
    return SS_OK;
}
}  // namespace

extern "C" ss_status ss_sparse_attention_static(const void *q, const void *kv_base, const int64_t *region_off,
                                                const int32_t *slots, const int32_t *capacity, int32_t slot_limit,
                                                int B, int Hq, int Hkv, int d, int blk, int k, float scale,
                                                float *out, void *stream)
{
    // shapes the main entry point rejects are rejected there; this only sizes the partials
    const size_t need = ss_sparse_attention_workspace(B, Hq, Hkv, d, blk, k);
    if (need > kStaticScratchBytes)
        return ss::fail(SS_ERR_OOM, "ss_sparse_attention_static: %zu bytes of split partials exceed the %zu-byte "
                        "static scratch", need, kStaticScratchBytes);
    void *ws = nullptr;
    if (need) {
        ss_status st = scratch_address(&ws);
        if (st) return st;
    }
    return ss_sparse_attention(q, kv_base, region_off, slots, capacity, slot_limit, B, Hq, Hkv, d, blk, k, scale,
                               out, ws, need, stream);
}
