// The scores of one 16-block tile by one wave, shared by the scoring kernel and
// the one that scores and selects short rows (see score.hip for the method).
#pragma once

#include "internal.hpp"

namespace ss {

constexpr int kTile = 16;                      // blocks per MFMA tile
constexpr int kMetaBufferFlags = 0x00020000;   // raw buffer descriptor word 3 for gfx9 (32-bit data)
constexpr int kMetaStream = 2;                 // cache policy of the metadata loads: non-temporal

template <int KIND>
struct tile_shape {
    static constexpr int NCH = KIND == 0 ? 8 : 4;        // MFMA steps (32 bf16 each) per row
    static constexpr int ROW = NCH * 4 * 16;             // bytes per metadata row
    static constexpr int NLD = kTile * ROW / 1024;       // 1 KiB loads per tile
    static constexpr int RU = ROW / 16;                  // 16-byte units per row
    // LDS row pitch in 16-byte units, padded so that each 16-lane group of a
    // fragment read touches 64 distinct banks
    static constexpr int LR = RU + 1;
    static constexpr int STAGE = kTile * LR;             // uint4 of LDS per wave
};

union frag_t {
    bf16x8_t v;
    uint4 u;
};

// Lane (L = lane/16, col = lane%16) reads 16-byte chunk c = 4*m + L of
// metadata row `col` of the staged tile for MFMA m.  The A fragments hold
// the matching weights of head `col`.
//
// KIND 0, cuboid rows [lo, hi] (512 B, NCH = 8): chunks 0..15 are lo and
// multiply min(q, 0), chunks 16..31 (m >= 4) are hi and multiply max(q, 0).
// KIND 1, mean-key rows (256 B, NCH = 4): each chunk multiplies q itself.
// AGG 0 takes the maximum over the group's heads, AGG 1 their sum.
// Blocks j0 .. j0+15 (j0 < n) of unit u = b*Hkv + g by the calling wave; `my`:
// tile_shape<KIND>::STAGE uint4 of LDS of its own.  Lane l returns the score
// of block j0 + l%16 (meaningless past n).
template <int KIND, int AGG>
__device__ __forceinline__ float score_tile(const uint16_t *__restrict__ q, const uint8_t *__restrict__ meta, int b,
                                            int g, int u, int n, int j0, int Hq, int G, int nblk_max, uint4 *my)
{
    typedef tile_shape<KIND> S;
    constexpr int D = kHeadDim;
    const int lane = threadIdx.x & 63;
    const int L = lane >> 4;
    const int col = lane & 15;

    // channel chunks of head g*G + col: 4*m + L for m < 4
    const bool live = col < G;
    const uint16_t *qh = q + ((int64_t)b * Hq + g * G + (live ? col : 0)) * D;
    uint4 x[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = *reinterpret_cast<const uint4 *>(qh + (4 * m + L) * 8);

    const uint8_t *mu = meta + (int64_t)u * nblk_max * S::ROW;
    // n * S::ROW <= kMaxBlocks * 512 bytes < 2^31
    const __amdgpu_buffer_rsrc_t mrs = __builtin_amdgcn_make_buffer_rsrc((void *)mu, (short)0, n * S::ROW, kMetaBufferFlags);
    uint4 r[S::NLD];
#pragma unroll
    for (int i = 0; i < S::NLD; ++i)  // rows at or past n read as zero (buffer bounds) and are not stored
        r[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                             mrs, (uint32_t)j0 * S::ROW + lane * 16 + i * 1024, 0, kMetaStream));
    // nothing is made of q before every row has been asked for, or the compiler
    // puts its wait for q in front of some of them: 3 to 11% slower
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 4; ++m) asm volatile("" : "+v"(x[m].x), "+v"(x[m].y), "+v"(x[m].z), "+v"(x[m].w));

    // weights of head g*G + col for chunks 4*m + L, selected branch-free with
    // masks on the 32-bit words (two bf16 each)
    frag_t w[S::NCH];
    {
        const uint32_t live_mask = live ? 0xFFFFFFFFu : 0u;
#pragma unroll
        for (int m = 0; m < S::NCH; ++m) {
            const bool hi_half = KIND == 0 && m >= 4;  // cuboid chunks 16..31 multiply hi
            uint32_t v[4] = {x[m & 3].x, x[m & 3].y, x[m & 3].z, x[m & 3].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t keep = live_mask;
                if (KIND == 0) {
                    const uint32_t neg = ((v[i] >> 15) & 0x00010001u) * 0xFFFFu;  // 0xFFFF per negative half
                    keep &= hi_half ? ~neg : neg;  // hi keeps max(q, 0), lo keeps min(q, 0)
                }
                v[i] &= keep;
            }
            w[m].u = make_uint4(v[0], v[1], v[2], v[3]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // ... and all of this is done before the first row is waited for

#pragma unroll
    for (int i = 0; i < S::NLD; ++i) {
        const int e = i * 64 + lane;
        my[(e / S::RU) * S::LR + e % S::RU] = r[i];
    }
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < S::NCH; ++m) {
        frag_t f;
        f.u = my[col * S::LR + 4 * m + L];
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m].v, f.v, acc, 0, 0, 0);
    }
    float s;
    if (AGG == 0) {
        s = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (L * 4 + i < G) s = fmaxf(s, acc[i]);
        s = fmaxf(s, __shfl_xor(s, 16));
        s = fmaxf(s, __shfl_xor(s, 32));
    } else {
        s = (acc[0] + acc[1]) + (acc[2] + acc[3]);  // padded heads hold exact zeros
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
    }
    return s;
}

}  // namespace ss
