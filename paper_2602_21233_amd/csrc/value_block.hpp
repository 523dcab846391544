// One block of V, for the kernels that transpose V or take its magnitudes.
#pragma once
#include "common.hpp"

namespace spa {
namespace {

// One block of V of one head: transposed to [D][BS] (halves: [2][D][BS / 2]) at vt (VT), and / or the ln of the mean L2 norm of its value vectors
// to *lvn (VN: the value-magnitude term of the output-aware ranking score, Sec. 4.1.2 Fig. "Stem" (c)).  The
// access pattern of pool_block, V is read once for both.  Norms: D/8 adjacent lanes cover one token, combine their
// partial sums of squares with lane-xor exchanges, and the token norms of the 16 (or 32) row groups are added
// through LDS in a fixed order; a block of all-zero values gives -inf.  Tokens past the end: zeros in V^T, a norm of 0.
// tile: BS * (D + 2) values of LDS (VT), part: 256 / (D / 8) floats (VN).  tid: the thread's place among the 256 of this
// block; every thread of the workgroup has to come here (barrier).  n_valid <= 0: no block, nothing is read or written.
template <int D, int BS, bool VT, bool VN>
__device__ __forceinline__ void value_block(const int tid, const uint16_t* __restrict__ src, int64_t stride_t, int n_valid, uint16_t* tile,
                                            float* part, uint16_t* __restrict__ vt, bool halves, float* __restrict__ lvn) {
    constexpr int TPR = D / 8, RPP = 256 / TPR, PASSES = BS / RPP, PITCH = D + 2;
    const int row0 = tid / TPR, chunk = tid % TPR;
    uint4 raw[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        raw[p] = make_uint4(0u, 0u, 0u, 0u);
        if (p * RPP + row0 < n_valid)
            raw[p] = stream_load16(src + (int64_t)(p * RPP + row0) * stride_t + chunk * 8);
    }
    if constexpr (VT) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            uint32_t* dst = reinterpret_cast<uint32_t*>(&tile[(p * RPP + row0) * PITCH + chunk * 8]);   // PITCH even: 4-byte aligned
            dst[0] = raw[p].x; dst[1] = raw[p].y; dst[2] = raw[p].z; dst[3] = raw[p].w;
        }
    }
    if constexpr (VN) {
        float acc = 0.f;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const uint32_t w[4] = {raw[p].x, raw[p].y, raw[p].z, raw[p].w};
            float sq = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = bf16_lo(w[e]), hi = bf16_hi(w[e]);
                sq = fmaf(lo, lo, sq);
                sq = fmaf(hi, hi, sq);
            }
#pragma unroll
            for (int off = 1; off < TPR; off <<= 1) sq += __shfl_xor(sq, off);
            acc += sqrtf(sq);
        }
        if (chunk == 0) part[row0] = acc;
    }
    __syncthreads();
    if (n_valid <= 0) return;
    if constexpr (VN) {
        if (tid == 0) {
            float s = 0.f;
#pragma unroll
            for (int r = 0; r < RPP; ++r) s += part[r];
            *lvn = logf(n_valid == BS ? s * (1.0f / (float)BS) : s / (float)n_valid);
        }
    }
    if constexpr (VT) {
        constexpr int CPR = BS / 8;         // 16-byte chunks per output row
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int c = p * 256 + tid;    // 16-byte chunk of the output, in memory order
            int d = c / CPR, t0 = (c % CPR) * 8;
            if (halves) {                   // rows half as long, then the second half of the tokens
                constexpr int HC = CPR / 2;
                d = c / HC % D;
                t0 = c / HC / D * (BS / 2) + c % HC * 8;
            }
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = (uint32_t)tile[(t0 + 2 * e) * PITCH + d] | ((uint32_t)tile[(t0 + 2 * e + 1) * PITCH + d] << 16);
            *reinterpret_cast<uint4*>(vt + c * 8) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

}  // namespace
}  // namespace spa
