// What reads K and V block by block before scoring and attention: block mean pooling of Q and K (pattern
// computation, step 1; Sec. 4.1.1 of the AngelSlim report: the dynamic regime first locates the sparse
// regions), the value magnitudes of the output-aware score, and V transposed per block for the attention
// kernel.  One kernel for each entry point that asks for one of them, and prepare_kv_kernel, which does what a
// fused (or output-aware select) call needs of K and V in one launch.
//
// Pooling is a pure HBM stream: every bf16 element of Q and K is read exactly once with
// 16-byte loads, one workgroup per (head, block).  A row of head_dim elements is
// covered by head_dim/8 adjacent lanes, so each wave instruction reads whole
// contiguous rows.  Partial sums are fp32; the 16 (or 32) row groups of a
// workgroup are combined through LDS in a fixed order, so results are
// deterministic.
#include "common.hpp"
#include "value_block.hpp"

namespace spa {
namespace {

// One block of one head: mean of its tokens.  src: the block's first token; n_valid: its tokens that exist; part:
// 256 / (D / 8) rows of D floats of LDS.
// layout: pooled K goes out in the operand layout of the score kernel (key_tile_offset) or row
// major fp32; in the former a wavefront of that kernel reads whole 1-KB pieces that are its
// MFMA operands as they are.  dst is then the block's tile, otherwise the block's row.
template <int D, int BS>
__device__ __forceinline__ void pool_block(const uint16_t* __restrict__ src, int64_t stride_t, int n_valid, float (*part)[D],
                                           float* __restrict__ dst, KeyLayout layout, int blk) {
    constexpr int TPR = D / 8;          // lanes per token row
    constexpr int RPP = 256 / TPR;      // token rows per pass
    constexpr int PASSES = BS / RPP;
    const int tid = threadIdx.x;
    const int row0 = tid / TPR, chunk = tid % TPR;

    // the last block of a sequence may be partial: tokens past the end are not read
    uint4 raw[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        raw[p] = make_uint4(0u, 0u, 0u, 0u);
        if (p * RPP + row0 < n_valid)
            raw[p] = stream_load16(src + (int64_t)(p * RPP + row0) * stride_t + chunk * 8);
    }
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        acc[0] += bf16_lo(raw[p].x); acc[1] += bf16_hi(raw[p].x);
        acc[2] += bf16_lo(raw[p].y); acc[3] += bf16_hi(raw[p].y);
        acc[4] += bf16_lo(raw[p].z); acc[5] += bf16_hi(raw[p].z);
        acc[6] += bf16_lo(raw[p].w); acc[7] += bf16_hi(raw[p].w);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[row0][chunk * 8 + e] = acc[e];
    __syncthreads();
    if (tid < D) {
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < RPP; ++r) s += part[r][tid];
        const float mean = n_valid == BS ? s * (1.0f / (float)BS) : s / (float)n_valid;
        if (layout != kKeyRows) {
            const __bf16 hi = (__bf16)mean;                       // round to nearest even, twice
            const __bf16 lo = (__bf16)(mean - (float)hi);
            __bf16* t = reinterpret_cast<__bf16*>(dst);
            const int at = key_tile_offset(layout, tid, blk);
            t[at] = hi;
            t[at + key_tail(layout)] = lo;
        } else {
            dst[tid] = mean;
        }
    }
}
// where pooled K block blk of head hy goes
template <int D>
__device__ __forceinline__ float* pooled_k(float* kp, int hy, int blk, int NBk, KeyLayout layout) {
    return layout != kKeyRows ? kp + ((int64_t)hy * ((NBk + 31) >> 5) + (blk >> 5)) * (32 * D) : kp + ((int64_t)hy * NBk + blk) * D;
}

template <int D, int BS>
__global__ __launch_bounds__(256) void pool_kernel(const uint16_t* __restrict__ q, Strides qs,
                                                   int n_q_rows /* B*Hq or 0 */, int Hq,
                                                   const uint16_t* __restrict__ k, Strides ks, int Hkv,
                                                   float* __restrict__ qp, float* __restrict__ kp, int NBq, int Sq,
                                                   int NBk, int Skv, KeyLayout k_layout,
                                                   const int32_t* __restrict__ seq_lens) {
    __shared__ float part[256 / (D / 8)][D];
    const int blk = blockIdx.x;
    int hy = blockIdx.y;
    // Each tensor has a branch of its own: with the operands selected first, a workgroup waits for both tensors' arguments
    // before its first load, which shows where blocks are small (111232 + 2511 tokens of 8 / 1 heads, head_dim 64, blocks of 64:
    // 8.4 -> 7.0 us).
    if (hy < n_q_rows) {
        const int b = hy / Hq, h = hy % Hq;
        const int S = entry_len(seq_lens, b, Sq);            // ragged batch: this entry's own length
        if (blk * BS >= S) return;                           // the grid spans the key blocks of the longest entry
        pool_block<D, BS>(q + b * qs.b + h * qs.h + (int64_t)blk * BS * qs.t, qs.t, S - blk * BS < BS ? S - blk * BS : BS, part,
                          qp + ((int64_t)hy * NBq + blk) * D, kKeyRows, blk);
    } else {
        hy -= n_q_rows;
        const int b = hy / Hkv, h = hy % Hkv;
        const int S = Skv - Sq + entry_len(seq_lens, b, Sq); // K may carry a prefix
        if (blk * BS >= S) return;
        pool_block<D, BS>(k + b * ks.b + h * ks.h + (int64_t)blk * BS * ks.t, ks.t, S - blk * BS < BS ? S - blk * BS : BS, part,
                          pooled_k<D>(kp, hy, blk, NBk, k_layout), k_layout, blk);
    }
}

template <int D, int BS>
hipError_t launch(const Dims& d, const void* q, Strides qs, const void* k, Strides ks, float* qp,
                  float* kp, KeyLayout k_layout, hipStream_t st) {
    int nq = q ? d.B * d.Hq : 0, nk = k ? d.B * d.Hkv : 0;
    if (nq + nk == 0) return hipSuccess;
    dim3 grid(nk ? d.NBk : d.NB, nq + nk);
    hipLaunchKernelGGL((pool_kernel<D, BS>), grid, dim3(256), 0, st, (const uint16_t*)q, qs, nq, d.Hq,
                       (const uint16_t*)k, ks, d.Hkv, qp, kp, d.NB, d.S, d.NBk, d.Skv, k_layout, d.seq_lens);
    return hipGetLastError();
}

template <int D, int BS>
__global__ __launch_bounds__(256) void vnorm_kernel(const uint16_t* __restrict__ v, Strides vs, int Hkv, int NB,
                                                    int S, float* __restrict__ lvn,
                                                    const int32_t* __restrict__ seq_lens, int Sq) {
    __shared__ float part[256 / (D / 8)];
    const int blk = blockIdx.x, hy = blockIdx.y;
    const int b = hy / Hkv, h = hy % Hkv;
    S = S - Sq + entry_len(seq_lens, b, Sq);                        // ragged batch: key tokens of this entry
    if (blk * BS >= S) return;
    value_block<D, BS, false, true>(threadIdx.x, v + b * vs.b + h * vs.h + (int64_t)blk * BS * vs.t, vs.t,
                                    S - blk * BS < BS ? S - blk * BS : BS, nullptr, part, nullptr, false, lvn + (int64_t)hy * NB + blk);
}

// V [B,Hkv,S,D] (strided) -> Vt [B,Hkv,vt_bph,D,BS] contiguous, blocks first .. first + gridDim.x - 1.
// vt_bph: blocks per head in the V^T allocation (>= the key blocks of the call); first: first block to do
template <int D, int BS>
__global__ __launch_bounds__(256) void transpose_v_kernel(const uint16_t* __restrict__ v, Strides vs, int Hkv,
                                                          int64_t vt_bph, int S, uint16_t* __restrict__ vt,
                                                          const int32_t* __restrict__ seq_lens, int Sq, int first, int halves) {
    __shared__ uint16_t tile[BS * (D + 2)];
    const int blk = first + blockIdx.x, bh = blockIdx.y;
    const int b = bh / Hkv, h = bh % Hkv;
    const int Sb = S - Sq + entry_len(seq_lens, b, Sq);    // ragged batch: key tokens of this entry
    if (blk * BS >= Sb) return;                            // block past its end: never read by the attention kernel
    value_block<D, BS, true, false>(threadIdx.x, v + b * vs.b + h * vs.h + (int64_t)blk * BS * vs.t, vs.t, Sb - blk * BS < BS ? Sb - blk * BS : BS,
                                    tile, nullptr, vt + ((int64_t)bh * vt_bph + blk) * D * BS, halves, nullptr);
}

// Everything a call needs of K and V before it scores: blockIdx.z = 0 pools a block of K, 1 takes a
// block of V (VT: transposed for the attention kernel, VN: its magnitude), 2 + g pools a block of query head g of the KV
// group, where the score kernel does not do that itself.  HBM-bound streams like the separate kernels,
// whose launches, ramps and second read of V this saves: fused calls of 512 tokens 27 -> 23 us, 1999 tokens 64 -> 57.6,
// 16384 tokens (D = 64, shared lists) 557 -> 553 us; 49000 tokens with the output-aware score 3.59 -> 3.51 ms.
template <int D, int BS, bool VT, bool VN>
__global__ __launch_bounds__(256) void prepare_kv_kernel(const uint16_t* __restrict__ k, Strides ks,
                                                         const uint16_t* __restrict__ v, Strides vs, int Hkv, int NBk, int Skv,
                                                         float* __restrict__ kp, uint16_t* __restrict__ vt,
                                                         float* __restrict__ lvn, const int32_t* __restrict__ seq_lens, int Sq,
                                                         int halves, KeyLayout k_layout, const uint16_t* __restrict__ q, Strides qs,
                                                         float* __restrict__ qp, int NBq) {
    constexpr int RPP = 256 / (D / 8);
    constexpr int TILE_B = VT ? BS * (D + 2) * 2 : 0, PART_B = RPP * D * 4;
    __shared__ __attribute__((aligned(16))) char lds[TILE_B > PART_B ? TILE_B : PART_B];
    __shared__ float norms[RPP];
    const int blk = blockIdx.x, hy = blockIdx.y;
    const int b = hy / Hkv, h = hy % Hkv;
    if (blockIdx.z >= 2) {                                 // a query head of the group
        const int Sb = entry_len(seq_lens, b, Sq), G = (int)gridDim.z - 2, g = (int)blockIdx.z - 2;
        if (blk * BS >= Sb) return;
        pool_block<D, BS>(q + b * qs.b + (h * G + g) * qs.h + (int64_t)blk * BS * qs.t, qs.t, Sb - blk * BS < BS ? Sb - blk * BS : BS,
                          reinterpret_cast<float(*)[D]>(lds), qp + (((int64_t)hy * G + g) * NBq + blk) * D, kKeyRows, blk);
        return;
    }
    const int S = Skv - Sq + entry_len(seq_lens, b, Sq);   // ragged batch: key tokens of this entry
    if (blk * BS >= S) return;
    const int n_valid = S - blk * BS < BS ? S - blk * BS : BS;
    if (blockIdx.z == 0)
        pool_block<D, BS>(k + b * ks.b + h * ks.h + (int64_t)blk * BS * ks.t, ks.t, n_valid, reinterpret_cast<float(*)[D]>(lds),
                          pooled_k<D>(kp, hy, blk, NBk, k_layout), k_layout, blk);
    else
        value_block<D, BS, VT, VN>(threadIdx.x, v + b * vs.b + h * vs.h + (int64_t)blk * BS * vs.t, vs.t, n_valid,
                                   reinterpret_cast<uint16_t*>(lds), norms, VT ? vt + ((int64_t)hy * NBk + blk) * D * BS : nullptr, halves,
                                   VN ? lvn + (int64_t)hy * NBk + blk : nullptr);
}

template <int D, int BS>
hipError_t launch_vn(const Dims& d, const void* v, Strides vs, float* lvn, hipStream_t st) {
    dim3 grid(d.NBk, d.B * d.Hkv);
    hipLaunchKernelGGL((vnorm_kernel<D, BS>), grid, dim3(256), 0, st, (const uint16_t*)v, vs, d.Hkv, d.NBk, d.Skv, lvn, d.seq_lens, d.S);
    return hipGetLastError();
}

template <int D, int BS>
hipError_t launch_tv(const Dims& d, const void* v, Strides vs, void* vt, int64_t vt_bph, int first, int n, bool halves, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((transpose_v_kernel<D, BS>), dim3(n, d.B * d.Hkv), dim3(256), 0, st,
                       (const uint16_t*)v, vs, d.Hkv, vt_bph, d.Skv, (uint16_t*)vt, d.seq_lens, d.S, first, halves ? 1 : 0);
    return hipGetLastError();
}

template <int D, int BS>
hipError_t launch_prep(const Dims& d, const void* q, Strides qs, float* qp, const void* k, Strides ks, const void* v, Strides vs,
                       float* kp, KeyLayout k_layout, void* vt, float* lvn, hipStream_t st) {
    const auto kernel = vt == nullptr ? prepare_kv_kernel<D, BS, false, true>
                                      : (lvn == nullptr ? prepare_kv_kernel<D, BS, true, false> : prepare_kv_kernel<D, BS, true, true>);
    hipLaunchKernelGGL(kernel, dim3(d.NBk, d.B * d.Hkv, qp == nullptr ? 2 : 2 + d.G), dim3(256), 0, st, (const uint16_t*)k, ks,
                       (const uint16_t*)v, vs, d.Hkv, d.NBk, d.Skv, kp, (uint16_t*)vt, lvn, d.seq_lens, d.S, vt_in_halves(d) ? 1 : 0,
                       k_layout, (const uint16_t*)q, qs, qp, d.NB);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_transpose_v(const Dims& d, const void* v, Strides vs, void* vt, int64_t vt_bph, int first, int n,
                              bool halves, hipStream_t st) {
    if (vt == nullptr || vt_bph < d.NBk || first < 0 || n < 0 || first + n > d.NBk) return hipErrorInvalidValue;
    if (d.D == 128 && d.Bs == 128) return launch_tv<128, 128>(d, v, vs, vt, vt_bph, first, n, halves, st);
    if (d.D == 128 && d.Bs == 64) return launch_tv<128, 64>(d, v, vs, vt, vt_bph, first, n, halves, st);
    if (d.D == 64 && d.Bs == 128) return launch_tv<64, 128>(d, v, vs, vt, vt_bph, first, n, halves, st);
    if (d.D == 64 && d.Bs == 64) return launch_tv<64, 64>(d, v, vs, vt, vt_bph, first, n, halves, st);
    return hipErrorInvalidValue;
}

hipError_t launch_prepare_kv(const Dims& d, const void* q, Strides qs, float* qp_or_null, const void* k, Strides ks, const void* v,
                             Strides vs, float* kp, KeyLayout k_layout, void* vt_or_null, float* lvn_or_null, hipStream_t st) {
    if (vt_or_null == nullptr && lvn_or_null == nullptr) return hipErrorInvalidValue;
    if (d.D == 128 && d.Bs == 128) return launch_prep<128, 128>(d, q, qs, qp_or_null, k, ks, v, vs, kp, k_layout, vt_or_null, lvn_or_null, st);
    if (d.D == 128 && d.Bs == 64) return launch_prep<128, 64>(d, q, qs, qp_or_null, k, ks, v, vs, kp, k_layout, vt_or_null, lvn_or_null, st);
    if (d.D == 64 && d.Bs == 128) return launch_prep<64, 128>(d, q, qs, qp_or_null, k, ks, v, vs, kp, k_layout, vt_or_null, lvn_or_null, st);
    if (d.D == 64 && d.Bs == 64) return launch_prep<64, 64>(d, q, qs, qp_or_null, k, ks, v, vs, kp, k_layout, vt_or_null, lvn_or_null, st);
    return hipErrorInvalidValue;
}

hipError_t launch_vnorm(const Dims& d, const void* v, Strides vs, float* lvn, hipStream_t st) {
    if (d.D == 128 && d.Bs == 128) return launch_vn<128, 128>(d, v, vs, lvn, st);
    if (d.D == 128 && d.Bs == 64) return launch_vn<128, 64>(d, v, vs, lvn, st);
    if (d.D == 64 && d.Bs == 128) return launch_vn<64, 128>(d, v, vs, lvn, st);
    if (d.D == 64 && d.Bs == 64) return launch_vn<64, 64>(d, v, vs, lvn, st);
    return hipErrorInvalidValue;
}

hipError_t launch_pool(const Dims& d, const void* q, Strides qs, const void* k, Strides ks,
                       float* qp, float* kp, KeyLayout k_layout, hipStream_t st) {
    if (d.D == 128 && d.Bs == 128) return launch<128, 128>(d, q, qs, k, ks, qp, kp, k_layout, st);
    if (d.D == 128 && d.Bs == 64) return launch<128, 64>(d, q, qs, k, ks, qp, kp, k_layout, st);
    if (d.D == 64 && d.Bs == 128) return launch<64, 128>(d, q, qs, k, ks, qp, kp, k_layout, st);
    if (d.D == 64 && d.Bs == 64) return launch<64, 64>(d, q, qs, k, ks, qp, kp, k_layout, st);
    return hipErrorInvalidValue;
}

}  // namespace spa
