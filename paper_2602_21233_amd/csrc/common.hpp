// Shared declarations of the sparse-prefill HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sparse_prefill.h"

namespace spa {

constexpr int kMaxBlocks = 4096;  // NB limit: one score row must fit a wave's LDS slice

// Derived sizes every launcher needs.
struct Dims {
    int B, Hq, Hkv, G, S, D, Bs, NB, T;   // S, NB: query tokens / query blocks of the call
    int Skv, NBk, off;                    // key tokens, key blocks, block position of query block 0
    int ns, nl, k;
    int shared;                   // 1: block lists are per KV head (group-shared selection)
    int stride, n_dense, reach;   // strided static columns, dense bottom strip, reach of the strided columns (0 = off)
    float scale;
    int gamma_q16;                // cumulative-mass budget in 16-bit fixed point, -1 = none
    const int32_t* seq_lens;      // device array [B] of per-entry token counts (ragged batch), or nullptr
    int head_budgets;             // 1: the lists are made with budgets of each head's own (known of a fused call only)
    int row_budgets;              // 1: with budgets of each query block's own, at most k (known of a fused call only)
};

inline Dims dims_of(const spa_params& p) {
    Dims d;
    d.B = p.batch; d.Hq = p.n_q_heads; d.Hkv = p.n_kv_heads; d.G = p.n_q_heads / p.n_kv_heads;
    d.S = p.seq_len; d.D = p.head_dim; d.Bs = p.block_size; d.NB = (p.seq_len + p.block_size - 1) / p.block_size;   // the last block may be partial
    d.ns = p.n_sink_blocks; d.nl = p.n_local_blocks; d.k = p.top_k_blocks;
    d.off = p.kv_prefix_len / p.block_size; d.Skv = p.kv_prefix_len + p.seq_len; d.NBk = d.off + d.NB;
    d.shared = p.lists_per_kv_head != 0;
    d.stride = p.stride_blocks; d.n_dense = p.n_dense_q_blocks; d.reach = p.stride_reach_blocks;
    int64_t far = d.NBk - 1;
    if (d.reach > 0 && d.reach - 1 < far) far = d.reach - 1;
    int64_t t = (int64_t)d.ns + d.nl + d.k + (d.stride > 0 ? far / d.stride : 0);
    d.T = (int)((t < d.NBk && d.n_dense <= 0) ? t : d.NBk);
    d.scale = p.softmax_scale;
    d.gamma_q16 = -1;
    d.seq_lens = p.seq_lens;
    d.head_budgets = d.row_budgets = 0;
    return d;
}

// How V^T lies where the library keeps it to itself (the workspace of the attention and fused calls): [2][D][Bs / 2], the
// two halves of a block's tokens one after the other, where the attention kernel loads a half block at a time and
// gains from finding it in one piece: blocks of 64 tokens in attn_chunked_kernel (429 -> 397 us at 16384 tokens)
// and, a little, head_dim 64 with blocks of 128 (fused calls of 300 tokens 16.6 -> 16.3 us, of 2048 queries over 98304 tokens of 8 / 1
// heads 120.7 -> 119.7; 538 us either way at 16384 tokens.  head_dim 128: 1.95 ms either way at 32768 tokens).  Everything
// else, and every V^T that a caller sees, is [D][Bs].
inline bool vt_in_halves(const Dims& d) { return d.Bs == 64 ? !(d.shared && d.G % 2 == 0) : d.D == 64; }

// Ragged batch: tokens of batch entry b (the tensors keep their padded length S)
__device__ __forceinline__ int entry_len(const int32_t* __restrict__ seq_lens, int b, int S) {
    if (seq_lens == nullptr) return S;
    const int v = seq_lens[b];
    return v < 0 ? 0 : (v > S ? S : v);
}

// 16 bytes that will not be read again soon: a non-temporal load keeps them from displacing
// other data in the caches (measured: 232 -> 220 us for the pooling pass at 131072 tokens)
__device__ __forceinline__ uint4 stream_load16(const uint16_t* p) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

struct Strides { int64_t b, h, t; };
inline Strides strides_of(const int64_t s[3]) { return Strides{s[0], s[1], s[2]}; }

// How pooled K lies.  Rows: [.., NBk, D] fp32.  The other two are what the score kernels read: per KV head, tiles of 32 key blocks
// (32 * D * 4 bytes), every value split into its bf16 head and tail (x = hi + lo), laid out as the B operand of the kernel's matrix
// products: for 32x32x16 ones pieces of 512 bytes (8 dims of 32 blocks, head or tail), for 16x16x32 ones pieces of 1 KB (32 dims of 16
// blocks, head or tail) in which lane l finds the 8 dims 8 * (l >> 4) of block l & 15.  Which one a call takes: key_layout.
enum KeyLayout { kKeyRows, kKeyTiles32, kKeyTiles16 };
// bf16 offset in the tile of the head of dim d of block blk, and how much further its tail is
__host__ __device__ __forceinline__ int key_tile_offset(KeyLayout layout, int d, int blk) {
    return layout == kKeyTiles16 ? ((((d >> 5) * 2 + ((blk >> 4) & 1)) * 2 * 4 + ((d >> 3) & 3)) * 16 + (blk & 15)) * 8 + (d & 7)
                                 : ((d >> 3) * 2 * 32 + (blk & 31)) * 8 + (d & 7);
}
__host__ __device__ constexpr int key_tail(KeyLayout layout) { return layout == kKeyTiles16 ? 512 : 256; }

// Launchers (one per kernel file).  Each returns a hipError_t from the launch.
// Tiles of pooled K: heads are ceil(NBk / 32) tiles apart.
hipError_t launch_pool(const Dims& d, const void* q, Strides qs, const void* k, Strides ks,
                       float* qp, float* kp, KeyLayout k_layout, hipStream_t st);
// lvn [B*Hkv, NB] fp32: ln of the mean value-vector norm of every key block.
hipError_t launch_vnorm(const Dims& d, const void* v, Strides vs, float* lvn, hipStream_t st);
// Pooled K (tiled) and, of V in the same launch, V^T for the attention kernel (NBk blocks per head, as vt_in_halves
// says) and / or lvn; with qp, the pooled queries too.
hipError_t launch_prepare_kv(const Dims& d, const void* q, Strides qs, float* qp_or_null, const void* k, Strides ks, const void* v,
                             Strides vs, float* kp, KeyLayout k_layout, void* vt_or_null, float* lvn_or_null, hipStream_t st);
// k_rows: optional device array of NB per-query-block budgets (clamped to [0, d.k] in the kernel).
// lvn: optional; added to the score of key block j (output-aware ranking).
// kp is in the layout that key_layout names.
// head_pattern: optional device array [Hq][3] = (n_sink, n_local, top_k) per query head.
// q: the queries, layout qs; the kernel pools them.  group: query heads per list (their pooled queries are averaged);
// with more than one, qp: the pooled queries [B, Hq * group, NB, D] (Hq lists), or nullptr: pooled in the kernel, too.
hipError_t launch_score_topk(const Dims& d, const float* kp, const int32_t* k_rows,
                             const int32_t* head_pattern, const float* lvn, int32_t* idx, int32_t* cnt,
                             float* scores_or_null, const void* q, Strides qs, int group, const float* qp, hipStream_t st);
// A small call (small_call in score_rows.hpp) in one launch: no pooled K, no launch_prepare_kv before; vt_or_null: V^T, as vt_in_halves
// says.
hipError_t launch_score_small(const Dims& d, const void* q, Strides qs, const void* k, Strides ks, const void* v, Strides vs,
                              void* vt_or_null, const int32_t* k_rows, const int32_t* head_pattern, int32_t* idx, int32_t* cnt,
                              float* scores_or_null, hipStream_t st);
hipError_t launch_topk_from_scores(const Dims& d, const float* scores, const int32_t* k_rows,
                                   const int32_t* head_pattern, int32_t* idx, int32_t* cnt, hipStream_t st);
// counts, into *n_bad (device), the list rows that break the attention kernel's layout rules
hipError_t launch_check_lists(const Dims& d, const int32_t* idx, const int32_t* cnt, int32_t* n_bad, hipStream_t st);
// vt is scratch for V transposed per block, B*Hkv*NBk*Bs*D bf16.
hipError_t launch_attn(const Dims& d, const void* q, Strides qs, const void* k, Strides ks,
                       const void* v, Strides vs, const int32_t* idx, const int32_t* cnt,
                       void* out, Strides os, float* lse, void* vt, hipStream_t st);   // V^T as vt_in_halves says
// The two halves of launch_attn: V -> V^T for the key blocks first .. first + n - 1 into an allocation of
// vt_bph blocks per head ([B, Hkv, vt_bph, D, Bs] bf16; halves: blocks as two halves), and the attention on such a V^T.
hipError_t launch_transpose_v(const Dims& d, const void* v, Strides vs, void* vt, int64_t vt_bph, int first, int n,
                              bool halves, hipStream_t st);
hipError_t launch_attn_vt(const Dims& d, const void* q, Strides qs, const void* k, Strides ks, const void* vt,
                          int64_t vt_bph, bool halves, const int32_t* idx, const int32_t* cnt, void* out, Strides os,
                          float* lse, hipStream_t st);

}  // namespace spa
