// Pooled scores, per-row top-k and merge with the static pattern
// (pattern computation, steps 2-4; Sec. 4.1.1 dynamic sparsity, uniform top-k
// budget of Sec. 4.1.2 Fig. "Stem" (a) or the per-query-block budget schedule of
// Token Position-Decay, Fig. "Stem" (b); optional value-magnitude term of the
// Output-Aware Metric, Fig. "Stem" (c); static patterns of Sec. 4.1.1: A-shape,
// Strided, Dilated, Tri-shape; optional per-head settings, a KV prefix, ragged
// batches and a cumulative-mass budget).
//
// score_topk_mfma_kernel: one workgroup (512 threads; two per CU) owns R consecutive
// query blocks of one query head.
//   Phase 0 - query pooling (step 1 for Q, in the kernel).  The workgroup streams its R
//   query blocks from Q and pools them itself, so that the Q stream of the select stage
//   (four fifths of its bytes) runs while other workgroups score and select; the split
//   pooled queries go straight to LDS.  (Lists shared by a group: the mean of its heads' pooled
//   queries.)
//   Phase 1 - scores on the matrix cores.  The fp32 pooled vectors are split
//   into a bf16 head and a bf16 tail (x = hi + lo, |x - hi - lo| <= 2^-18 |x|)
//   and each tile of Qp Kp^T is accumulated in fp32 from three bf16
//   products (hi.hi + hi.lo + lo.hi; v_mfma_f32_16x16x32_bf16 for 16 rows of head_dim 128, otherwise 32x32x16); the dropped
//   lo.lo term is below 2^-17 of a product.  The wavefronts take the key-block
//   tiles round robin, reading Kp straight from L2 in operand layout.  The scores
//   of the R rows stay in LDS; the NB x NB matrix never exists in memory unless
//   the caller asks for it.
//   Phase 2 - exact selection.  A wavefront owns a row: lane l holds the keys of
//   blocks l, l+64, ... in registers as order-preserving uint32 and finds the k-th
//   largest in two steps: a bound from the lanes (the smallest of the 64 lanes' largest
//   keys is reached by at least 64 keys), below which keys drop out, then radix
//   selection among the rest, 8 bits per pass (the wavefront histograms the current
//   digit into 256 LDS counters, a prefix sum over the lanes finds the bin of the wanted
//   rank; a pass that takes its whole bin ends early).  Ties at the threshold are
//   resolved by block index with a running prefix count, and static U top-k is written
//   in ascending order from the keys in registers.  Longer rows whose static blocks are sinks and
//   window alone first try a tighter bound that leaves a short list (take_best).  With a cumulative-mass budget a
//   weighted variant of the same search first finds how many blocks the row may take.
// topk_from_scores_kernel applies the same rule to caller-supplied scores (one
// wavefront per row, keys in LDS).
//
// This file is the implementation, included by three translation units so that the many kernel
// instantiations compile in parallel: select.hip (top-k on caller scores and the dispatcher) and
// select_d128.hip / select_d64.hip (score/top-k kernels for one head_dim each, SPA_SELECT_D set).
#pragma once
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "score_rows.hpp"
#include "value_block.hpp"

namespace spa {
namespace {

template <int N>
using IC_sel = std::integral_constant<int, N>;
// f(IC_sel<0>{}), ..., f(IC_sel<N-1>{})
template <int N, typename F>
__device__ __forceinline__ void static_for_sel(F&& f) {
    if constexpr (N > 0) {
        static_for_sel<N - 1>(f);
        f(IC_sel<N - 1>{});
    }
}

// Total order used for ranking: larger score first, -0 == +0, NaN below
// everything (including -inf).  The +1 keeps 0 free to mean "not a candidate".
__device__ __forceinline__ uint32_t rank_key(float s) {
    uint32_t u = __float_as_uint(s);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 1u;           // NaN
    if (u == 0x80000000u) u = 0u;                             // -0 -> +0
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return u + 1u;                                            // max finite/inf key is 0xff800000, no wrap
}

// number of set bits of `mask` that belong to lanes below the calling lane
__device__ __forceinline__ int lanes_below(uint64_t mask, int /*lane*/) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// The static pattern.  Plain A-shape: sink blocks + local window.  EXT adds the strided columns
// ((i - j) % stride == 0, within a reach for the Dilated pattern) and the dense bottom strip of the Tri-shape (rows i >= NB - n_dense).
struct Pattern {
    int ns, nl, stride, n_dense, NB, reach;   // reach: strided blocks count while i - j < reach
    float inv_stride;
};
inline Pattern pattern_of(const Dims& d) {
    return Pattern{d.ns, d.nl, d.stride, d.n_dense, d.NBk, d.reach > 0 ? d.reach : d.NBk,
                   d.stride > 0 ? 1.0f / (float)d.stride : 0.f};
}
inline bool extended(const Dims& d) { return d.stride > 0 || d.n_dense > 0; }

// is key block j (0 <= j <= i) static for the query block at block position i (pt.NB = key blocks)?
template <bool EXT>
__device__ __forceinline__ bool static_block(const Pattern& pt, int i, int j) {
    bool s = j < pt.ns || j >= i - pt.nl + 1;
    if constexpr (EXT) {
        if (pt.stride > 0) {
            // i - j < 4096: the nearest integer to (i - j) / stride is exact for multiples
            const int dist = i - j;
            const int quot = (int)__builtin_rintf((float)dist * pt.inv_stride);
            s = s || (quot * pt.stride == dist && dist < pt.reach);
        }
        s = s || (i >= pt.NB - pt.n_dense);
    }
    return s;
}

// keys[0 .. 64*ceil((i+1)/64)): rank_key of candidates, 0 for static blocks and padding.
// Runs on one full wave; all control flow is wave-uniform.
template <bool EXT>
__device__ void select_row(const uint32_t* keys, int i, const Pattern& pt, int k, int T,
                           int32_t* __restrict__ idx_row, int32_t* __restrict__ cnt_out) {
    const int lane = threadIdx.x & 63;
    const int n = i + 1;
    const int chunks = (n + 63) >> 6;
    int n_cand = 0;                                           // candidates are the nonzero keys
    for (int m = 0; m < chunks; ++m) n_cand += __popcll(__ballot(keys[(m << 6) + lane] != 0u));
    const int kk = k < n_cand ? k : n_cand;

    uint32_t thr = 0xffffffffu;   // select key > thr ... nothing, by default
    int need_eq = 0;              // plus the first need_eq candidates with key == thr
    if (kk > 0) {
        if (kk == n_cand) {
            thr = 0u;             // every candidate has key >= 1
        } else {
            uint32_t p = 0u;
            int c_at_p = n_cand;
            for (int bit = 31; bit >= 0; --bit) {
                uint32_t trial = p | (1u << bit);
                int c = 0;
                for (int m = 0; m < chunks; ++m)
                    c += __popcll(__ballot(keys[(m << 6) + lane] >= trial));
                if (c >= kk) { p = trial; c_at_p = c; if (c == kk) break; }
            }
            // p = k-th largest candidate key (or a bound that isolates exactly kk keys)
            if (c_at_p == kk) {
                thr = p - 1u;     // key >= p  <=>  key > p-1 ; p >= 1
            } else {
                int gt = 0;
                for (int m = 0; m < chunks; ++m)
                    gt += __popcll(__ballot(keys[(m << 6) + lane] > p));
                thr = p;
                need_eq = kk - gt;
            }
        }
    }
    int eq_seen = 0, out_pos = 0;
    for (int m = 0; m < chunks; ++m) {
        int j = (m << 6) + lane;
        uint32_t key = keys[j];
        bool is_static = j < n && static_block<EXT>(pt, i, j);
        bool is_eq = need_eq > 0 && key == thr && key != 0u;
        uint64_t eq_mask = __ballot(is_eq);
        bool take = is_static || (key != 0u && key > thr) ||
                    (is_eq && eq_seen + lanes_below(eq_mask, lane) < need_eq);
        uint64_t take_mask = __ballot(take);
        if (take) idx_row[out_pos + lanes_below(take_mask, lane)] = j;
        eq_seen += __popcll(eq_mask);
        out_pos += __popcll(take_mask);
    }
    for (int t = out_pos + lane; t < T; t += 64) idx_row[t] = -1;
    if (lane == 0) *cnt_out = out_pos;
}

constexpr int kWaves = 4;

// scores come from memory: [rows_total = heads * NB, NBk]
// budget of query block i: the uniform k, or the schedule's entry clamped to [0, k]
__device__ __forceinline__ int row_budget(const int32_t* __restrict__ k_rows, int i, int k) {
    if (k_rows == nullptr) return k;
    const int v = k_rows[i];
    return v < 0 ? 0 : (v > k ? k : v);
}

// Per-head configuration: head h replaces (n_sink, n_local, top_k) by its own triple, clamped to
// [0, ns], [1, nl], [0, k] of the call (which are then the maxima that fix the row capacity).
__device__ __forceinline__ void head_config(const int32_t* __restrict__ head_pattern, int h, Pattern& pt, int& k) {
    if (head_pattern == nullptr) return;
    const int32_t* hp = head_pattern + 3 * h;
    const int a = hp[0], b = hp[1], c = hp[2];
    pt.ns = a < 0 ? 0 : (a > pt.ns ? pt.ns : a);
    pt.nl = b < 1 ? 1 : (b > pt.nl ? pt.nl : b);
    k = c < 0 ? 0 : (c > k ? k : c);
}

// cumulative-mass budget of a row, defined further down
template <bool EXT, typename ScoreFn>
__device__ int mass_budget_row(ScoreFn score, int i, const Pattern& pt, uint32_t gamma_q16, uint32_t* hist, int lane);

template <bool EXT>
__global__ __launch_bounds__(kWaves * 64) void topk_from_scores_kernel(
    const float* __restrict__ scores, int64_t n_rows, int NB /* query blocks */, int NBk, int off, Pattern pt, int k,
    const int32_t* __restrict__ k_rows, const int32_t* __restrict__ head_pattern, int Hq, int T,
    int32_t* __restrict__ idx, int32_t* __restrict__ cnt, int gamma_q16 /* -1: no mass budget */,
    const int32_t* __restrict__ seq_lens, int S, int Bs) {
    extern __shared__ uint32_t lds_keys[];       // [kWaves][padded NBk] keys, then 256 counters per wave (mass budget)
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * kWaves + wave;
    if (row >= n_rows) return;                               // whole wave leaves together
    const int iq = (int)(row % NB);
    const int i = iq + off;                                  // block position in the sequence
    const int NB_b = (entry_len(seq_lens, (int)(row / NB / Hq), S) + Bs - 1) / Bs;   // ragged batch
    if (iq >= NB_b) {                                        // a row past its entry's end: empty list
        for (int t = lane; t < T; t += 64) idx[row * T + t] = -1;
        if (lane == 0) cnt[row] = 0;
        return;
    }
    pt.NB = off + NB_b;
    head_config(head_pattern, (int)((row / NB) % Hq), pt, k);
    const int padded = ((NBk + 63) >> 6) << 6;
    uint32_t* keys = lds_keys + wave * padded;
    const float* srow = scores + row * NBk;
    const int chunks = (i + 64) >> 6;
    for (int m = 0; m < chunks; ++m) {
        int j = (m << 6) + lane;
        uint32_t key = 0u;
        if (j <= i && !static_block<EXT>(pt, i, j)) key = rank_key(srow[j]);
        keys[j] = key;
    }
    // each wave reads back only its own slice; LDS ops of one wave are ordered
    int k_i = row_budget(k_rows, iq, k);
    if (gamma_q16 >= 0) {
        uint32_t* hist = lds_keys + kWaves * padded + 256 * wave;
        const int k_m = mass_budget_row<EXT>([&](int j) { return srow[j]; }, i, pt, (uint32_t)gamma_q16, hist, lane);
        k_i = k_m < k_i ? k_m : k_i;
    }
    select_row<EXT>(keys, i, pt, k_i, T, idx + row * T, cnt + row);
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// words between the score rows in LDS beyond a multiple of 64: with 16-row products the four lane groups of a store, rows 4 apart, hit
// different banks, with 32-row ones the two lane halves (4 words there take no measurably longer: 118.5 against 118.2 us at 65536 tokens)
constexpr int row_pad(int D, int R) { return sixteen_row_products(D, R) ? 4 : 8; }

// does the row's static pattern consist of sinks and window alone?
__device__ __forceinline__ bool plain_row(const Pattern& pt, int i) { return pt.stride <= 0 && i < pt.NB - pt.n_dense; }

// sum of v over the 64 lanes (DPP row reductions + row broadcasts), returned wave-uniform
__device__ __forceinline__ int wave_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);    // quad_perm [1,0,3,2]
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);   // row_half_mirror
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);   // row_mirror: every lane = its row's sum
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, true);   // row_bcast15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, true);   // row_bcast31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}


// inclusive prefix sum of v over the 64 lanes (Hillis-Steele inside the rows of 16 with DPP row
// shifts, then the row totals are carried over with the row broadcasts)
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1, lanes shifted out read 0
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, true);   // row_bcast15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, true);   // row_bcast31 into rows 2 and 3
    return v;
}

// maximum / minimum of v over the 64 lanes, returned wave-uniform (same lane walk as wave_sum;
// lanes of rows that a step leaves out combine with the neutral element)
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    auto mx = [](uint32_t a, int b) { return a > (uint32_t)b ? a : (uint32_t)b; };
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true));
    v = mx(v, __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) { return ~wave_max_u32(~v); }

// Exact k-th largest key of a row, in two steps.
// 1. A bound from the lanes: with t = ceil(kk / 64), every lane's t-th largest key is matched or
//    beaten by t keys of that lane, so at least 64 t >= kk keys reach L = the smallest of the 64
//    lanes' t-th largest keys: the k-th largest is >= L, keys below L can neither be selected nor
//    tie with the threshold and drop out.  With 16 keys per lane and kk = 64 that leaves about a
//    tenth of the row.  (t <= 2 here; a lane without t candidates gives L = 0: no bound.)
// 2. Most-significant-digit radix selection among the keys in [L, H] (H = the row maximum), up
//    to 8 bits per pass, starting at the highest bit in which L and H differ (the bits above are
//    common to all of them): the wavefront histograms the current digit of the keys that still match
//    the decided prefix into its own 256 LDS counters (LDS atomics), lane l then owns the four bins
//    255-4l .. 252-4l, a prefix sum over the lanes finds the bin that holds the wanted rank, and
//    that bin's digit extends the prefix.  A pass that takes its whole bin ends the search.
// key[m] belongs to block 64*m + lane and is 0 for static blocks, blocks beyond i and unused chunks
// (0 is never counted); NC <= MAXC: only key[0 .. NC) can be nonzero for this row.  Returns
// thr / need_eq: take key > thr, plus the first need_eq keys equal to thr in block order.
// hist: this wavefront's 256 counters.
template <int MAXC, int NC>
__device__ __forceinline__ void find_threshold_hist(const uint32_t (&key)[MAXC], int kk, int n_cand, uint32_t* hist,
                                                    int lane, uint32_t& thr, int& need_eq) {
    thr = 0xffffffffu;
    need_eq = 0;
    if (kk <= 0) return;
    if (kk == n_cand) { thr = 0u; return; }
    uint32_t m1 = 0u, m2 = 0u;           // largest and second largest key of the lane
#pragma unroll
    for (int m = 0; m < NC; ++m) {
        const uint32_t v = key[m];
        const uint32_t lo = v < m1 ? v : m1;
        m2 = m2 > lo ? m2 : lo;
        m1 = m1 > v ? m1 : v;
    }
    const uint32_t H = wave_max_u32(m1);
    uint32_t L = kk <= 64 ? wave_min_u32(m1) : (kk <= 128 ? wave_min_u32(m2) : 0u);
    if (L == 0u) L = 1u;                 // no bound: every candidate (keys are >= 1) takes part
    if (L == H) {                        // all keys that matter are equal
        thr = H;
        need_eq = kk;
        return;
    }
    const int hb = 31 - __builtin_clz(L ^ H);                 // highest bit in which the keys in [L, H] can differ
    uint32_t prefix = hb == 31 ? 0u : (H >> (hb + 1)) << (hb + 1);   // decided bits, the rest zero
    int want = kk;                       // rank wanted among the keys that match the prefix (1 = largest)
    int top = hb + 1;                    // bits [top, 32) are decided
#pragma nounroll
    while (top > 0) {
        const int shift = top > 8 ? top - 8 : 0;              // this pass decides bits [shift, top)
        const uint32_t dmask = (1u << (top - shift)) - 1u;
        *reinterpret_cast<uint4*>(hist + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
        for (int m = 0; m < NC; ++m) {
            const uint32_t kv = key[m];
            // kv >= L, and its decided bits match (two shifts: top may be 32)
            if (kv >= L && (((kv ^ prefix) >> (top - 1)) >> 1) == 0u) atomicAdd(&hist[(kv >> shift) & dmask], 1u);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint4 h = *reinterpret_cast<const uint4*>(hist + 252 - 4 * lane);   // .w = bin 255-4l ... .x = bin 252-4l
        const int own = (int)(h.x + h.y + h.z + h.w);
        const int incl = wave_inclusive_scan(own);
        const int Ln = __ffsll((unsigned long long)__ballot(incl >= want)) - 1;  // lane whose bins hold the wanted rank
        const int before = __builtin_amdgcn_readlane(incl - own, Ln);                // keys in higher bins
        const int b3 = __builtin_amdgcn_readlane((int)h.w, Ln), b2 = __builtin_amdgcn_readlane((int)h.z, Ln);
        const int b1 = __builtin_amdgcn_readlane((int)h.y, Ln), b0 = __builtin_amdgcn_readlane((int)h.x, Ln);
        const int rem = want - before;                                               // 1 .. own(Ln)
        int digit, above, in_bin;
        if (rem <= b3) { digit = 255 - 4 * Ln; above = 0; in_bin = b3; }
        else if (rem <= b3 + b2) { digit = 254 - 4 * Ln; above = b3; in_bin = b2; }
        else if (rem <= b3 + b2 + b1) { digit = 253 - 4 * Ln; above = b3 + b2; in_bin = b1; }
        else { digit = 252 - 4 * Ln; above = b3 + b2 + b1; in_bin = b0; }
        want = rem - above;                                                          // rank inside the chosen bin
        prefix |= (uint32_t)digit << shift;
        if (want == in_bin) {          // the whole bin is taken: every key that reaches both the bin's
            const uint32_t edge = prefix > L ? prefix : L;    // lower edge and L, none below
            thr = edge - 1u;           // edge >= L >= 1
            return;
        }
        top = shift;
    }
    thr = prefix;                      // the k-th largest key itself; `want` of its copies are taken
    need_eq = want;
}

// the score a rank key came from (keys >= 2; -0 has become +0)
__device__ __forceinline__ float score_of_key(uint32_t key) {
    uint32_t u = key - 1u;
    u = (u & 0x80000000u) ? (u ^ 0x80000000u) : ~u;
    return __uint_as_float(u);
}

// v_max_f32 as it is: a NaN operand gives the other one.  (From C the compiler quiets every operand first, another instruction a score.)
__device__ __forceinline__ float max_num(float x, float y) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

// A row of the plain A-shape by its few best candidates: the lists of the general way (rank keys of the whole row, find_threshold_hist, one
// pass over the row to write it) for a third of the instructions.  x[m] is the score of block 64 m + lane; candidates are the blocks [c0, c1),
// sinks those before, the local window those from c1 to i; kk candidates are wanted.
//   1. Every lane keeps its two largest scores.  At least kk of these 128 values reach L, their kk-th largest to within 2^-10 of the span, and
//      so do as many blocks; on scores without a pattern along the row about kk / 8 more of them do.
//   2. The blocks that reach L go to a list in LDS, in block order.  Whatever L is, the kk best are among them if there are kk or more, as all
//      others rank lower (NaN, which ranks lowest, never reaches L).
//   3. The kk-th largest rank key of the list, by halves: a compare and a count of the ballot per 64 of them.  Ties go to the first in the list.
// Returns false, with nothing written to memory, where that does not do: too many wanted (below), sinks beyond the first 64
// blocks, fewer than kk finite scores in the lanes' pairs, or a list that would not fit (many equal scores).  Which calls come here: lists_by_bound.
// What bounds it: instructions issued, with four wavefronts to a SIMD.  At 262144 tokens a workgroup of the general way spent 21 of its 63 us
// here, 7 each on rank keys, search and writing.  Select calls, general way against this one: 262144 tokens of 40/8 heads 704 -> 630 us (with a
// budget of 16 663 -> 582), of 8 heads 225 -> 215, 2048 blocks of 64 402 -> 336, all scores equal 356 -> 315, 8192 queries
// over 98304 tokens, blocks of 64, 86 -> 79, 131072 tokens 244 -> 236, head_dim 64 154 -> 143, with a dense strip 286 -> 275.
// Few rows, 4 to a workgroup: 512 queries over 130048 tokens, blocks of 64, head_dim 64, 47.6 -> 40.6, 2000 over 196608, blocks of 128, 55.3 -> 49.9, with
// head_dim 128 94.6 -> 88.9.  Rows without finite scores, which the general way is done with at once, take 1 to 6 % longer, as it has to follow.
// Short rows and large budgets: the closer the wanted ones come to the 128 of the lanes' pairs, the lower the bound and the longer the list, up to most
// of a short row, whereas the general way costs by quarters of the row.  Rows of one length, 64 heads of 64 query blocks, blocks of 64, head_dim 64,
// general way and this one: in kernels of up to 1024 blocks 64 wanted of 288 22.4 and 23.5 us, of 480 26.4 and 26.6, of 640 30.2 and 29.0, 112 of 288
// 22.1 and 25.3, of 640 30.8 and 30.6, 128 of 1024 39.6 and 43.1; in those of up to 2048, whose quarters are longer, 64 wanted gain 1.4 at 288 and lose
// 0.4 at 160, 112 gain 0.6 at 352 and lose 0.8 at 288, 128 lose 2.4 to 5 at any length.  That is weighed for the call (lists_by_bound), not the row,
// as a kernel that does both pays for it: 65533 tokens of 16 heads, 64 wanted, 58.4 us the general way, 55.4 this way, 59.0 with rows of up to 320
// blocks the general way and the others this way; over 350 random calls such lines are worth 0.2 %.  Above 112 wanted there is one, at 1024.
// For rows of 1025 to 2048 blocks, and from 513 on in workgroups of 16 rows: with 8 a wavefront has one row, and the other workgroups' streams
// hide it (131072 tokens of 8 heads 106.1 and 107.4, 98304 of 16 heads 86.6 and 88.6).  With 512 blocks it gives nothing (117.1 and 117.0 us at
// 65536 tokens), with 256 the general way is a few instructions a score already (59.6 and 60.8 at 32768), and with 4096 the 64 scores of a lane
// do not stay in registers (448 and 517).  Not for lists that heads share, where the query stream of all heads hides the selection (131072
// tokens 210 and 212).
template <int MAXC>
__device__ __forceinline__ bool take_best(const float (&x)[MAXC], int i, int c0, int c1, int kk, int T, float2* list, int32_t* __restrict__ idx_row,
                                          int32_t* __restrict__ cnt_out, int lane) {
    constexpr int Q = MAXC / 4, LQ = Q == 4 ? 2 : 3;          // the row goes by quarters, so that a short one is not paid in full
    static_assert(Q == 1 << LQ, "rows of 1024 or 2048 blocks");
    constexpr int CAP = 512, NY = CAP / 64;                   // list entries: in the place of the row's scores, which are in x alone from here on
    const int n = i + 1, n_cand = c1 - c0;
    int n_list = 0;
    uint32_t y[NY];                                           // rank keys of the list, 0 past its end
    int yj[NY];                                               // and their blocks
    uint32_t thr = 0u;
    int need_eq = 0;
    const bool all = kk == n_cand;                            // every block up to i
    if (!all && kk > 0) {
        if (kk > 128 || c0 > 64 || (kk > kFewWanted && n_cand < 1024)) return false;
        const int q_last = (c1 - 1) >> (6 + LQ);              // quarter of the last candidate
        float m1 = -INFINITY, m2 = -INFINITY;
        asm("" : "+v"(m2));                                   // a known -infinity would make the second score's med3 min(m1, v): m1 twice if v is a NaN
        // only in the first and the last quarter can a block not be a candidate
        auto candidate = [&](int m, bool edge) {
            return !edge || (uint32_t)((m << 6) + lane - c0) < (uint32_t)n_cand ? x[m] : -INFINITY;
        };
        static_for_sel<4>([&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value;
            if (q > q_last) return;                           // wave-uniform, as are all branches here
            auto quarter = [&](bool edge) {
#pragma unroll
                for (int m = q * Q; m < (q + 1) * Q; ++m) {
                    const float v = candidate(m, edge);
                    m2 = __builtin_amdgcn_fmed3f(m1, m2, v);
                    m1 = max_num(m1, v);
                }
            };
            if (q == 0 || q == q_last) quarter(true); else quarter(false);
        });
        const uint32_t u1 = rank_key(m1), u2 = rank_key(m2);
        const uint32_t H = wave_max_u32(u1), L0 = wave_min_u32(kk <= 64 ? u1 : u2);
        uint32_t L = L0;                                      // kk or more of the 128 reach it
        uint32_t over = H + 1u;                               // fewer than kk do
#pragma nounroll
        for (int step = 0; step < 10 && over - L > 1u; ++step) {
            const uint32_t mid = L + ((over - L) >> 1);
            const int c = __popcll(__ballot(u1 >= mid)) + __popcll(__ballot(u2 >= mid));
            if (c >= kk) L = mid; else over = mid;
            if (c == kk) break;
        }
        if (L <= rank_key(-INFINITY)) return false;           // what is no candidate must not reach it
        const float Lf = score_of_key(L);
        bool fits = true;
        static_for_sel<4>([&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value;
            if (q > q_last || !fits || (L == H && n_list >= kk)) return;      // of equal scores the first kk will do
            auto quarter = [&](bool edge) {
#pragma unroll
                for (int m = q * Q; m < (q + 1) * Q; ++m) {
                    const float v = candidate(m, edge);
                    const bool in = v >= Lf;
                    const uint64_t mask = __ballot(in);
                    const int at = n_list;
                    n_list += __popcll(mask);
                    fits = n_list <= CAP;
                    if (in && fits) list[at + lanes_below(mask, lane)] = make_float2(v, __int_as_float((m << 6) + lane));
                }
            };
            if (q == 0 || q == q_last) quarter(true); else quarter(false);
        });
        if (!fits || n_list < kk) return false;               // (fewer only if a lane had counted a score twice)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        static_for_sel<NY>([&](auto t_tag) {
            constexpr int t = decltype(t_tag)::value;
            y[t] = 0u;
            if (64 * t >= n_list) return;
            const float2 e = list[64 * t + lane];
            y[t] = 64 * t + lane < n_list ? rank_key(e.x) : 0u;
            yj[t] = __float_as_int(e.y);
        });
        if (n_list > kk) {
            auto count = [&](uint32_t at_least) {
                int c = 0;
                static_for_sel<NY>([&](auto t_tag) {
                    constexpr int t = decltype(t_tag)::value;
                    if (64 * t < n_list) c += __popcll(__ballot(y[t] >= at_least));
                });
                return c;
            };
            uint32_t lo = L, hi = H + 1u;                     // kk or more of the list reach lo, fewer hi
            int c_lo = n_list;
#pragma nounroll
            while (hi - lo > 1u && c_lo != kk) {
                const uint32_t mid = lo + ((hi - lo) >> 1);
                const int c = count(mid);
                if (c >= kk) { lo = mid; c_lo = c; } else hi = mid;
            }
            thr = lo - 1u;
            if (c_lo != kk) { need_eq = kk - count(lo + 1u); thr = lo; }
        }
    }
    // sinks, the chosen candidates, the window: ascending as they are
    int out_pos;
    if (all) {
        for (int t = lane; t < n; t += 64) idx_row[t] = t;
        out_pos = n;
    } else {
        for (int t = lane; t < c0; t += 64) idx_row[t] = t;
        out_pos = c0;
        if (kk > 0) {
            int eq_seen = 0;
            static_for_sel<NY>([&](auto t_tag) {
                constexpr int t = decltype(t_tag)::value;
                if (64 * t >= n_list) return;
                const bool is_eq = need_eq > 0 && y[t] == thr;
                const uint64_t eq_mask = __ballot(is_eq);
                const bool take = y[t] > thr || (is_eq && eq_seen + lanes_below(eq_mask, lane) < need_eq);
                const uint64_t take_mask = __ballot(take);
                if (take) idx_row[out_pos + lanes_below(take_mask, lane)] = yj[t];
                eq_seen += __popcll(eq_mask);
                out_pos += __popcll(take_mask);
            });
        }
        for (int t = lane; t < n - c1; t += 64) idx_row[out_pos + t] = c1 + t;
        out_pos += n - c1;
    }
    for (int t = out_pos + lane; t < T; t += 64) idx_row[t] = -1;
    if (lane == 0) *cnt_out = out_pos;
    return true;
}

// ---- cumulative-mass budget (the rule of the FlexPrefill family, named among the dynamic algorithms
// in Sec. 4.1.1 / "Other Sparse Attention Strategies" of Sec. 4.1.2; no formula in the paper) ----------
// A row takes, in ranking order, the fewest candidates for which the selected blocks (static ones
// included) hold the fraction gamma of the row's block-level softmax mass.  The mass is defined in
// integers so that the number of blocks does not depend on the order of a floating-point sum:
//   W_j = mass_weight(x_j, m) in [0, 2^19], m = the row's largest score that is not NaN,
//   target = ceil(Gamma * sum_j W_j / 65536), Gamma = gamma in 16-bit fixed point.
// mass_weight ~ 2^19 exp(x - m): every step is one IEEE fp32 operation, written with the
// never-contracted intrinsics, so that a CPU gets the same bits from the same sequence.
__device__ __forceinline__ uint32_t mass_weight(float x, float m) {
    if (x != x || m != m) return 0u;
    if (x == m) return 1u << 19;                          // also m = +inf
    if (__builtin_isinf(x) || __builtin_isinf(m)) return 0u;
    const float t = __fmul_rn(__fsub_rn(x, m), 1.44269504088896340736f);
    if (!(t >= -40.0f)) return 0u;
    const float n = __builtin_rintf(t);                   // ties to even
    const float f = __fsub_rn(t, n);
    float p = 1.5403530393381609954e-4f;                  // Taylor coefficients of e^(f ln 2), degree 6 .. 0
    p = __fmaf_rn(p, f, 1.3333558146428443423e-3f);
    p = __fmaf_rn(p, f, 9.6181291076284771619e-3f);
    p = __fmaf_rn(p, f, 5.5504108664821579953e-2f);
    p = __fmaf_rn(p, f, 2.4022650695910071233e-1f);
    p = __fmaf_rn(p, f, 6.9314718055994530942e-1f);
    p = __fmaf_rn(p, f, 1.0f);
    const float w = ldexpf(p, (int)n);
    return (uint32_t)__fadd_rn(__fmul_rn(w, 524288.0f), 0.5f);
}

// Number of candidates the mass budget lets the query block at block position i take (before the
// count budgets cap it).  One full wavefront; score(j) returns the ranking score of key block j <= i.
// hist: 256 LDS counters of this wavefront.  gamma_q16 = Gamma.
template <bool EXT, typename ScoreFn>
__device__ int mass_budget_row(ScoreFn score, int i, const Pattern& pt, uint32_t gamma_q16, uint32_t* hist, int lane) {
    const int chunks = (i + 64) >> 6;
    float mloc = -INFINITY;
    for (int c = 0; c < chunks; ++c) {
        const int j = (c << 6) + lane;
        const float x = j <= i ? score(j) : -INFINITY;
        if (x == x && x > mloc) mloc = x;
    }
    // wave maximum of floats through the order-preserving keys (mloc is never NaN)
    const uint32_t mk = wave_max_u32(rank_key(mloc));
    const float m = mk >= 2u ? score_of_key(mk) : -INFINITY;
    int z_l = 0, ms_l = 0;                                 // lane sums; a row's total is < 2^31
    for (int c = 0; c < chunks; ++c) {
        const int j = (c << 6) + lane;
        if (j <= i) {
            const int w = (int)mass_weight(score(j), m);
            z_l += w;
            if (static_block<EXT>(pt, i, j)) ms_l += w;
        }
    }
    const uint32_t Z = (uint32_t)wave_sum(z_l), Ms = (uint32_t)wave_sum(ms_l);
    const uint32_t target = (uint32_t)(((uint64_t)gamma_q16 * Z + 65535ull) >> 16);
    if (Ms >= target) return 0;
    uint32_t need = target - Ms;                           // mass still wanted from the candidates, >= 1
    // weighted radix selection: the key at which the mass of the better-ranked candidates reaches `need`
    uint32_t prefix = 0u;
#pragma nounroll
    for (int shift = 24; shift >= 0; shift -= 8) {
        *reinterpret_cast<uint4*>(hist + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        for (int c = 0; c < chunks; ++c) {
            const int j = (c << 6) + lane;
            if (j <= i && !static_block<EXT>(pt, i, j)) {
                const float x = score(j);
                const uint32_t kv = rank_key(x);
                if ((((kv ^ prefix) >> shift) >> 8) == 0u) {
                    const uint32_t w = mass_weight(x, m);
                    if (w != 0u) atomicAdd(&hist[(kv >> shift) & 255u], w);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint4 h = *reinterpret_cast<const uint4*>(hist + 252 - 4 * lane);   // .w = bin 255-4l ... .x = bin 252-4l
        const int own = (int)(h.x + h.y + h.z + h.w);
        const int incl = wave_inclusive_scan(own);
        const int Ln = __ffsll((unsigned long long)__ballot((uint32_t)incl >= need)) - 1;   // exists: candidates' mass >= need
        const uint32_t before = (uint32_t)__builtin_amdgcn_readlane(incl - own, Ln);
        const uint32_t b3 = (uint32_t)__builtin_amdgcn_readlane((int)h.w, Ln), b2 = (uint32_t)__builtin_amdgcn_readlane((int)h.z, Ln);
        const uint32_t b1 = (uint32_t)__builtin_amdgcn_readlane((int)h.y, Ln);
        const uint32_t rem = need - before;
        uint32_t digit, above;
        if (rem <= b3) { digit = 255 - 4 * Ln; above = 0; }
        else if (rem <= b3 + b2) { digit = 254 - 4 * Ln; above = b3; }
        else if (rem <= b3 + b2 + b1) { digit = 253 - 4 * Ln; above = b3 + b2; }
        else { digit = 252 - 4 * Ln; above = b3 + b2 + b1; }
        need = rem - above;                                // mass wanted from the chosen bin, >= 1
        prefix |= digit << shift;
    }
    // prefix = the key tau of the last block taken; all of the better keys, plus as many copies of tau
    // (equal keys have equal weights) as it takes to cover what is left
    int n_above = 0;
    for (int c = 0; c < chunks; ++c) {
        const int j = (c << 6) + lane;
        const bool gt = j <= i && !static_block<EXT>(pt, i, j) && rank_key(score(j)) > prefix;
        n_above += __popcll(__ballot(gt));
    }
    const uint32_t w_tau = mass_weight(score_of_key(prefix), m);
    return n_above + (int)((need + w_tau - 1u) / w_tau);
}

// The same budget for a row whose keys already sit in registers (the select kernel): the weights are
// computed once per block, the weighted radix passes run over registers.  key[m] / is_static_bits
// as in the select kernel (block 64 m + lane; 0 = not a candidate); score(j) returns the ranking
// score of block j; chunks = chunks of 64 blocks the row reaches.  Integer arithmetic: the result is
// the one mass_budget_row gives, whatever the order of the sums, or k_count, the count budget, where the row may take that many or more.
// A weight is 2^19 at most, so k_count blocks cannot hold more than k_count times that: where the target is beyond it, which is most rows if
// their scores are close to each other, the four passes over the row are left out.  Select calls, gamma 0.9, scores of random keys: 65536
// tokens 134.9 -> 122.3 us, 131072 298 -> 264, 262144 of 40/8 heads 894 -> 816, 2048 blocks of 64 of 16 heads 322 -> 273; rows that keep a few
// blocks 131.0 and 130.8.  (Longer rows and caller-supplied scores go through mass_budget_row, which always searches.)
template <int MAXC, typename ScoreFn>
__device__ __forceinline__ int mass_budget_regs(const uint32_t (&key)[MAXC], uint64_t is_static_bits, ScoreFn score, int i,
                                                int chunks, uint32_t gamma_q16, int k_count, uint32_t* hist, int lane) {
    float x[MAXC];
    float mloc = -INFINITY;
#pragma unroll
    for (int m = 0; m < MAXC; ++m) {
        x[m] = -INFINITY;
        if (m < chunks) {
            const int j = (m << 6) + lane;
            x[m] = j <= i ? score(j) : __builtin_nanf("");   // NaN: weighs nothing, never the maximum
            if (x[m] == x[m] && x[m] > mloc) mloc = x[m];
        }
    }
    const uint32_t mk = wave_max_u32(rank_key(mloc));
    const float mx = mk >= 2u ? score_of_key(mk) : -INFINITY;
    uint32_t w[MAXC];
    int z_l = 0, ms_l = 0;
#pragma unroll
    for (int m = 0; m < MAXC; ++m) {
        w[m] = 0u;
        if (m < chunks) {
            w[m] = mass_weight(x[m], mx);
            z_l += (int)w[m];
            if ((is_static_bits >> m) & 1ull) ms_l += (int)w[m];
        }
    }
    const uint32_t Z = (uint32_t)wave_sum(z_l), Ms = (uint32_t)wave_sum(ms_l);
    const uint32_t target = (uint32_t)(((uint64_t)gamma_q16 * Z + 65535ull) >> 16);
    if (Ms >= target) return 0;
    uint32_t need = target - Ms;
    if ((uint64_t)(uint32_t)k_count << 19 < need) return k_count;
    uint32_t prefix = 0u;
#pragma nounroll
    for (int shift = 24; shift >= 0; shift -= 8) {
        *reinterpret_cast<uint4*>(hist + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
        for (int m = 0; m < MAXC; ++m) {
            const uint32_t kv = key[m];
            if (m < chunks && kv != 0u && w[m] != 0u && (((kv ^ prefix) >> shift) >> 8) == 0u)
                atomicAdd(&hist[(kv >> shift) & 255u], w[m]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint4 h = *reinterpret_cast<const uint4*>(hist + 252 - 4 * lane);   // .w = bin 255-4l ... .x = bin 252-4l
        const int own = (int)(h.x + h.y + h.z + h.w);
        const int incl = wave_inclusive_scan(own);
        const int Ln = __ffsll((unsigned long long)__ballot((uint32_t)incl >= need)) - 1;
        const uint32_t before = (uint32_t)__builtin_amdgcn_readlane(incl - own, Ln);
        const uint32_t b3 = (uint32_t)__builtin_amdgcn_readlane((int)h.w, Ln), b2 = (uint32_t)__builtin_amdgcn_readlane((int)h.z, Ln);
        const uint32_t b1 = (uint32_t)__builtin_amdgcn_readlane((int)h.y, Ln);
        const uint32_t rem = need - before;
        uint32_t digit, above;
        if (rem <= b3) { digit = 255 - 4 * Ln; above = 0; }
        else if (rem <= b3 + b2) { digit = 254 - 4 * Ln; above = b3; }
        else if (rem <= b3 + b2 + b1) { digit = 253 - 4 * Ln; above = b3 + b2; }
        else { digit = 252 - 4 * Ln; above = b3 + b2 + b1; }
        need = rem - above;
        prefix |= digit << shift;
    }
    int n_above_l = 0;
#pragma unroll
    for (int m = 0; m < MAXC; ++m) n_above_l += (m < chunks && key[m] > prefix) ? 1 : 0;
    const int n_above = wave_sum(n_above_l);
    const uint32_t w_tau = mass_weight(score_of_key(prefix), mx);
    return n_above + (int)((need + w_tau - 1u) / w_tau);
}

// Everything the score + top-k step of one workgroup needs besides its rows.
struct ScoreArgs {
    const float* kp;              // pooled K, tiled in operand layout by the pooling kernel
    int Hq, G, NB /* query blocks */, NBk, off /* block position of query block 0 */;
    Pattern pt;
    int k;
    const int32_t* k_rows;
    const int32_t* head_pattern;
    const float* lvn;
    int T;
    float scale;
    int32_t* idx;
    int32_t* cnt;
    float* scores_out;
    uint32_t gamma_q16;           // cumulative-mass budget in 16-bit fixed point (MASS kernels only)
    const int32_t* seq_lens;      // ragged batch: tokens per batch entry, or nullptr
    int S, Bs;                    // padded query tokens, block size (to turn seq_lens into block counts)
    const uint16_t* q;            // the queries themselves (pooled in the kernel), layout qs
    Strides qs;
    int group;                    // GROUP kernels: query heads h * group .. + group - 1 share list h
    const float* qp;              // GROUP kernels: pooled queries [B * Hq * group, NB, D] fp32, or nullptr: pooled in the kernel
};

// LDS copy of the split queries, the A operands of the kernel's matrix products: bf16 offset of the head of dim d of row r; its
// tail is query_tail further
template <int D, int R>
__device__ __forceinline__ int query_offset(int d, int r) {
    if constexpr (sixteen_row_products(D, R)) return ((((d >> 5) * 2) * 4 + ((d >> 3) & 3)) * R + r) * 8 + (d & 7);
    return ((((d >> 4) * 2) * R + r) * 2 + ((d >> 3) & 1)) * 8 + (d & 7);
}
template <int D, int R>
constexpr int query_tail() { return (sixteen_row_products(D, R) ? 4 : 2) * R * 8; }

// Phase 0 of the score kernels: the split pooled queries (MFMA A operands) of the query blocks
// i0 .. i0 + R - 1 of head bh go to LDS behind the SW words of score space at S, in the space of the
// phase-2 counters, instead of being held in 8 * D / 16 registers per lane: the kernels stay within
// 128 registers.  Needs R * D * 4 bytes <= the counters' NWV KB.
// The workgroup pools its R query blocks from Q itself (the block mean pooling of step 1,
// same arithmetic in the same order as pool_kernel).  Streaming
// 16 blocks (512 KB) per workgroup with two blocks per 256 threads in flight keeps the HBM busy
// while the other workgroup of the CU scores and selects: the Q stream, four fifths of the bytes
// of the select stage, hides the rest of the stage.  Ends with a barrier.
// GROUP: a row's query is the mean of the pooled queries of a.group heads (lists shared by a KV group).  Their blocks are streamed one
// after the other and added in head order, so that here, too, the Q stream hides the rest: select calls of 32/8 heads against
// pooled and averaged queries from two launches before 32768 tokens 65 -> 56 us, 65536 126 -> 109, 131072 256 -> 211, 262144 of
// 40/8 heads 634 -> 503.  A workgroup then reads 512 KB and more; where there are too few of them to fill the chip (the
// rule is group_pooled_in_kernel), the pooling launch of K has pooled the heads' queries, too, and they are averaged here.
template <int D, int R, int SW, int NWV, bool GROUP>
__device__ __forceinline__ void stage_queries(const ScoreArgs& a, const int bh, const int i0, float* S) {
    const int NB = a.NB;
    const int b = bh / a.Hq, h = bh % a.Hq;
    __bf16* const qlds = reinterpret_cast<__bf16*>(S + SW);
    static_assert(R * D * 4 <= NWV * 256 * 4, "staged queries must fit the counters' space");
    if (GROUP && a.qp != nullptr) {
        for (int x = threadIdx.x; x < R * D; x += NWV * 64) {
            const int r = x / D, d = x % D;
            const int row = i0 + r < NB ? i0 + r : NB - 1;    // rows past the end are computed but never used
            const float* src = a.qp + ((int64_t)bh * a.group * NB + row) * D + d;
            float sum = src[0];
            for (int g = 1; g < a.group; ++g) sum += src[(int64_t)g * NB * D];
            float mean = sum * (1.0f / (float)a.group);
            asm("" : "+v"(mean));                            // rounded before it is split
            const __bf16 hi = (__bf16)mean;
            const int at = query_offset<D, R>(d, r);
            qlds[at] = hi;
            qlds[at + query_tail<D, R>()] = (__bf16)(mean - (float)hi);
        }
        __syncthreads();
    } else {
        constexpr int TPR = D / 8, RPP = 256 / TPR;      // lanes per token row, token rows per pass
        constexpr int NGRP = NWV / 4;                    // groups of 256 threads, one block at a time each
        constexpr int ROWS = (R + NGRP - 1) / NGRP;      // query blocks per group
        constexpr int DEPTH = 2;                         // blocks in flight per group
        // the partial sums live in the score rows' space, or (short rows) behind the counters
        constexpr bool PART_IN_S = 2 * NGRP * RPP * D <= SW;
        const int t = threadIdx.x, grp = t >> 8, t256 = t & 255;
        const int prow = t256 / TPR, chunk = t256 % TPR;
        const int Bs = a.Bs, passes = Bs / RPP;          // at most 8
        const int Sq_b = entry_len(a.seq_lens, b, a.S);
        typedef float (*Part)[D];
        Part const part = reinterpret_cast<Part>(PART_IN_S ? S : S + SW + NWV * 256) + grp * 2 * RPP;   // two buffers of RPP rows per group
        const uint16_t* const qhead = a.q + b * a.qs.b + (GROUP ? h * a.group : h) * a.qs.h;
        const int64_t tstride = a.qs.t;
        // tokens of this group's rr-th block that exist (0: block past the call, the entry or the tile)
        auto valid_tokens = [&](int rr) {
            const int r = grp + rr * NGRP, iq = i0 + r;
            if (r >= R || iq >= NB) return 0;
            const int n = Sq_b - iq * Bs;
            return n < 0 ? 0 : (n > Bs ? Bs : n);
        };
        // One instantiation per number of passes (block size / token rows per pass) and per kind of
        // tile.  FULL: every block of the tile exists and is whole, so all loads are unconditional: the
        // compiler can then wait for exactly the block it is about to reduce while the next two stay in
        // flight (with a conditional load anywhere in the loop it waits for all of them, and a
        // workgroup streams at a third of the rate).  Otherwise (last tile of a sequence) rows are
        // predicated; that path is rare and not tuned.
        auto pool_rows = [&](auto passes_tag, auto full_tag) {
            constexpr int PASSES = decltype(passes_tag)::value;
            constexpr bool FULL = decltype(full_tag)::value != 0;
            uint4 raw[DEPTH][PASSES];
            // per-lane byte offsets inside a block (fixed for the kernel; token stride <= 2^22 elements,
            // so they fit 32 bits) on top of a wave-uniform block base
            uint32_t voff[PASSES];
#pragma unroll
            for (int p2 = 0; p2 < PASSES; ++p2) voff[p2] = 2u * ((uint32_t)(p2 * RPP + prow) * (uint32_t)tstride + (uint32_t)chunk * 8u);
            const int grp_u = __builtin_amdgcn_readfirstlane(grp);
            auto load = [&](auto slot_tag, int rr, int g) {      // block rr of this group of threads, head g of the KV group
                constexpr int SLOT = decltype(slot_tag)::value;
                const char* const base = reinterpret_cast<const char*>(qhead + (GROUP ? g * a.qs.h : 0) + (int64_t)(i0 + grp_u + rr * NGRP) * Bs * tstride);
                const int nv = FULL ? Bs : valid_tokens(rr);
#pragma unroll
                for (int p2 = 0; p2 < PASSES; ++p2) {
                    if constexpr (FULL) {
                        raw[SLOT][p2] = stream_load16(reinterpret_cast<const uint16_t*>(base + voff[p2]));
                    } else {
                        raw[SLOT][p2] = make_uint4(0u, 0u, 0u, 0u);
                        if (p2 * RPP + prow < nv) raw[SLOT][p2] = stream_load16(reinterpret_cast<const uint16_t*>(base + voff[p2]));
                    }
                }
            };
            // the block in a slot: partial sums of its token rows to LDS, the slot's next load, then the means of the D columns
            float mean = 0.f;                             // threads 0 .. D - 1 of the group
            auto reduce = [&](auto slot_tag, int rr, auto&& next) {
                constexpr int SLOT = decltype(slot_tag)::value;
                float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int p2 = 0; p2 < PASSES; ++p2) {
                    acc[0] += bf16_lo(raw[SLOT][p2].x); acc[1] += bf16_hi(raw[SLOT][p2].x);
                    acc[2] += bf16_lo(raw[SLOT][p2].y); acc[3] += bf16_hi(raw[SLOT][p2].y);
                    acc[4] += bf16_lo(raw[SLOT][p2].z); acc[5] += bf16_hi(raw[SLOT][p2].z);
                    acc[6] += bf16_lo(raw[SLOT][p2].w); acc[7] += bf16_hi(raw[SLOT][p2].w);
                }
                Part const buf = part + SLOT * RPP;       // slots alternate: one barrier a block
#pragma unroll
                for (int e = 0; e < 8; ++e) buf[prow][chunk * 8 + e] = acc[e];
                next();
                __syncthreads();
                if (t256 < D) {
                    float sum = 0.f;
#pragma unroll
                    for (int rr2 = 0; rr2 < RPP; ++rr2) sum += buf[rr2][t256];
                    const int nv = FULL ? Bs : valid_tokens(rr);
                    mean = nv == Bs ? sum * (1.0f / (float)Bs) : (nv > 0 ? sum / (float)nv : 0.f);
                }
            };
            auto put = [&](int rr, float x) {             // the pooled query of block rr, split
                const int r = grp + rr * NGRP;
                if (t256 < D && r < R) {
                    const __bf16 hi = (__bf16)x;                      // round to nearest even, twice
                    const __bf16 lo = (__bf16)(x - (float)hi);
                    const int at = query_offset<D, R>(t256, r);
                    qlds[at] = hi;
                    qlds[at + query_tail<D, R>()] = lo;
                }
            };
            static_assert(DEPTH == 2, "the slots alternate");
            if constexpr (!GROUP) {
                static_for_sel<(DEPTH < ROWS ? DEPTH : ROWS)>([&](auto rr_tag) { load(rr_tag, decltype(rr_tag)::value, 0); });
                static_for_sel<ROWS>([&](auto rr_tag) {
                    constexpr int RR = decltype(rr_tag)::value;
                    reduce(IC_sel<RR % DEPTH>{}, RR, [&]() { if constexpr (RR + DEPTH < ROWS) load(IC_sel<RR % DEPTH>{}, RR + DEPTH, 0); });
                    put(RR, mean);
                });
            } else {
                // the ROWS * group blocks in a row, two in flight; the loop's loads are all unconditional, its last two
                // blocks are peeled
                static_assert(ROWS % 2 == 0, "an even number of blocks");
                const int ng = a.group;
                const float inv = 1.0f / (float)ng;
                int rr = 0, g = 0, rr_l = 0, g_l = 0;     // next block to reduce, to load
                float sum_g = 0.f;
                auto load_next = [&](auto slot_tag) {
                    load(slot_tag, rr_l, g_l);
                    if (++g_l == ng) { g_l = 0; ++rr_l; }
                };
                auto add = [&]() {
                    sum_g = g == 0 ? mean : sum_g + mean;
                    if (++g == ng) {
                        float x = sum_g * inv;
                        asm("" : "+v"(x));               // rounded before it is split, not contracted with the difference
                        put(rr, x);
                        g = 0;
                        ++rr;
                    }
                };
                load_next(IC_sel<0>{});
                load_next(IC_sel<1>{});
#pragma nounroll
                for (int x = 2; x < ROWS * ng; x += 2) {
                    reduce(IC_sel<0>{}, rr, [&]() { load_next(IC_sel<0>{}); });
                    add();
                    reduce(IC_sel<1>{}, rr, [&]() { load_next(IC_sel<1>{}); });
                    add();
                }
                reduce(IC_sel<0>{}, rr, []() {});
                add();
                reduce(IC_sel<1>{}, rr, []() {});
                add();
            }
        };
        // whole tile inside the call, the entry and (rows per group) the tile: every block is full
        const bool full = R % NGRP == 0 && (int64_t)(i0 + R) * Bs <= (int64_t)Sq_b;
        constexpr int P128 = 128 / RPP, P64 = 64 / RPP;  // passes for blocks of 128 / 64 tokens
        if (passes == P128) {
            if (full) pool_rows(IC_sel<P128>{}, IC_sel<1>{}); else pool_rows(IC_sel<P128>{}, IC_sel<0>{});
        } else {
            if (full) pool_rows(IC_sel<P64>{}, IC_sel<1>{}); else pool_rows(IC_sel<P64>{}, IC_sel<0>{});
        }
        __syncthreads();
    }
}

// One score of row mrow and key block j to the LDS rows, whose first column is key block col0, and to memory if asked for.  Output-aware
// ranking: the key block's ln(value magnitude) lv joins.
template <int LD>
__device__ __forceinline__ void store_score(const ScoreArgs& a, float dot, float* S, int col0, int mrow, int j, int bh, int i0,
                                            bool with_lv, float lv) {
    const float sc = with_lv ? a.scale * dot + lv : a.scale * dot;
    S[mrow * LD + j - col0] = sc;
    const int i = i0 + mrow;
    if (a.scores_out != nullptr && i < a.NB && j < a.NBk)
        a.scores_out[((int64_t)bh * a.NB + i) * a.NBk + j] = j <= i + a.off ? sc : -INFINITY;
}

// Scores of the key tiles jt_first, jt_first + NWV, .. below jt_end for R rows.  The pooled K arrives tiled in operand layout and already
// split into bf16 head and tail (key_tile_offset), so a load instruction of a wavefront covers whole pieces (row-major rows would
// cost 32 cache lines per instruction) and what it loads is the MFMA operand.  NBUF = D / 16: a register buffer of a whole tile, each piece
// refilled with the same piece of the wave's next tile as soon as its three products are issued, so every load has a full tile of
// MFMA work to arrive.  NBUF = D / 32: a rolling buffer of half a tile; slot x % NBUF holds piece x and is refilled with piece x + NBUF, of
// this tile or the next, so a load still has half a tile of MFMA work.  Blocks past NBk in the last tile hold whatever the workspace held:
// their columns are never ranked or written out.  Which products: sixteen_row_products.
template <int D, int R, int LD, int NBUF, int NWV>
__device__ __forceinline__ void score_tiles(const ScoreArgs& a, const float* kbase, const __bf16* qlds, float* S, int col0, int jt_first,
                                            int jt_end, int bh, int i0, const float* lvbase) {
    constexpr int DS = D / 16;                            // pieces of a tile: 16 dims of 32 blocks, or 32 dims of 16 blocks
    constexpr bool ROWS16 = sixteen_row_products(D, R);
    constexpr int TAIL = key_tail(ROWS16 ? kKeyTiles16 : kKeyTiles32);
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int at = ROWS16 ? lane * 8 : (half * 64 + l32) * 8;
    auto tile_ptr = [&](int jt) { return reinterpret_cast<const __bf16*>(kbase + (int64_t)jt * (32 * D)) + at; };
    bf16x8 kraw[2 * NBUF];                                // [2b] = hi, [2b + 1] = lo of the piece in slot b
    if (jt_first < jt_end) {
        const __bf16* src = tile_ptr(jt_first);
#pragma unroll
        for (int x = 0; x < NBUF; ++x) {
            kraw[2 * x] = *reinterpret_cast<const bf16x8*>(src + x * 1024);
            kraw[2 * x + 1] = *reinterpret_cast<const bf16x8*>(src + x * 1024 + TAIL);
        }
    }
    for (int jt = jt_first; jt < jt_end; jt += NWV) {
        const __bf16* cur = tile_ptr(jt);
        const __bf16* next = tile_ptr(jt + NWV < jt_end ? jt + NWV : jt);      // the last tile refills from itself: in bounds, never used
        auto refill = [&](int x) {                        // piece x has been used
            const int slot = x % NBUF, x_fill = (x + NBUF) % DS;
            const __bf16* from = x + NBUF < DS ? cur : next;
            kraw[2 * slot] = *reinterpret_cast<const bf16x8*>(from + x_fill * 1024);
            kraw[2 * slot + 1] = *reinterpret_cast<const bf16x8*>(from + x_fill * 1024 + TAIL);
        };
        if constexpr (ROWS16) {
            const __bf16* const qlane = qlds + ((lane >> 4) * R + (lane & 15)) * 8;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};       // blocks lane & 15 and 16 more, rows 4 * (lane >> 4) .. + 3
#pragma unroll
            for (int s = 0; s < DS / 2; ++s) {
                const bf16x8 qh = *reinterpret_cast<const bf16x8*>(qlane + (s * 2 + 0) * 4 * R * 8);
                const bf16x8 ql = *reinterpret_cast<const bf16x8*>(qlane + (s * 2 + 1) * 4 * R * 8);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const bf16x8 k_hi = kraw[2 * ((2 * s + u) % NBUF)], k_lo = kraw[2 * ((2 * s + u) % NBUF) + 1];
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ql, k_hi, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qh, k_lo, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qh, k_hi, acc[u], 0, 0, 0);
                    refill(2 * s + u);
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j = 32 * jt + 16 * u + (lane & 15);
                const float lv = lvbase != nullptr ? lvbase[j < a.NBk ? j : a.NBk - 1] : 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) store_score<LD>(a, acc[u][r], S, col0, 4 * (lane >> 4) + r, j, bh, i0, lvbase != nullptr, lv);
            }
        } else {
            const int j = 32 * jt + l32;
            const float lv = lvbase != nullptr ? lvbase[j < a.NBk ? j : a.NBk - 1] : 0.f;
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int s = 0; s < DS; ++s) {
                const bf16x8 k_hi = kraw[2 * (s % NBUF)], k_lo = kraw[2 * (s % NBUF) + 1];
                const bf16x8 qh = *reinterpret_cast<const bf16x8*>(qlds + (((s * 2 + 0) * R + l32 % R) * 2 + half) * 8);
                const bf16x8 ql = *reinterpret_cast<const bf16x8*>(qlds + (((s * 2 + 1) * R + l32 % R) * 2 + half) * 8);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ql, k_hi, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qh, k_lo, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qh, k_hi, acc, 0, 0, 0);
                refill(s);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int mrow = 8 * (r >> 2) + 4 * half + (r & 3);            // row of the 32x32 result held in acc[r]
                if (mrow < R) store_score<LD>(a, acc[r], S, col0, mrow, j, bh, i0, lvbase != nullptr, lv);
            }
        }
    }
}

// Small calls: what a workgroup needs to pool K itself, and the call's V^T.
struct KeyArgs {
    const uint16_t* k;
    Strides ks;
    const uint16_t* v;            // with vt: V -> V^T, blocks of Bs tokens, halves as vt_in_halves says
    Strides vs;
    uint16_t* vt;
    int Skv, Hkv, halves;
    int n_heads;                  // batch entries times KV heads
};

// where the pooled K tile of such a workgroup lies in its LDS (words): behind scores, counters and partial sums
template <int D, int R, int LD, int NWV>
__host__ __device__ constexpr int key_tile_at() {
    return R * LD + NWV * 256 + 2 * (NWV / 4) * (256 / (D / 8)) * D;
}

// Means of the key blocks 0 .. n_blk - 1 (n_blk <= most_small_blocks; kh: the head's first token, Skv tokens) to an operand tile in LDS, in the
// layout and with the arithmetic of the pooling kernel (pool.hip).  Two groups of 256 threads take the blocks in turn.  What bounds it is latency,
// so all of the blocks are asked for before the first is reduced (up to 64 KB of K in 32 registers a lane, three blocks of 32 KB in 64); two in flight,
// a memory latency and a barrier a round, took 3.1 us of a workgroup's 6.7 at 512 tokens, head_dim 64, blocks of 64.  Asking for them before the
// queries are pooled as well gives 0.1 us more there and needs 94 to 163 registers instead of 72 and 111: a workgroup less to a CU, and
// batches of short prompts up to 40 % slower (10 prompts of 384 tokens, 32/8 heads, head_dim 128, blocks of 128, from a graph: 53.7 us, this way 48.7, two in
// flight 49.8; their selection 18.7, 14.4, 15.8; 32 chunks of 64 queries over 448 tokens, head_dim 64, blocks of 64, 41.8, 37.4, 39.0).
// part_base: 2 * NGRP * RPP * D words of LDS.  All loads are unconditional within a block, tokens past the end re-read the last one and count 0.
// Ends with a barrier.
template <int D, int BS, int NWV>
__device__ __forceinline__ void stage_keys(const uint16_t* kh, int64_t stride_t, int n_blk, int Skv, float* part_base, __bf16* tile) {
    constexpr int TPR = D / 8, RPP = 256 / TPR, PASSES = BS / RPP, NGRP = NWV / 4, SLOTS = (most_small_blocks(D, BS) + NGRP - 1) / NGRP;
    static_assert(SLOTS % 2 == 0, "reduced in pairs");
    const int grp = threadIdx.x >> 8, t256 = threadIdx.x & 255, prow = t256 / TPR, chunk = t256 % TPR;
    typedef float (*Part)[D];
    Part const part = reinterpret_cast<Part>(part_base) + grp * 2 * RPP;
    uint4 raw[SLOTS][PASSES];
    static_for_sel<SLOTS>([&](auto s_tag) {
        constexpr int s = decltype(s_tag)::value;
        if (s * NGRP >= n_blk) return;                        // workgroup-uniform
        const int j = s * NGRP + grp < n_blk ? s * NGRP + grp : n_blk - 1, last = Skv - 1 - j * BS;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int row = p * RPP + prow < last ? p * RPP + prow : last;
            raw[s][p] = *reinterpret_cast<const uint4*>(kh + (int64_t)(j * BS + row) * stride_t + chunk * 8);
        }
    });
    static_for_sel<SLOTS / 2>([&](auto pair_tag) {
        constexpr int s0 = 2 * decltype(pair_tag)::value;
        if (s0 * NGRP >= n_blk) return;
        static_for_sel<2>([&](auto o_tag) {                   // partial sums of the pair's token rows
            constexpr int s = s0 + decltype(o_tag)::value;
            if (s * NGRP >= n_blk) return;
            const int j = s * NGRP + grp < n_blk ? s * NGRP + grp : n_blk - 1, n_valid = Skv - j * BS < BS ? Skv - j * BS : BS;
            float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < PASSES; ++p) {
                const uint32_t keep = p * RPP + prow < n_valid ? 0xffffffffu : 0u;
                const uint4 w = make_uint4(raw[s][p].x & keep, raw[s][p].y & keep, raw[s][p].z & keep, raw[s][p].w & keep);
                acc[0] += bf16_lo(w.x); acc[1] += bf16_hi(w.x);
                acc[2] += bf16_lo(w.y); acc[3] += bf16_hi(w.y);
                acc[4] += bf16_lo(w.z); acc[5] += bf16_hi(w.z);
                acc[6] += bf16_lo(w.w); acc[7] += bf16_hi(w.w);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) part[(s - s0) * RPP + prow][chunk * 8 + e] = acc[e];
        });
        __syncthreads();
        const int s = s0 + t256 / D, d = t256 % D, j = s * NGRP + grp;       // threads 0 .. D - 1 the first block's columns, D .. 2 D - 1 the second's
        if (t256 < 2 * D && j < n_blk) {
            const int n_valid = Skv - j * BS < BS ? Skv - j * BS : BS;
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < RPP; ++r) sum += part[(s - s0) * RPP + r][d];
            float mean = n_valid == BS ? sum * (1.0f / (float)BS) : sum / (float)n_valid;
            asm("" : "+v"(mean));                             // rounded before it is split, as in the pooling kernel
            const __bf16 hi = (__bf16)mean;
            const int at = key_tile_offset(kKeyTiles32, d, j);
            tile[at] = hi;
            tile[at + key_tail(kKeyTiles32)] = (__bf16)(mean - (float)hi);
        }
        __syncthreads();
    });
}

// Scores, top-k and merged lists of the query blocks i0 .. i0 + R - 1 of head bh = b * Hq + h, by a
// 512-thread workgroup.  S: R * (MAXC * 64 + row_pad) floats of LDS for the scores, then 256 counters per
// wavefront.  Ends without a barrier; the caller must not reuse S before one.
// The split pooled queries are staged in LDS by stage_queries.
template <int D, int R, int MAXC, bool EXT, bool MASS, int NWV, bool GROUP, bool BEST, int KIN = 0>
__device__ __forceinline__ void score_topk_rows(const ScoreArgs& a, const int bh, const int i0, float* S, const KeyArgs* keys = nullptr) {
    static_assert(!BEST || (!MASS && !GROUP && has_lists_by_bound(R, MAXC)), "lists by bound are for these kernels");
    constexpr int LD = MAXC * 64 + row_pad(D, R);
    const float* __restrict__ kp = a.kp;
    const int Hq = a.Hq, G = a.G, NB = a.NB, NBk = a.NBk, off = a.off, T = a.T;
    Pattern pt = a.pt;
    int k = a.k;
    const int32_t* __restrict__ k_rows = a.k_rows;
    const int32_t* __restrict__ head_pattern = a.head_pattern;
    const float* __restrict__ lvn = a.lvn;
    const float scale = a.scale;
    int32_t* __restrict__ idx = a.idx;
    int32_t* __restrict__ cnt = a.cnt;
    float* __restrict__ scores_out = a.scores_out;

    const int b = bh / Hq, h = bh % Hq;
    const int Hkv = Hq / G;
    const float* kbase = KIN ? nullptr : kp + (int64_t)(b * Hkv + h / G) * ((NBk + 31) >> 5) * (32 * D);   // tiles, see key_layout
    const float* lvbase = lvn != nullptr ? lvn + (int64_t)(b * Hkv + h / G) * NBk : nullptr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i_last = (i0 + R - 1 < NB - 1) ? i0 + R - 1 : NB - 1;
    const int n_jt = ((i_last + off) >> 5) + 1;           // 32-wide key-block tiles with some causal j

    // ---- phase 0 / phase 1 ------------------------------------------------------------
    stage_queries<D, R, R * LD, NWV, GROUP>(a, bh, i0, S);
    const __bf16* const qlds = reinterpret_cast<const __bf16*>(S + R * LD);
    if constexpr (KIN > 0) {                              // one tile, pooled by the workgroup itself, KIN tokens a block
        constexpr int part_at = 2 * (NWV / 4) * (256 / (D / 8)) * D <= R * LD ? 0 : R * LD + NWV * 256;
        float* const tile = S + key_tile_at<D, R, LD, NWV>();
        const int Skv_b = keys->Skv - a.S + entry_len(a.seq_lens, b, a.S);
        const uint16_t* const kh = keys->k + b * keys->ks.b + (h / G) * keys->ks.h;
        int n_blk = (Skv_b + KIN - 1) / KIN;              // the entry's blocks; causally visible ones
        n_blk = n_blk < i_last + off + 1 ? n_blk : i_last + off + 1;
        // an empty entry has no blocks: its rows get empty lists
        if (n_blk > 0) stage_keys<D, KIN, NWV>(kh, keys->ks.t, n_blk, Skv_b, S + part_at, reinterpret_cast<__bf16*>(tile));
        kbase = tile;
    }
    score_tiles<D, R, LD, D / 16, NWV>(a, kbase, qlds, S, 0, wave, n_jt, bh, i0, lvbase);
    if (scores_out != nullptr) {                          // key blocks past the last computed tile
        const int j_first = 32 * n_jt;
        for (int r = 0; r < R && i0 + r < NB; ++r)
            for (int j = j_first + (int)threadIdx.x; j < NBk; j += NWV * 64)
                scores_out[((int64_t)bh * NB + i0 + r) * NBk + j] = -INFINITY;
    }
    __syncthreads();

    // ---- phase 2 ---------------------------------------------------------------------
    head_config(head_pattern, h, pt, k);
    // ragged batch: this entry's own block count; its rows beyond get empty lists, and the dense
    // strip of the Tri-shape means the entry's own last rows
    const int NB_b = (entry_len(a.seq_lens, b, a.S) + a.Bs - 1) / a.Bs;
    pt.NB = off + NB_b;
#pragma nounroll
    for (int r = wave; r < R; r += NWV) {
        const int iq = i0 + r;                            // query block of the call
        if (iq >= NB) break;                              // wave-uniform
        if (iq >= NB_b) {
            const int64_t row = (int64_t)bh * NB + iq;
            for (int t = lane; t < T; t += 64) idx[row * T + t] = -1;
            if (lane == 0) cnt[row] = 0;
            continue;
        }
        const int i = iq + off;                           // its block position in the sequence
        const int n = i + 1;
        const float* srow = S + r * LD;
        // keys and static flags of the row's blocks stay in registers until the lists are written;
        // rows are causal: a row early in the sequence fills only its first chunks of 64 blocks
        const int chunks = (n + 63) >> 6;                 // wave-uniform
        int k_i = row_budget(k_rows, iq, k);
        const int64_t row = (int64_t)bh * NB + iq;
        int32_t* idx_row = idx + row * T;
        float x[BEST ? MAXC : 1];
        if constexpr (BEST) {
            static_for_sel<4>([&](auto q_tag) {
                constexpr int q = decltype(q_tag)::value, Q = MAXC / 4;
                if (q * Q >= chunks) return;
#pragma unroll
                for (int m = q * Q; m < (q + 1) * Q; ++m) x[m] = srow[(m << 6) + lane];
            });
            if (!EXT || plain_row(pt, i)) {
                const int c0 = pt.ns < n ? pt.ns : n, c1 = i - pt.nl + 1 > c0 ? i - pt.nl + 1 : c0;
                const int kk = k_i < c1 - c0 ? k_i : c1 - c0;
                if (take_best<MAXC>(x, i, c0, c1, kk, T, reinterpret_cast<float2*>(S + r * LD), idx_row, cnt + row, lane)) continue;
            }
        }
        uint32_t key[MAXC];
        uint64_t is_static_bits = 0ull;                   // bit m: block 64 m + lane is static
#pragma unroll
        for (int m = 0; m < MAXC; ++m) {
            key[m] = 0u;
            if (m < chunks) {
                const int j = (m << 6) + lane;            // < MAXC*64 <= LD: always inside the row
                const bool st = j <= i && static_block<EXT>(pt, i, j);
                const uint32_t kv = rank_key(BEST ? x[BEST ? m : 0] : srow[j]);    // columns past the computed tiles hold junk: masked next
                key[m] = (j <= i && !st) ? kv : 0u;
                is_static_bits |= st ? (1ull << m) : 0ull;
            }
        }
        int n_cand;
        if constexpr (EXT) {                              // count the candidates: no closed form worth having
            int ncl = 0;
#pragma unroll
            for (int m = 0; m < MAXC; ++m) ncl += key[m] != 0u ? 1 : 0;
            n_cand = wave_sum(ncl);
        } else {
            const int lo = i - pt.nl + 1;
            int n_sink = pt.ns < n ? pt.ns : n;
            int n_local = pt.nl < n ? pt.nl : n;
            int first_local = lo > 0 ? lo : 0;
            int overlap = n_sink - first_local; if (overlap < 0) overlap = 0;
            n_cand = n - (n_sink + n_local - overlap);
        }
        uint32_t* hist = reinterpret_cast<uint32_t*>(S + R * LD) + 256 * wave;
        if constexpr (MASS) {                             // the mass budget on top of the count budgets
            int k_m;                                      // rows of up to 2048 blocks: weights kept in registers
            if constexpr (MAXC <= 32)
                k_m = mass_budget_regs<MAXC>(key, is_static_bits, [&](int j) { return srow[j]; }, i, chunks, a.gamma_q16, k_i, hist, lane);
            else
                k_m = mass_budget_row<EXT>([&](int j) { return srow[j]; }, i, pt, a.gamma_q16, hist, lane);
            k_i = k_m < k_i ? k_m : k_i;
        }
        const int kk = k_i < n_cand ? k_i : n_cand;
        uint32_t thr;
        int need_eq;
        const int nc4 = 4 * chunks;
        if (nc4 <= MAXC) find_threshold_hist<MAXC, (MAXC + 3) / 4>(key, kk, n_cand, hist, lane, thr, need_eq);
        else if (nc4 <= 2 * MAXC) find_threshold_hist<MAXC, (MAXC + 1) / 2>(key, kk, n_cand, hist, lane, thr, need_eq);
        else if (nc4 <= 3 * MAXC) find_threshold_hist<MAXC, (3 * MAXC + 3) / 4>(key, kk, n_cand, hist, lane, thr, need_eq);
        else find_threshold_hist<MAXC, MAXC>(key, kk, n_cand, hist, lane, thr, need_eq);

        // emit static U top-k in ascending block order
        int eq_seen = 0, out_pos = 0;
#pragma unroll
        for (int m = 0; m < MAXC; ++m) {
            if (m < chunks) {
                const uint32_t kv = key[m];
                const bool is_eq = need_eq > 0 && kv == thr && kv != 0u;
                const uint64_t eq_mask = __ballot(is_eq);
                const bool take = ((is_static_bits >> m) & 1ull) != 0ull || (kv != 0u && kv > thr) ||
                                  (is_eq && eq_seen + lanes_below(eq_mask, lane) < need_eq);
                const uint64_t take_mask = __ballot(take);
                if (take) idx_row[out_pos + lanes_below(take_mask, lane)] = (m << 6) + lane;
                eq_seen += __popcll(eq_mask);
                out_pos += __popcll(take_mask);
            }
        }
        for (int t = out_pos + lane; t < T; t += 64) idx_row[t] = -1;
        if (lane == 0) cnt[row] = out_pos;
    }
}

// Column-chunked variant for rows of 1025 .. 2048 key blocks: R = 16 query blocks per workgroup, as
// for 1024-block rows, so that every pooled-K tile a workgroup reads from L2 serves 16 rows (8-row
// workgroups re-read the pooled K twice as often: 5.2 GB against the 2.7 GB Q stream at 262144
// tokens, and use a quarter of every MFMA), while the scores in LDS stay those of one chunk of
// CW = 1024 key blocks: 66 KB, two workgroups per CU.  A wavefront owns two rows; the scores of the
// first chunk wait in registers (16 per lane and row) while the second chunk is scored, then each
// row is selected exactly as in the plain kernel, from 32 scores per lane.  (No cumulative-mass
// variant: that budget keeps the 8-row kernel.)
template <int D, int R, int MAXCH, bool EXT, int NWV, bool GROUP, bool BEST>
__device__ __forceinline__ void score_topk_rows_chunked(const ScoreArgs& a, const int bh, const int i0, float* S) {
    constexpr int CC = 16;                     // 64-block register chunks per column chunk
    constexpr int CW = CC * 64;                // key blocks per column chunk
    constexpr int LD = CW + row_pad(D, R);
    constexpr int RPW = R / NWV;               // rows per wavefront
    constexpr int MAXC = MAXCH * CC;
    static_assert(R % NWV == 0 && MAXCH == 2, "two column chunks");
    const float* __restrict__ kp = a.kp;
    const int Hq = a.Hq, G = a.G, NB = a.NB, NBk = a.NBk, off = a.off, T = a.T;
    Pattern pt = a.pt;
    int k = a.k;
    int32_t* __restrict__ idx = a.idx;
    int32_t* __restrict__ cnt = a.cnt;
    float* __restrict__ scores_out = a.scores_out;

    const int b = bh / Hq, h = bh % Hq;
    const int Hkv = Hq / G;
    const float* kbase = kp + (int64_t)(b * Hkv + h / G) * ((NBk + 31) >> 5) * (32 * D);
    const float* lvbase = a.lvn != nullptr ? a.lvn + (int64_t)(b * Hkv + h / G) * NBk : nullptr;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i_last = (i0 + R - 1 < NB - 1) ? i0 + R - 1 : NB - 1;
    const int n_jt = ((i_last + off) >> 5) + 1;           // 32-wide key-block tiles with some causal j
    const int n_ch = (i_last + off) / CW + 1;             // column chunks with some causal j (workgroup-uniform)

    stage_queries<D, R, R * LD, NWV, GROUP>(a, bh, i0, S);
    const __bf16* const qlds = reinterpret_cast<const __bf16*>(S + R * LD);

    head_config(a.head_pattern, h, pt, k);
    const int NB_b = (entry_len(a.seq_lens, b, a.S) + a.Bs - 1) / a.Bs;      // ragged batch
    pt.NB = off + NB_b;

    // Scores of column chunk c into S; of the second one with half a tile in registers, when 32 registers per lane hold the first
    // one's scores
    auto score_chunk = [&](int c, auto nbuf_tag) {
        const int jt_end = n_jt < (c + 1) * (CW / 32) ? n_jt : (c + 1) * (CW / 32);
        score_tiles<D, R, LD, decltype(nbuf_tag)::value, NWV>(a, kbase, qlds, S, c * CW, c * (CW / 32) + wave, jt_end, bh, i0, lvbase);
    };
    // scores of the blocks c * CW + 64 m + lane of row r from the chunk's scores in S (columns past the
    // computed tiles hold junk; they lie beyond the causal limit and are never candidates)
    auto load_scores = [&](int r, float* x) {
        const float* srow = S + r * LD;
#pragma unroll
        for (int m = 0; m < CC; ++m) x[m] = srow[(m << 6) + lane];
    };

    float x0[RPW][CC];                                    // first-chunk scores of this wavefront's rows
#pragma unroll
    for (int rr = 0; rr < RPW; ++rr)
#pragma unroll
        for (int m = 0; m < CC; ++m) x0[rr][m] = -INFINITY;
    score_chunk(0, IC_sel<D / 16>{});
    __syncthreads();
    if (n_ch > 1) {                                       // workgroup-uniform
#pragma unroll
        for (int rr = 0; rr < RPW; ++rr) {
            const int iq = i0 + wave + rr * NWV;
            if (iq < NB && iq < NB_b) load_scores(wave + rr * NWV, x0[rr]);
        }
        __syncthreads();                                  // every row's first-chunk scores are in registers
        score_chunk(1, IC_sel<D / 32>{});
        __syncthreads();
    }
    if (scores_out != nullptr) {                          // key blocks past the last computed tile
        const int j_first = 32 * n_jt;
        for (int r = 0; r < R && i0 + r < NB; ++r)
            for (int j = j_first + (int)threadIdx.x; j < NBk; j += NWV * 64)
                scores_out[((int64_t)bh * NB + i0 + r) * NBk + j] = -INFINITY;
    }

    // ---- selection, row by row, as in the plain kernel; the staged queries are not needed any more,
    // their space holds the counters of the search ----
    uint32_t* const hist = reinterpret_cast<uint32_t*>(S + R * LD) + 256 * wave;
    static_for_sel<RPW>([&](auto rr_tag) {
        constexpr int rr = decltype(rr_tag)::value;
        const int r = wave + rr * NWV;
        const int iq = i0 + r;
        if (iq >= NB) return;                             // wave-uniform
        const int64_t row = (int64_t)bh * NB + iq;
        int32_t* idx_row = idx + row * T;
        if (iq >= NB_b) {                                 // past the entry's end: empty list
            for (int t = lane; t < T; t += 64) idx_row[t] = -1;
            if (lane == 0) cnt[row] = 0;
            return;
        }
        const int i = iq + off;
        const int n = i + 1;
        const int chunks = (n + 63) >> 6;
        float x[MAXC];
        if (n_ch > 1) {
#pragma unroll
            for (int m = 0; m < CC; ++m) x[m] = x0[rr][m];
            load_scores(r, x + CC);
        } else {
            load_scores(r, x);
#pragma unroll
            for (int m = CC; m < MAXC; ++m) x[m] = -INFINITY;
        }
        const int k_i = row_budget(a.k_rows, iq, k);
        if (BEST && (!EXT || plain_row(pt, i))) {
            const int c0 = pt.ns < n ? pt.ns : n, c1 = i - pt.nl + 1 > c0 ? i - pt.nl + 1 : c0;
            const int kk = k_i < c1 - c0 ? k_i : c1 - c0;
            if (take_best<MAXC>(x, i, c0, c1, kk, T, reinterpret_cast<float2*>(S + r * LD), idx_row, cnt + row, lane)) return;
        }
        {
            uint32_t key[MAXC];
            uint64_t is_static_bits = 0ull;
            int ncl = 0;
#pragma unroll
            for (int m = 0; m < MAXC; ++m) {
                key[m] = 0u;
                if (m < chunks) {
                    const int j = (m << 6) + lane;
                    const bool st = j <= i && static_block<EXT>(pt, i, j);
                    key[m] = (j <= i && !st) ? rank_key(x[m]) : 0u;
                    is_static_bits |= st ? (1ull << m) : 0ull;
                    if constexpr (EXT) ncl += key[m] != 0u ? 1 : 0;
                }
            }
            int n_cand;
            if constexpr (EXT) {
                n_cand = wave_sum(ncl);
            } else {                                      // sinks 0 .. ns-1, window i-nl+1 .. i, the rest are candidates
                const int n_sink = pt.ns < n ? pt.ns : n;
                const int first_local = i - pt.nl + 1 > n_sink ? i - pt.nl + 1 : n_sink;
                n_cand = first_local - n_sink;
            }
            const int kk = k_i < n_cand ? k_i : n_cand;
            uint32_t thr;
            int need_eq;
            const int nc4 = 4 * chunks;
            if (nc4 <= MAXC) find_threshold_hist<MAXC, (MAXC + 3) / 4>(key, kk, n_cand, hist, lane, thr, need_eq);
            else if (nc4 <= 2 * MAXC) find_threshold_hist<MAXC, (MAXC + 1) / 2>(key, kk, n_cand, hist, lane, thr, need_eq);
            else if (nc4 <= 3 * MAXC) find_threshold_hist<MAXC, (3 * MAXC + 3) / 4>(key, kk, n_cand, hist, lane, thr, need_eq);
            else find_threshold_hist<MAXC, MAXC>(key, kk, n_cand, hist, lane, thr, need_eq);
            int eq_seen = 0, out_pos = 0;
#pragma unroll
            for (int m = 0; m < MAXC; ++m) {
                if (m < chunks) {
                    const uint32_t kv = key[m];
                    const bool is_eq = need_eq > 0 && kv == thr && kv != 0u;
                    const uint64_t eq_mask = __ballot(is_eq);
                    const bool take = ((is_static_bits >> m) & 1ull) != 0ull || (kv != 0u && kv > thr) ||
                                      (is_eq && eq_seen + lanes_below(eq_mask, lane) < need_eq);
                    const uint64_t take_mask = __ballot(take);
                    if (take) idx_row[out_pos + lanes_below(take_mask, lane)] = (m << 6) + lane;
                    eq_seen += __popcll(eq_mask);
                    out_pos += __popcll(take_mask);
                }
            }
            for (int t = out_pos + lane; t < T; t += 64) idx_row[t] = -1;
            if (lane == 0) cnt[row] = out_pos;
        }
    });
}

template <int D, int R, int MAXCH, bool EXT, int NWV, bool GROUP, bool BEST>
__global__ __launch_bounds__(NWV * 64, 4) void score_topk_chunked_kernel(ScoreArgs a, int n_tiles) {
    extern __shared__ __attribute__((aligned(128))) float S[];   // [R][1024 + row_pad] scores of one column chunk, then the staged queries
    const int nwg = gridDim.x;
    int wg = blockIdx.x;
    if ((nwg & 7) == 0) wg = (wg & 7) * (nwg >> 3) + (wg >> 3);   // each XCD a contiguous slice, as in the plain kernel
    const int tile = n_tiles - 1 - wg % n_tiles;          // long rows first
    score_topk_rows_chunked<D, R, MAXCH, EXT, NWV, GROUP, BEST>(a, wg / n_tiles, tile * R, S);
}

// Two workgroups per CU (4 wavefronts per SIMD): at most 128 registers, which is why the query
// operands are staged in LDS.
template <int D, int R, int MAXC, bool EXT, bool MASS, int NWV, bool GROUP, bool BEST>
__global__ __launch_bounds__(NWV * 64, 4) void score_topk_mfma_kernel(ScoreArgs a, int n_tiles) {
    extern __shared__ __attribute__((aligned(128))) float S[];   // [R][LD] scores of this workgroup's rows, then 256 counters per wave
    // Workgroup ids go round robin over the 8 XCDs; give each XCD a contiguous slice of the
    // (b, head, row tile) order so that one L2 serves few KV heads and their Kp stays resident.
    const int nwg = gridDim.x;
    int wg = blockIdx.x;
    if ((nwg & 7) == 0) wg = (wg & 7) * (nwg >> 3) + (wg >> 3);
    const int tile = n_tiles - 1 - wg % n_tiles;          // long rows first
    score_topk_rows<D, R, MAXC, EXT, MASS, NWV, GROUP, BEST>(a, wg / n_tiles, tile * R, S);
}

// Small calls (small_call): one launch instead of prepare_kv_kernel (or pool_kernel) and the score kernel.  Every workgroup pools the K blocks
// its rows can see itself, from L2, and the workgroups behind the first n_score transpose two blocks of V each.
// Bound by launches and latency.  Against two launches 512 tokens of one head, head_dim 64, blocks of 64, took 16.8 us instead of 18.8; with all of
// a workgroup's K in flight at once 16.2 (replayed from a graph 16.3 -> 15.5; 300 tokens of 32/8 heads 15.4 -> 14.7, 384 tokens with head_dim 128,
// blocks of 128, 21.3 -> 20.4).  Batches of short prompts have up to 2048 workgroups, so as many share a CU as its LDS holds: two, three with
// head_dim 64, within 128 and 80 registers.
template <int D, int BS, bool EXT>
__global__ __launch_bounds__(512, D == 64 ? 6 : 4) void score_topk_small_kernel(ScoreArgs a, KeyArgs keys, int n_tiles, int n_score) {
    extern __shared__ __attribute__((aligned(128))) float S[];
    constexpr int R = 4, NWV = 8;
    const int wg = blockIdx.x;
    if (wg < n_score) {
        score_topk_rows<D, R, 4, EXT, false, NWV, false, false, BS>(a, wg / n_tiles, (n_tiles - 1 - wg % n_tiles) * R, S, &keys);
        return;
    }
    const int half = threadIdx.x >> 8, x = 2 * (wg - n_score) + half;        // block of V
    const int hy = x / a.NBk, blk = x % a.NBk;
    const int b = hy / keys.Hkv, h = hy % keys.Hkv;
    const int Sb = hy < keys.n_heads ? keys.Skv - a.S + entry_len(a.seq_lens, b, a.S) : 0;
    int n_valid = Sb - blk * BS;
    n_valid = n_valid < 0 ? 0 : (n_valid > BS ? BS : n_valid);
    const uint16_t* src = keys.v + (n_valid > 0 ? b * keys.vs.b + h * keys.vs.h + (int64_t)blk * BS * keys.vs.t : 0);
    uint16_t* dst = keys.vt + (int64_t)x * D * BS;
    uint16_t* tile = reinterpret_cast<uint16_t*>(S) + half * (BS * (D + 2));
    const int tid = threadIdx.x & 255;
    value_block<D, BS, true, false>(tid, src, keys.vs.t, n_valid, tile, nullptr, dst, keys.halves, nullptr);
}

// Dynamic LDS above the default cap has to be requested per kernel and device.  That is done on the
// first launch of a (kernel, device) pair and remembered: later launches, also those recorded into a
// stream capture, make no runtime call besides the launch itself.
hipError_t allow_lds(const void* kernel, size_t bytes) {
    if (bytes <= 32768) return hipSuccess;
    struct Granted { const void* kernel; int device; size_t bytes; };
    static std::mutex mu;
    static std::vector<Granted> granted;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    for (Granted& g : granted)
        if (g.kernel == kernel && g.device == dev) {
            if (g.bytes >= bytes) return hipSuccess;
            e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
            if (e == hipSuccess) g.bytes = bytes;
            return e;
        }
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) granted.push_back(Granted{kernel, dev, bytes});
    return e;
}

ScoreArgs score_args(const Dims& d, const float* kp, const int32_t* k_rows, const int32_t* head_pattern,
                     const float* lvn, int32_t* idx, int32_t* cnt, float* scores_or_null, const void* q, Strides qs,
                     int group, const float* qp) {
    return ScoreArgs{kp, d.Hq, d.G, d.NB, d.NBk, d.off, pattern_of(d), d.k, k_rows, head_pattern, lvn, d.T, d.scale,
                     idx, cnt, scores_or_null, d.gamma_q16 >= 0 ? (uint32_t)d.gamma_q16 : 0u, d.seq_lens, d.S, d.Bs, (const uint16_t*)q, qs, group, qp};
}

size_t keys_lds_bytes(int NB) { return (size_t)kWaves * (((NB + 63) >> 6) << 6) * sizeof(uint32_t); }

}  // namespace

#define SPA_SCORE_TOPK_ARGS const Dims& d, const float* kp, const int32_t* k_rows, const int32_t* head_pattern, \
    const float* lvn, int32_t* idx, int32_t* cnt, float* scores_or_null, const void* q, Strides qs, int group, const float* qp, hipStream_t st

#define SPA_SCORE_SMALL_ARGS const Dims& d, const void* q, Strides qs, const void* k, Strides ks, const void* v, Strides vs, void* vt_or_null, \
    const int32_t* k_rows, const int32_t* head_pattern, int32_t* idx, int32_t* cnt, float* scores_or_null, hipStream_t st

#ifdef SPA_SELECT_D
namespace {
// one call of the score / top-k kernel
struct ScoreCall {
    const Dims& d;
    ScoreArgs a;
    hipStream_t st;
};

template <int D, int R, int MAXC, bool EXT, bool MASS, bool GROUP, bool BEST = false, int NWV = (R * (MAXC * 64 + row_pad(D, R)) * 4 > 80 * 1024 ? 16 : 8)>
hipError_t launch_mfma_e(const ScoreCall& c) {
    constexpr size_t part_words = 2 * (NWV / 4) * (256 / (D / 8)) * D;    // partial sums of the in-kernel pooling
    constexpr size_t lds = ((size_t)R * (MAXC * 64 + row_pad(D, R)) + NWV * 256 +
                            (part_words > (size_t)R * (MAXC * 64 + row_pad(D, R)) ? part_words : 0)) * sizeof(float);
    hipError_t e = allow_lds((const void*)score_topk_mfma_kernel<D, R, MAXC, EXT, MASS, NWV, GROUP, BEST>, lds);
    if constexpr (!MASS && !GROUP && has_lists_by_bound(R, MAXC))         // a capture may follow calls with another budget, which is the other kernel
        if (e == hipSuccess) e = allow_lds((const void*)score_topk_mfma_kernel<D, R, MAXC, EXT, MASS, NWV, GROUP, !BEST>, lds);
    if (e != hipSuccess) return e;
    const int n_tiles = (c.d.NB + R - 1) / R;
    dim3 grid((unsigned)(n_tiles * c.d.B * c.d.Hq));
    hipLaunchKernelGGL((score_topk_mfma_kernel<D, R, MAXC, EXT, MASS, NWV, GROUP, BEST>), grid, dim3(NWV * 64), lds, c.st, c.a, n_tiles);
    return hipGetLastError();
}

template <int D, int R, int MAXC, bool EXT, bool MASS>
hipError_t launch_mfma_q(const ScoreCall& c) {
    if (c.a.group > 1) return launch_mfma_e<D, R, MAXC, EXT, MASS, true>(c);
    if constexpr (!MASS && has_lists_by_bound(R, MAXC))
        if (lists_by_bound(c.d)) return launch_mfma_e<D, R, MAXC, EXT, MASS, false, true>(c);
    return launch_mfma_e<D, R, MAXC, EXT, MASS, false>(c);
}

template <int D, int MAXCH, bool EXT, bool GROUP, bool BEST = false>
hipError_t launch_chunked_e(const ScoreCall& c) {
    constexpr int R = 16, NWV = 8;
    constexpr size_t lds = ((size_t)R * (1024 + row_pad(D, R)) + NWV * 256) * sizeof(float);
    static_assert(2 * (NWV / 4) * (256 / (D / 8)) * D <= R * (1024 + row_pad(D, R)), "the pooling partial sums fit the score space");
    hipError_t e = allow_lds((const void*)score_topk_chunked_kernel<D, R, MAXCH, EXT, NWV, GROUP, BEST>, lds);
    if constexpr (!GROUP)
        if (e == hipSuccess) e = allow_lds((const void*)score_topk_chunked_kernel<D, R, MAXCH, EXT, NWV, GROUP, !BEST>, lds);
    if (e != hipSuccess) return e;
    const int n_tiles = (c.d.NB + R - 1) / R;
    dim3 grid((unsigned)(n_tiles * c.d.B * c.d.Hq));
    hipLaunchKernelGGL((score_topk_chunked_kernel<D, R, MAXCH, EXT, NWV, GROUP, BEST>), grid, dim3(NWV * 64), lds, c.st, c.a, n_tiles);
    return hipGetLastError();
}

template <int D, int MAXCH>
hipError_t launch_chunked(const ScoreCall& c) {
    const bool group = c.a.group > 1, best = lists_by_bound(c.d), ext = extended(c.d);
    if (group) return ext ? launch_chunked_e<D, MAXCH, true, true>(c) : launch_chunked_e<D, MAXCH, false, true>(c);
    if (best) return ext ? launch_chunked_e<D, MAXCH, true, false, true>(c) : launch_chunked_e<D, MAXCH, false, false, true>(c);
    return ext ? launch_chunked_e<D, MAXCH, true, false>(c) : launch_chunked_e<D, MAXCH, false, false>(c);
}

template <int D, int R, int MAXC>
hipError_t launch_mfma(const ScoreCall& c) {
    const bool mass = c.d.gamma_q16 >= 0;
    if (extended(c.d)) return mass ? launch_mfma_q<D, R, MAXC, true, true>(c) : launch_mfma_q<D, R, MAXC, true, false>(c);
    return mass ? launch_mfma_q<D, R, MAXC, false, true>(c) : launch_mfma_q<D, R, MAXC, false, false>(c);
}

// without the mass-budget kernels
template <int D, int R, int MAXC>
hipError_t launch_plain(const ScoreCall& c) {
    return extended(c.d) ? launch_mfma_q<D, R, MAXC, true, false>(c) : launch_mfma_q<D, R, MAXC, false, false>(c);
}

// LDS of a small call's workgroups: those that score, those that transpose V
template <int D>
constexpr size_t small_score_lds() { return (key_tile_at<D, 4, 4 * 64 + row_pad(D, 4), 8>() + 32 * D) * sizeof(float); }
template <int D, int BS>
constexpr size_t small_v_lds() { return 2 * BS * (D + 2) * sizeof(uint16_t); }
template <int D, int BS, bool EXT>
hipError_t allow_small_lds() {
    return allow_lds((const void*)score_topk_small_kernel<D, BS, EXT>, small_v_lds<D, BS>() > small_score_lds<D>() ? small_v_lds<D, BS>() : small_score_lds<D>());
}

template <int D, int BS, bool EXT>
hipError_t launch_small_e(const ScoreCall& c, const KeyArgs& keys) {
    if (c.d.NBk > most_small_blocks(D, BS)) return hipErrorInvalidValue;
    const size_t v_lds = keys.vt != nullptr ? small_v_lds<D, BS>() : 0;
    const size_t lds = v_lds > small_score_lds<D>() ? v_lds : small_score_lds<D>();
    // asked for once, for the largest call and for both block sizes: a fused call in a capture may follow calls that need less, or another kernel
    hipError_t e = allow_small_lds<D, 64, EXT>();
    if (e == hipSuccess) e = allow_small_lds<D, 128, EXT>();
    if (e != hipSuccess) return e;
    const int n_tiles = (c.d.NB + 3) / 4, n_score = n_tiles * c.d.B * c.d.Hq;
    const int n_v = keys.vt != nullptr ? (c.d.B * c.d.Hkv * c.d.NBk + 1) / 2 : 0;
    hipLaunchKernelGGL((score_topk_small_kernel<D, BS, EXT>), dim3((unsigned)(n_score + n_v)), dim3(512), lds, c.st, c.a, keys, n_tiles, n_score);
    return hipGetLastError();
}

template <int D>
hipError_t launch_mfma_d(const ScoreCall& c) {
    const int NBk = c.d.NBk, R = score_rows(c.d);
    if (NBk <= 256) return R == 4 ? launch_plain<D, 4, 4>(c) : launch_mfma<D, 8, 4>(c);
    if (NBk <= 512) return R == 4 ? launch_plain<D, 4, 8>(c) : launch_mfma<D, 8, 8>(c);
    if (NBk <= 1024) return R == 4 ? launch_plain<D, 4, 16>(c) : R == 8 ? launch_plain<D, 8, 16>(c) : launch_mfma<D, 16, 16>(c);
    if (NBk <= 2048) return R == 4 ? launch_plain<D, 4, 32>(c) : R == 8 ? launch_mfma<D, 8, 32>(c) : launch_chunked<D, 2>(c);
    return launch_mfma<D, 4, 64>(c);
}

}  // namespace

#define SPA_CAT2(a, b) a##b
#define SPA_CAT(a, b) SPA_CAT2(a, b)
hipError_t SPA_CAT(launch_score_topk_d, SPA_SELECT_D)(SPA_SCORE_TOPK_ARGS) {
    const ScoreCall c{d, score_args(d, kp, k_rows, head_pattern, lvn, idx, cnt, scores_or_null, q, qs, group, qp), st};
    return launch_mfma_d<SPA_SELECT_D>(c);
}
hipError_t SPA_CAT(launch_score_small_d, SPA_SELECT_D)(SPA_SCORE_SMALL_ARGS) {
    const ScoreCall c{d, score_args(d, nullptr, k_rows, head_pattern, nullptr, idx, cnt, scores_or_null, q, qs, 1, nullptr), st};
    const KeyArgs keys{(const uint16_t*)k, ks, (const uint16_t*)v, vs, (uint16_t*)vt_or_null, d.Skv, d.Hkv, vt_in_halves(d) ? 1 : 0, d.B * d.Hkv};
    const bool ext = extended(d);
    if (d.Bs == 128) return ext ? launch_small_e<SPA_SELECT_D, 128, true>(c, keys) : launch_small_e<SPA_SELECT_D, 128, false>(c, keys);
    return ext ? launch_small_e<SPA_SELECT_D, 64, true>(c, keys) : launch_small_e<SPA_SELECT_D, 64, false>(c, keys);
}

#else
hipError_t launch_score_topk_d128(SPA_SCORE_TOPK_ARGS);
hipError_t launch_score_small_d128(SPA_SCORE_SMALL_ARGS);
hipError_t launch_score_small_d64(SPA_SCORE_SMALL_ARGS);
hipError_t launch_score_topk_d64(SPA_SCORE_TOPK_ARGS);

hipError_t launch_topk_from_scores(const Dims& d, const float* scores, const int32_t* k_rows,
                                   const int32_t* head_pattern, int32_t* idx, int32_t* cnt, hipStream_t st) {
    int64_t n_rows = (int64_t)d.B * d.Hq * d.NB;
    unsigned grid = (unsigned)((n_rows + kWaves - 1) / kWaves);
    const void* fn = extended(d) ? (const void*)topk_from_scores_kernel<true> : (const void*)topk_from_scores_kernel<false>;
    const size_t lds = keys_lds_bytes(d.NBk) + (d.gamma_q16 >= 0 ? kWaves * 256 * sizeof(uint32_t) : 0);
    hipError_t e = allow_lds(fn, lds);
    if (e != hipSuccess) return e;
    if (extended(d))
        hipLaunchKernelGGL(topk_from_scores_kernel<true>, dim3(grid), dim3(kWaves * 64), lds, st,
                           scores, n_rows, d.NB, d.NBk, d.off, pattern_of(d), d.k, k_rows, head_pattern, d.Hq, d.T, idx, cnt, d.gamma_q16, d.seq_lens, d.S, d.Bs);
    else
        hipLaunchKernelGGL(topk_from_scores_kernel<false>, dim3(grid), dim3(kWaves * 64), lds, st,
                           scores, n_rows, d.NB, d.NBk, d.off, pattern_of(d), d.k, k_rows, head_pattern, d.Hq, d.T, idx, cnt, d.gamma_q16, d.seq_lens, d.S, d.Bs);
    return hipGetLastError();
}

hipError_t launch_score_topk(SPA_SCORE_TOPK_ARGS) {
    if (d.D == 128) return launch_score_topk_d128(d, kp, k_rows, head_pattern, lvn, idx, cnt, scores_or_null, q, qs, group, qp, st);
    if (d.D == 64) return launch_score_topk_d64(d, kp, k_rows, head_pattern, lvn, idx, cnt, scores_or_null, q, qs, group, qp, st);
    return hipErrorInvalidValue;
}

hipError_t launch_score_small(SPA_SCORE_SMALL_ARGS) {
    if (d.D == 128) return launch_score_small_d128(d, q, qs, k, ks, v, vs, vt_or_null, k_rows, head_pattern, idx, cnt, scores_or_null, st);
    if (d.D == 64) return launch_score_small_d64(d, q, qs, k, ks, v, vs, vt_or_null, k_rows, head_pattern, idx, cnt, scores_or_null, st);
    return hipErrorInvalidValue;
}
#endif

}  // namespace spa
