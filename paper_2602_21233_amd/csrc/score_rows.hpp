// How many query blocks (rows) a workgroup of the score / selection kernel takes: the rule, for the launcher.
#pragma once
#include "common.hpp"

namespace spa {

// What the score kernel selects for a call: with one list per KV head as if the KV heads were the query heads; shared: several heads share
// one
inline Dims list_dims(Dims d) {
    if (!d.shared) return d;
    d.shared = d.G > 1;
    d.Hq = d.Hkv;
    d.G = 1;
    return d;
}

// Rows per workgroup for the lists d (list_dims): 4, 8 or 16; 16 with more than 1024 key blocks is the kernel that scores the columns in two
// chunks.  Fewer rows as rows get longer: up to 1024 blocks R * (NB padded) fp32 scores stay within 66 KB of LDS, so that two 8-wave
// workgroups share a CU (measured at 131072 tokens: 125 -> 106 us against 32 rows with one 8-wave workgroup per CU).
inline int score_rows(const Dims& d) {
    const int64_t heads = (int64_t)d.B * d.Hq, rows = heads * d.NB;
    const bool plain = d.gamma_q16 < 0;
    if (d.NBk > 2048) return 4;
    // Few rows (a chunk over a long prefix, a short prompt): 4 per workgroup, or most CUs would be idle while a few pool, score and select 8
    // or 16 rows one after the other.  Up to 1024 rows, where 8 per workgroup give half of the CUs one; 1.05 to 1.1 times the time of 8 from
    // 2048 rows on.  Whole select calls, 32 heads: 2048 queries over 29952 tokens 25.9 -> 23.1 us, over 98304 tokens 67 -> 53 (34 of them
    // pool K), over 131072 tokens 85 -> 67. Lists shared by several heads, whose workgroups stream the queries of all of them: up to 2048
    // rows (2040 rows, 8 against 4 per workgroup: 32/8 heads 63.3 and 56.7 us, 16/8 40.6 and 38.4, 40/8 74.9 and 66.0; 1400 rows 45.1 and
    // 44.9, 29.0 and 30.2, 52.8 and 52.2). (A mass budget keeps the larger groups: its second search makes the kernels twice as many, for
    // rare calls.)
    if (plain && rows <= (d.shared ? 2048 : 1024)) return 4;
    // up to 512 blocks: 8 rows per workgroup give the chip more rounds of workgroups, so that one round's streaming overlaps another's
    // scoring (0.065 -> 0.062 ms at 32768 tokens, 0.135 -> 0.124 ms at 65536)
    if (d.NBk <= 512) return 8;
    const bool two_chunks = d.NBk > 1024;
    if (!plain) return two_chunks ? 8 : 16;
    // 513 .. 2048 blocks.  All figures from here on: select calls over 8 KV heads, us with 8 and with 16 rows.  The lines were drawn before the
    // 16-row kernels selected from lists by bound (take_best), which the 8-row ones do only beyond 1024 blocks, and have not been moved since:
    // some calls on the side of 8 now lose up to 13 % against 16.
    // Many rows: 16, as 8 re-read the pooled K twice as often (blocks of 128: 186 and 181 at 768 blocks and 24576 rows, 257 and 237 at 1024 and
    // 32768; 703 and 619 at 262144 tokens and 81920 rows, 326 and 304 at 163840 tokens and 40960, where 16 rows are scored in two chunks of
    // 1024 columns to keep two workgroups per CU; but 221 and 224 at 768 blocks and 30720 rows).
    if (rows > (two_chunks ? 32768 : 16384)) return 16;
    // Fewer: more workgroups, unless they only make more rounds.  With blocks of 128 the query stream, twice as long for a row, hides the
    // rounds, and 8 are the better choice up to 1024 blocks (8192 queries over 98304 tokens, 2048 rows, 62.7 and 68.2; 98304 tokens of 8 heads
    // 78.7 and 84.1; 131072 of 16 heads, 16384 rows, 154 and 162; but with head_dim 64 92.2 and 90.2).  In two chunks 16 have become the
    // better choice from about 20000 rows on (160 and 162 at 196608 tokens of 8 heads, 219 and 222 at 262144, but 197 and 189 at 163840 of 16
    // heads, 242 and 234 at 196608, 336 and 310 at 262144, 32768 rows) and over a long prefix (25600 queries over 230400 tokens, 172 and 158).
    if (d.Bs == 128) return 8;
    // With blocks of 64 the rounds of 512 workgroups (two per CU) show.  Up to 1.5 rounds of 8-row workgroups (6144 rows) 8 rows win (1600 rows
    // of 1000 blocks 45.5 and 50.3, 5120 of 640 43.4 and 46.9).  From there on:
    //   - over a prefix at least as long as the chunk all rows are about as long, and what counts is `depth`, how many of them a place works
    //     through one after the other: 16 where that is the same (12797 queries over 51200 tokens, 32 heads, 77.2 and 66.9; 25597 over 102400
    //     tokens, 40 heads, 183 and 150), 8 rows where that is less, which since lists by bound no longer pays (12797 over 51200 tokens, 40
    //     heads, 81.5 and 77.7, 19197 over 44800 103 and 89.6, 38397 over 51200 of 16 heads 102 and 95.7);
    //   - rows that differ in length are dealt longest first and even the rounds out.  8 rows win up to one round of 16-row workgroups (52413
    //     tokens of 8 heads 57.0 and 57.8) and, with head_dim 64 or two chunks, up to 14336 rows (95997 tokens of 8 heads 105 and 105; 47485
    //     tokens of 16 heads, head_dim 64, 47.3 and 48.9).  16 elsewhere: 113341 tokens of 16 heads, head_dim 64, 135 and 121, 28288 rows of 1247
    //     blocks 183 and 160, 64000 tokens of 16 heads 103 and 97.4, 40957 62.2 and 60.4.
    const int64_t wg8 = heads * ((d.NB + 7) / 8), wg16 = heads * ((d.NB + 15) / 16);
    if (wg8 <= 768) return 8;
    if (d.off >= d.NB) {
        const int64_t depth8 = (wg8 + 511) / 512 * 8, depth16 = (wg16 + 511) / 512 * 16;
        return depth8 < depth16 && rows <= 16384 ? 8 : 16;
    }
    return wg16 <= 512 || (rows <= 14336 && (two_chunks || d.D == 64)) ? 8 : 16;
}

// Is a call's kernel one that selects rows from a list of the blocks that reach a bound (take_best) where it can?  Not where no row does: static
// columns, more than 64 sinks, a budget too close to the 128 values that the bound is taken from.  And only where enough rows get one, as
// the others pay for both ways' instructions in one kernel (61437 tokens of 16 heads, head_dim 64, blocks of 64, 128 wanted and so the general
// way for all of them, 56.8 us in a kernel without lists, 61.5 in one with them).  Select calls, us without and with lists:
//   - up to 1024 blocks, 16 rows a workgroup, it takes rows of 352 blocks and more with the budget on average, less of that for many rows of head_dim
//     128: 40 heads from the first block on, head_dim 64, 64 wanted, 826 blocks of 64 105.5 and 107.5, 951 of 128 164.8 and 161.5; 32
//     heads, 8 wanted, 768 of 128 100.4 and 98.6; head_dim 128, blocks of 64, 32 heads, 64 wanted, 799 119.7 and 116.6, 670 99.1 and 99.6, 16
//     heads, 8 wanted, 700 53.1 and 55.2.  Over 900 random calls with such kernels this choice takes 0.15 % more time than the better one of
//     each, lists always 0.9, lists never 2.6 (at most 4, 10 and 19 %).
//   - beyond 1024 blocks all up to 124 wanted (116 to 124 wanted of 1025 to 1280 blocks 0.91 to 1.01 of the time without, of 1536 and more
//     0.84 to 0.98), and 128 of many long rows (more than 1536 blocks, more than 16384 rows 0.95 to 0.99; up to 16384 rows 0.96 to 1.06; 1025 to
//     1280 blocks 0.99 to 1.09).
constexpr int kFewWanted = 112;
constexpr bool has_lists_by_bound(int R, int max_chunks) { return max_chunks == 32 || (max_chunks == 16 && R == 16); }
inline bool lists_by_bound(const Dims& d) {
    if (d.gamma_q16 >= 0 || d.shared || d.stride > 0 || d.ns > 64 || d.NBk <= 512 || d.NBk > 2048) return false;
    const bool many = (int64_t)d.B * d.Hq * d.NB > 16384;
    if (d.NBk <= 1024) return score_rows(d) == 16 && d.k <= kFewWanted && d.off + d.NB / 2 >= 352 + (d.D == 128 && many ? d.k / 4 : d.k);
    return d.k <= 124 || (d.k <= 128 && d.NBk > 1536 && many);
}

// Which matrix products score R rows: 16x16x32 ones for 16 rows of head_dim 128, 32x32x16 ones, whose surplus rows are copies, for the
// others.  With 16 rows of head_dim 128 the former halve the matrix work and the LDS reads, and their 8 accumulators instead of 16 end the
// spills of the two-chunk kernel (select calls, 262144 tokens of 40/8 heads 759 -> 695 us, blocks of 64 2048 of 32 heads 431 -> 406, 1247 of
// 32 heads 185 -> 174).  With head_dim 64 nothing spilled, and they cost as much as they give (1771 blocks of 16 heads 133.9 -> 137.9 us,
// 131072 tokens of 32 heads 155.1 -> 157.7, 1000 blocks 112.0 -> 111.0).  With 4 or 8 rows few tiles fall to a wavefront (65536 tokens 117.5
// -> 120 us, with a mass budget 132 -> 137), and 32x32x16 products on the other's tiles, a quarter of a KB at a time, take 1 to 2.5 % longer
// (12800 queries over 51200 tokens, 40 heads, 89.4 -> 91.2).
constexpr bool sixteen_row_products(int D, int R) { return D == 128 && R == 16; }
inline KeyLayout key_layout(const Dims& d) { return sixteen_row_products(d.D, score_rows(d)) ? kKeyTiles16 : kKeyTiles32; }

// Does a call go through score_topk_small_kernel, one launch instead of two?  Where the launches are what it takes: the score workgroups then
// pool all of the K they see themselves, which pays up to 64 KB of K a head, and to 96 KB in 4 blocks.  Two launches against one, 32/8 heads, calls
// in a row, fused: 300 tokens with head_dim 64, blocks of 128, 18.6 and 15.9 us, 384 with head_dim 128 (3 blocks, 96 KB) 22.7 and 21.2, 512 with
// head_dim 64, blocks of 64 (8 blocks, 64 KB), 18.7 and 16.7, of one head 18.5 and 15.9; replayed from a graph, where a launch costs less, 16.3 and
// 15.1, 21.7 and 20.4, 16.0 and 16.1, 15.4 and 14.9.  Selections alone 14.6 and 11.7 in a row; from a graph 7.6 and 6.2 with 4 blocks of 64, 7.6
// and 7.4 with 8, 8.1 and 7.0 with 2 of 128, head_dim 128.  Batches, from a graph: 10 prompts of 384 tokens, head_dim 128, 50.6 and 48.8, their
// selection alone 12.4 and 14.4; 8 of 256 in blocks of 64 30.6 and 29.2, alone 8.0 and 8.6.
// 128 KB in up to 6 blocks would gain 1 to 5 % as well (fused in a row, 512 tokens with head_dim 128, blocks of 128, 23.8 and 22.7, 384 with blocks of 64
// 19.4 and 19.0, 640 with head_dim 64, blocks of 128, 20.3 and 19.8), more blocks lose 1 to 5 % (512 with head_dim 128, blocks of 64, 19.3 and 19.5, 768
// with head_dim 64 18.5 and 19.0): the line, drawn when K was pooled two blocks at a time, has not been moved.
// (At most 8 key blocks: they are one tile.)  Not with a mass budget, shared lists or the output-aware score, whose kernels it would double.
constexpr int kSmallKeys = 64 << 10, kSmallKeysFewBlocks = 96 << 10, kFewBlocks = 4;
inline bool small_call(const Dims& d, bool rank_by_values) {
    const int64_t k_bytes = (int64_t)d.Skv * d.D * 2;
    return d.gamma_q16 < 0 && !d.shared && !rank_by_values && (k_bytes <= kSmallKeys || (k_bytes <= kSmallKeysFewBlocks && d.NBk <= kFewBlocks)) &&
           score_rows(d) == 4;
}
// the most key blocks such a call has: what its workgroups hold registers for
constexpr int most_small_blocks(int D, int Bs) {
    const int block = 2 * D * Bs, few = kSmallKeysFewBlocks / block < kFewBlocks ? kSmallKeysFewBlocks / block : kFewBlocks;
    return kSmallKeys / block > few ? kSmallKeys / block : few;
}

// Lists shared by several heads: do the workgroups of the score kernel pool the queries of all of them themselves?  Each streams as many
// blocks as it has rows times the heads of a group, 50 to 60 GB/s for a workgroup, so it takes enough of them: 352, with head_dim 64, whose
// blocks are half as long, 384.  Select calls, pooled beforehand with K against in the kernel, 32/8 heads: 38000 tokens (304 workgroups) 74.0
// and 78.3 us, 40000 (320) 77.7 and 80.6, 42000 (336) 81.3 and 82.5, 44000 (344) 85.1 and 84.3, 46000 (360) 88.7 and 86.5, 50000 (392) 95.8
// and 89.4, with 4 rows 22000 (344) 43.4 and 44.5, 26000 (408) 51.3 and 48.5; head_dim 64, 40000 40.4 and 42.8, 48000 (376) 46.4 and 47.2,
// 50000 (392) 48.8 and 48.0.
inline bool group_pooled_in_kernel(const Dims& d) {
    const int R = score_rows(d);
    return (int64_t)d.B * d.Hq * ((d.NB + R - 1) / R) >= (d.D == 64 ? 384 : 352);
}

}  // namespace spa
