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
    // 513 .. 2048 blocks.  Many rows: 16, as 8 re-read the pooled K twice as often (blocks of 128, 8 against 16: 186 and 181 us at 768 blocks
    // and 24576 rows, 257 and 248 at 1024 and 32768; 731 and 700 at 262144 tokens and 81920 rows, 385 and 363 at 40960, where 16 rows are
    // scored in two chunks of 1024 columns to keep two workgroups per CU).
    if (rows > (two_chunks ? 32768 : 16384)) return 16;
    // Fewer: more workgroups, unless they only make more rounds.  With blocks of 128 the query stream, twice as long for a row, hides the
    // rounds, and 8 are the better or equal choice up to 1024 blocks (16 against 8: 8192 queries over 98304 tokens, 2048 rows, 71.8 and 63.8
    // us; 98304 tokens of 8 heads 85.3 and 79.4; 131072 of 16 heads, 16384 rows, 144 and 134).  In two chunks, with their 16-row products, 16
    // have become the better choice in places (175 and 167 at 196608 tokens of 8 heads, 238 and 231 at 262144, but 304 and 318 with 16 heads,
    // 32768 rows; 174 and 177 at 163840 of 16 heads; 177 and 187 for 25600 queries over 230400 tokens); the line has not been moved since.
    if (d.Bs == 128) return 8;
    // With blocks of 64 the rounds of 512 workgroups (two per CU) show.  Up to 1.5 rounds of 8-row workgroups (6144 rows) 8 rows win whatever
    // the count, by up to 27 %.  From there on:
    //   - over a prefix at least as long as the chunk all rows are about as long, and what counts is `depth`, how many of them a place works
    //     through one after the other: 8 rows where that is less (12797 queries over 51200 tokens, 40 heads, 89.7 with 16, 88.7 us with 8;
    //     but since 16-row products 19197 over 44800 tokens 101 and 110, 38397 over 51200 of 16 heads 91.5 and 94.9), 16 where it is the same
    //     (12797 over 51200 tokens, 32 heads, 72.5 against 78.5 us with 8; 25597 over 102400 tokens, 40 heads, 190 against 215);
    //   - rows that differ in length are dealt longest first and even the rounds out.  8 rows win up to one round of 16-row workgroups (52413
    //     tokens of 8 heads, 59.1 with 16, 57.7 us with 8) and, with head_dim 64 or two chunks, up to 14336 rows (95997 tokens of 8 heads
    //     113.9 and 112.0; 47485 tokens of 16 heads, head_dim 64, 45.1 and 43.7).  16 elsewhere: 40957 tokens of 16 heads 52.7 against 55.0
    //     us with 8, 113341 tokens of 16 heads, head_dim 64, 134 against 142, 28288 rows of 1247 blocks 177 against 199.
    const int64_t wg8 = heads * ((d.NB + 7) / 8), wg16 = heads * ((d.NB + 15) / 16);
    if (wg8 <= 768) return 8;
    if (d.off >= d.NB) {
        const int64_t depth8 = (wg8 + 511) / 512 * 8, depth16 = (wg16 + 511) / 512 * 16;
        return depth8 < depth16 && rows <= 16384 ? 8 : 16;
    }
    return wg16 <= 512 || (rows <= 14336 && (two_chunks || d.D == 64)) ? 8 : 16;
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
// pool all of the K they see themselves, which pays up to 64 KB of K a head, and to 96 KB in 4 blocks.  The line was drawn when they pooled two
// blocks at a time, one round after the other; with all of K asked for at once 128 KB in up to 6 blocks would gain 2 to 4 % (512 tokens, head_dim
// 128, blocks of 128, 23.6 and 22.7, 384 with blocks of 64 19.0 and 18.8, 640 with head_dim 64, blocks of 128, 20.4 and 19.6) and more blocks
// lose as much (768 with head_dim 64, blocks of 64, from a graph 17.2 and 18.0).  Two launches against one as it was then, calls in a row, fused:
// 300 tokens of 32/8 heads with head_dim 64 (3 blocks) 19.9 and 17.5 us, 384 with head_dim 128 (3 blocks, 96 KB) 22.2 and 21.9, 512 with head_dim 64, blocks of 64 (8 blocks, 64 KB), 19.8 and 18.9, of one head 19.9
// and 17.5; but 384 with head_dim 128, blocks of 64 (6 blocks, 96 KB), 19.7 and 20.1, 640 with head_dim 64 (10 and 5 blocks, 80 KB) 20.0 and
// 21.2, 20.3 and 20.9.  Replayed from a graph, where a launch costs less, the first four are 17.1 and 16.6, 21.8 and 21.4, 17.5 and 18.1,
// 16.8 and 17.1.  Selections alone 15.7 and 12.9 in a row; from a graph 6.9 and 6.5 with 4 blocks of 64, 7.4 and 7.7 with 8, 8.1 and 8.7 with
// 2 of 128, head_dim 128. (At most 8 key blocks then: they are one tile.)  Not with a mass budget, shared lists or the output-aware score,
// whose kernels it would double.
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
