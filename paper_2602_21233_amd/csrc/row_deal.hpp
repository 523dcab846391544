// Which workgroup of an attention launch serves which row (batch entry, KV head, query block): the deal itself, for the host that sizes the
// grid and for the workgroups that look themselves up in it.
#pragma once
#include "common.hpp"

namespace spa {

// Which XCD serves which rows.  Workgroup ids go round robin over the 8 XCDs and are dispatched in id order, so the XCDs advance through
// their sequences in step: what has to be equal is the work of the rows that sit at the same position of the 8 sequences.
//
// Gangs.  A KV head is served by a gang of `gang` XCDs (8, 4, 2 or 1), 8 / gang heads side by side.  With long sequences it is all eight;
// with few query blocks an eighth of a head's rows does not fill an XCD, which would have rows of several heads in flight and fetch each of
// their K and V^T tiles for a few rows only; a smaller gang puts more rows of one head behind one L2.  Attention kernel alone: 1999 tokens
// 58 -> 50 us, 2048 queries over the prefix 306 -> 286 us, 1024 queries 174 -> 169 us.
// In a ragged batch only heads of one entry sit side by side: entries differ in length, which the host does not see, and an XCD that serves
// one entry's head alone idles after a short one.  Attention kernel, 8 entries of 4 / 1 heads with blocks of 128, one of 3900 tokens and the
// others of 325: 106 us with an entry for each XCD, 57 this way; lengths down from 3900 in steps 109 -> 79; all of 3900 tokens 131 -> 150,
// the price of not knowing.
//
// Width.  At any time `width` of the gang's XCDs are at the same head, so that 8 / width heads are in flight, each behind few L2s: fewer of
// its tiles are fetched more than once.  The XCDs go from head to head after every piece of row positions (at least what an XCD has in
// flight; pieces half as long cost 2 to 3 % with blocks of 64, twice as long give nothing more), so that in the end all of the gang have
// served all of the heads alike.  Where width is the whole gang they stay: a change only has more L2s fetch a head (5312 queries over 30464
// tokens, blocks of 64, 398 -> 391 us; 2763 tokens, blocks of 64, 43.3 -> 43.0).
// As few XCDs are at a head as half of the memory-side cache (128 of 256 MB, for queries and outputs pass through it too) holds K and V^T of
// the heads in flight, up to 32 MB a head (65536 tokens of head_dim 128).  Attention kernel, 32/8 heads, eight XCDs at a head against one:
// 8192 tokens 501 -> 480 us, 12000 with lists of 35 blocks 695 -> 615, 24000 1429 -> 1361, with blocks of 64 1006 -> 918, 24000 with lists of
// 19 blocks 873 -> 815.  With 8, 4, 2, 1 at a head: 49152 tokens (25 MB a head) of 40/8 heads 6.96, 6.83, 6.77, 6.71 ms, 65536 9.46, 9.39,
// 9.29, 9.27, of 32/8 heads 7.32, 7.34, 7.32, 7.33.  Beyond that it depends on the lists, and mostly costs: 81920 tokens 9.65, 9.49, 9.42,
// 9.55, but with keys that drift along the sequence 98304 tokens 12.16, 12.28, 12.31, 12.57, 131072 16.67, 16.83, 16.95, 17.35, 196608 25.66,
// 25.93, 26.31, 27.18, 262144 of 40/8 heads 67.1, 67.2, 68.2, 70.5; 8192 queries over 131072 tokens 1111, 1125, 1121, 1137 us (two runs of one
// side differ by 0.5 %).
//   - Calls with a Tri-shape strip have no limit of 32 MB: with all XCDs at one head they all wait for its dense rows, head after head (8
//     dense rows and lists of 21 blocks, eight and four at a head: 73728 tokens 4.61 and 4.26 ms, 131072 8.73 and 8.08, lists of 69 18.7 and
//     18.2; 2 dense rows, 131072 12.0 and 10.6).
//   - Gangs of two whose rows visit less than a quarter of the blocks stay, with blocks of 128: what a row reads is then little beside what
//     the second L2 fetches for a head (two and one at a head: 7680 tokens, lists of 11 blocks, 154 and 156 us, shared by a group 166 and 170;
//     6272 queries over 24064 tokens, shared lists of 10, 119 and 123; but lists of 19 blocks 236 and 235, 5000 tokens, shared lists of 19,
//     156 and 146; blocks of 64, 5000 tokens, lists of 7 and 11, 55.0 and 54.6, 73.9 and 73.4).
//   - All heads have to have lists of one length: the XCDs advance in step, so those at heads with short lists wait for those at long ones,
//     and changing heads evens that out only in part.  A fused call with budgets per head or a mass budget keeps width = gang: one KV head of
//     8 with eight times the budget of the others, 16384 tokens, 789 us, 949 with one XCD at a head (8192 tokens 335 and 389, 32768 1809 and
//     1996, blocks of 64 579 and 645); every second KV head 1290 and 1293, every fourth query head 1361 and 1335; budgets drawn at random 0.95
//     to 1.11 times the time; a mass budget of 0.9, 32768 tokens, 3442 and 3476.  An attention call does not say how its lists came about and
//     is taken at its pattern's word: the same budget for all.
//
// Runs.  Among the XCDs at a head:
//   - the n_dense rows of a Tri-shape strip (each visits up to NB blocks) are dealt one by one;
//   - the other rows are dealt in runs of `run` consecutive rows, last row first; with `snake` every other round of runs goes backwards, so
//     that the XCD that gets the longest row of one round gets the shortest of the next.  Which rounds alternates with the KV head; where the
//     XCDs change heads, with those one after the other: with the head at hand, an XCD that goes on to the next one with every round had the
//     same place in all of them (16 / 2 heads of 12288 tokens: 18 % more than its share for one XCD, 503 -> 590 us).
// Neighbouring rows share their local-window blocks in the XCD's L2, which favours runs of 8 once K and V^T of a head outgrow that L2 (4 MB).
// But the XCD with the most rows decides: 16 query blocks in runs of 8 kept two XCDs busy and six idle.  So the runs get shorter until no
// more than a sixteenth of the dealt places are empty, and rows whose length varies with the position (strided columns, dense strip) are
// dealt one by one, as are those of heads that fit the L2 whatever the deal.  The snake is for rows dealt one by one, and for calls with at
// most 8 T key blocks: without a prefix the ramp of the first T rows, which are shorter than T, is then an eighth of the rows or more.
// Elsewhere it only moves neighbouring rows apart.  Over a prefix of T blocks or more no row is shorter and the snake does nothing for the
// balance, nor against it: 1024 to 8192 queries over 8192 to 65536 tokens, blocks of 64 and 128, take the same time with it, without it, and
// by the ramp that is left (within 0.5 %).
// Measured against runs of 8, all forwards, whole calls with 32/8 heads: 1999 tokens 190 -> 74 us; 2048 queries over a prefix of 98304 tokens
// 1048 -> 368 us; 6 ragged prompts of up to 6000 tokens, blocks of 64, 727 -> 591 us; 32768 tokens 2.10 -> 2.03 ms; group-shared lists, 16384
// tokens, D = 64, 628 -> 582 us.  The snake at 131072 tokens (a ramp of 69 of 1024 rows): 17.05 -> 17.18 ms, which is why it is left out there.
//
// Fold.  Launches of 33 to 64 workgroups per XCD, two to a CU, all in flight at once: the first 32 go to CUs of their own, longest row first,
// and the others join them in that order, so the CU that has the longest row would get the longest of the rest.  `fold` (that count) deals the
// others shortest first, where the longest rows are the last ones for sure:
//   - there is room for all blocks (T >= NBk; with a Tri-shape strip there is, whatever the other rows do): rows cut to one length are about as
//     long as each other;
//   - no budget per row may cut the last ones short.  Of a fused call's budgets only the largest is known here; a quarter of it has to do, the
//     least of the decaying budgets that the package makes.  An attention call is taken at its pattern's word here, too;
//   - the batch is not ragged: the first 32 are then often rows past an entry's end, and it depends on which entry is the long one.
// Attention kernel, 32/8 heads: 1999 tokens 44.5 -> 42.2 us, two of 1000 32.6 -> 27.8, four of 500 22.0 -> 20.1, 2000 with two dense rows and
// 4 blocks of budget 43.8 -> 41.1, 2000 with a budget that falls from 64 to 16 44.5 -> 42.0, but from 12 to 3 35.5 -> 36.6, from 8 to 2 34.0
// -> 35.9, 8000 tokens of 8/8 heads from 64 to 16 101.8 -> 109.6; entries of 166 and 1000 tokens 21.1 -> 24.1, of 1000 and 667 25.5 -> 24.1,
// with blocks of 64 and 16/4 heads 19.7 -> 20.5.  With more than two to a CU (blocks of 64, 2000 tokens) it gives nothing, with more than one
// round (4096 tokens) it costs 3 %.
//
// seq_len = workgroups per (head, XCD) in the grid; surplus workgroups exit at once.  places = workgroups of an XCD for the heads that are
// side by side; what divides workgroup ids is kept as a shift where it can be, every workgroup starts with these.
constexpr int kNoChange = 30;   // piece_log2 of XCDs that stay at their heads

struct RowDeal {
    int gang, n_dense, run, snake, seq_len;
    int places, width_log2, run_log2, piece_log2, n_single, fold;
};

// nh: query heads served by one workgroup (their workgroups per row position number G / nh)
inline RowDeal deal_rows(const Dims& d, int nh) {
    RowDeal r;
    r.n_dense = d.n_dense < d.NB ? d.n_dense : d.NB;
    const int n = d.NB - r.n_dense;                       // rows dealt in runs
    const int GH = d.G / nh;
    // Workgroups an XCD has in flight, by the LDS that head_dim 128 needs.  With head_dim 64 a CU holds half as many again; gangs are then
    // larger than they have to be, which is the better choice at some sizes and not at others (32 / 8 heads: 4096 tokens 91 us, 83 with the
    // gang of the true count; 8192 tokens 298 and 302; 16 / 2 heads: 8192 tokens 164 and 145, with blocks of 64 131 and 137).
    const int slots = 32 * (d.Bs == 64 ? 4 : 2) / nh;
    const int heads = d.seq_lens != nullptr ? d.Hkv : d.B * d.Hkv;    // heads with the same rows: may sit side by side
    r.gang = 8;
    while (r.gang > 1 && (int64_t)d.NB * GH < (int64_t)slots * r.gang && heads % (16 / r.gang) == 0) r.gang >>= 1;
    const int64_t kv_bytes = (int64_t)d.Skv * d.D * 4;                // K and V^T of a head, bf16
    int width = r.gang;
    const bool alike = !d.head_budgets && d.gamma_q16 < 0;            // lists of all heads as long as each other
    const bool few = r.gang == 2 && d.Bs == 128 && 4 * (int64_t)d.T < d.NBk;
    const bool spread = kv_bytes <= 32 << 20 || d.n_dense > 0;
    while (alike && !few && spread && width > 1 && heads % (16 / width) == 0 && (16 / width) * kv_bytes <= 128 << 20) width >>= 1;
    r.width_log2 = __builtin_ctz(width);
    r.piece_log2 = 0;
    while ((GH << r.piece_log2) < slots) ++r.piece_log2;
    if (width == r.gang) r.piece_log2 = kNoChange;
    r.run = (d.stride > 0 || d.n_dense > 0 || kv_bytes <= 4 << 20) ? 1 : 8;
    while (r.run > 1 && (n + width * r.run - 1) / (width * r.run) * (width * r.run) > n + n / 16) r.run >>= 1;
    r.snake = r.run == 1 || 8 * (int64_t)d.T >= d.NBk;
    r.run_log2 = __builtin_ctz(r.run);
    r.n_single = (r.n_dense + width - 1) / width;
    const int runs = (n + r.run - 1) / r.run;
    const int turns = r.gang / width;                     // heads that the gang has side by side
    r.seq_len = ((r.n_single + (runs + width - 1) / width * r.run) * GH + turns - 1) / turns;
    r.places = r.seq_len * turns;
    const int64_t per_xcd = (int64_t)r.gang * r.seq_len * d.B * d.Hkv / 8;
    const bool rows_in_full = d.T >= d.NBk && (!d.row_budgets || (int64_t)d.ns + d.nl + d.k / 4 >= d.NBk);
    r.fold = slots >= 64 && rows_in_full && d.seq_lens == nullptr && per_xcd > 32 && per_xcd <= 64 ? (int)per_xcd : 0;
    return r;
}

struct DealtRow {
    int head_slot, i;   // b * Hkv + kv head; query block
    int turn;           // which of the row's GH workgroups
};

// Row of workgroup `block`, GH workgroups per row; false: a surplus workgroup.
__host__ __device__ __forceinline__ bool dealt_row(const RowDeal& deal, int GH, int NB, int block, DealtRow& r) {
    const int wl = deal.width_log2, width = 1 << wl;
    const int xcd = block & (width - 1);                  // which of the XCDs that are at this head now
    int slot = block >> 3;
    if (slot >= 32 && deal.fold != 0) slot = deal.fold + 31 - slot;
    const int group = slot / deal.places, within = slot - group * deal.places;
    const int pos = within / GH;                          // position in this XCD's row sequence
    r.turn = within - pos * GH;
    const int side = 8 >> wl;                             // heads side by side
    r.head_slot = group * side + ((((block & 7) >> wl) + (pos >> deal.piece_log2)) & (side - 1));
    if (pos < deal.n_single) {
        const int hidx = pos * width + xcd;
        r.i = NB - 1 - hidx;
        return hidx < deal.n_dense;
    }
    const int rr = pos - deal.n_single;
    const int round = rr >> deal.run_log2;
    const int turned = deal.piece_log2 == kNoChange ? r.head_slot : group;
    const int x = (deal.snake & (round ^ turned)) ? width - 1 - xcd : xcd;
    const int ridx = ((round * width + x) << deal.run_log2) + (rr & (deal.run - 1));
    r.i = NB - deal.n_dense - 1 - ridx;
    return ridx < NB - deal.n_dense;
}

}  // namespace spa
