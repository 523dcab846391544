// Which workgroup of an attention launch serves which row (batch entry, KV head, query block): the deal itself, for the
// host that sizes the grid and for the workgroups that look themselves up in it.
#pragma once
#include "common.hpp"

namespace spa {

// Which XCD serves which rows.  Workgroup ids go round robin over the 8 XCDs and are dispatched in id order,
// so the XCDs advance through their sequences in step: what has to be equal is the work of the rows that
// sit at the same position of the 8 sequences.
// A KV head is served by a gang of `gang` XCDs (8, 4, 2 or 1), 8 / gang heads side by side.  With long sequences it is all
// eight: the whole chip then works through one head after the other, and what an XCD has in flight
// are rows of one head anyway.  With few query blocks an eighth of a head's rows does not fill an XCD, which would have
// rows of several heads in flight and fetch each of their K and V^T tiles for a few rows only; a smaller gang
// puts more rows of one head behind one L2.  In a ragged batch only heads of one entry sit side by side: entries differ in
// length, which the host does not see, and an XCD that serves one entry's head alone idles after a short one.  Attention
// kernel, 8 entries of 4 / 1 heads with blocks of 128, one of 3900 tokens and the others of 325: 106 us with an entry
// for each XCD, 57 this way; lengths down from 3900 in steps 109 -> 79; all of 3900 tokens 131 -> 150, the price of not knowing.
// Within the gang:
//   - the n_dense rows of a Tri-shape strip (each visits up to NB blocks) are dealt one by one;
//   - the other rows are dealt in runs of `run` consecutive rows, last row first; with `snake` every
//     other round of runs goes backwards (which rounds: alternating with the KV head), so that the XCD
//     that gets the longest row of one round gets the shortest of the next.
// Neighbouring rows share their local-window blocks in the XCD's L2, which favours runs of 8 once K and
// V^T of a head outgrow that L2 (4 MB).  But the XCD with the most rows decides: 16 query blocks in runs of
// 8 kept two XCDs busy and six idle.  So the runs get shorter until no more than a sixteenth of
// the dealt places are empty, and rows whose length varies with the position (strided columns, dense
// strip) are dealt one by one, as are those of heads that fit the L2 whatever the deal.  The snake is
// for rows dealt one by one, and for calls with at most 8 T key blocks: without a prefix the ramp of the first T rows, which
// are shorter than T, is then an eighth of the rows or more.  Elsewhere it only moves neighbouring rows apart.  Over a prefix
// of T blocks or more no row is shorter and the snake does nothing for the balance, nor against it: 1024 to 8192 queries over 8192 to
// 65536 tokens, blocks of 64 and 128, take the same time with it, without it, and by the ramp that is left (within 0.5 %).
// Measured against runs of 8, all forwards, whole calls with 32/8 heads: 1999 tokens 190 -> 74 us; 2048 queries over a
// prefix of 98304 tokens 1048 -> 368 us; 6 ragged prompts of up to 6000 tokens, blocks of 64, 727 -> 591 us;
// 32768 tokens 2.10 -> 2.03 ms; group-shared lists, 16384 tokens, D = 64, 628 -> 582 us.  The snake at 131072
// tokens (a ramp of 69 of 1024 rows): 17.05 -> 17.18 ms, which is why it is left out there.  Gangs, attention kernel
// alone: 1999 tokens 58 -> 50 us, 2048 queries over the prefix 306 -> 286 us, 1024 queries 174 -> 169 us.
// seq_len = workgroups per (head, XCD) in the grid; surplus workgroups exit at once.
struct RowDeal {
    int gang, n_dense, run, snake, seq_len;
};

// nh: query heads served by one workgroup (their workgroups per row position number G / nh)
inline RowDeal deal_rows(const Dims& d, int nh) {
    RowDeal r;
    r.n_dense = d.n_dense < d.NB ? d.n_dense : d.NB;
    const int n = d.NB - r.n_dense;                       // rows dealt in runs
    // Workgroups an XCD has in flight, by the LDS that head_dim 128 needs.  With head_dim 64 a CU holds half as many again; gangs
    // are then larger than they have to be, which is the better choice at some sizes and not at others (32 / 8 heads: 4096
    // tokens 91 us, 83 with the gang of the true count; 8192 tokens 298 and 302; 16 / 2 heads: 8192 tokens 164 and 145, with
    // blocks of 64 131 and 137).
    const int slots = 32 * (d.Bs == 64 ? 4 : 2) / nh;
    const int heads = d.seq_lens != nullptr ? d.Hkv : d.B * d.Hkv;    // heads with the same rows: may sit side by side
    r.gang = 8;
    while (r.gang > 1 && (int64_t)d.NB * (d.G / nh) < (int64_t)slots * r.gang && heads % (16 / r.gang) == 0) r.gang >>= 1;
    const bool fits_l2 = (int64_t)d.Skv * d.D * 4 <= 4 << 20;         // K and V^T of a head, bf16
    r.run = (d.stride > 0 || d.n_dense > 0 || fits_l2) ? 1 : 8;
    while (r.run > 1 && (n + r.gang * r.run - 1) / (r.gang * r.run) * (r.gang * r.run) > n + n / 16) r.run >>= 1;
    r.snake = r.run == 1 || 8 * (int64_t)d.T >= d.NBk;
    const int runs = (n + r.run - 1) / r.run;
    r.seq_len = ((r.n_dense + r.gang - 1) / r.gang + (runs + r.gang - 1) / r.gang * r.run) * (d.G / nh);
    return r;
}

struct DealtRow {
    int head_slot, i;   // b * Hkv + kv head; query block
    int turn;           // which of the row's GH workgroups
};

// Row of workgroup `block`, GH workgroups per row; false: a surplus workgroup.
__host__ __device__ __forceinline__ bool dealt_row(const RowDeal& deal, int GH, int NB, int block, DealtRow& r) {
    const int gang = deal.gang;
    const int xcd = block & (gang - 1);                   // member of the gang
    const int slot = block >> 3;
    r.head_slot = slot / deal.seq_len * (8 / gang) + (block & 7) / gang;
    const int within = slot % deal.seq_len;
    const int pos = within / GH;                          // position in this XCD's row sequence
    const int n_single = (deal.n_dense + gang - 1) / gang;
    r.turn = within % GH;
    if (pos < n_single) {
        const int hidx = pos * gang + xcd;
        r.i = NB - 1 - hidx;
        return hidx < deal.n_dense;
    }
    const int rr = pos - n_single;
    const int round = rr / deal.run;
    const int x = (deal.snake & (round ^ r.head_slot)) ? gang - 1 - xcd : xcd;
    const int ridx = (round * gang + x) * deal.run + rr % deal.run;
    r.i = NB - deal.n_dense - 1 - ridx;
    return ridx < NB - deal.n_dense;
}

}  // namespace spa
