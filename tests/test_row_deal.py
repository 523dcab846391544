"""The deal of an attention launch (csrc/row_deal.hpp, compiled for the host): which XCD serves which rows."""
import ctypes

import numpy as np
import pytest

from host_shim import compile_shim
from paper_2602_21233_amd import binding

SHIM = r"""
#include "row_deal.hpp"
// what only a fused call knows of its lists
static int head_budgets, mass, row_budgets;
extern "C" void lists_by(int by_head, int by_mass, int by_row) { head_budgets = by_head; mass = by_mass; row_budgets = by_row; }
static spa::Dims dims(const spa_params* p) {
    spa::Dims d = spa::dims_of(*p);
    if (head_budgets) d.head_budgets = 1;
    if (mass) d.gamma_q16 = 58982;
    if (row_budgets) d.row_budgets = 1;
    return d;
}
// every workgroup of the launch: (head_slot, query block, turn), or -1 three times for a surplus one
extern "C" int deal(const spa_params* p, int nh, int* gang, int* out, int cap) {
    const spa::Dims d = dims(p);
    const spa::RowDeal r = spa::deal_rows(d, nh);
    const int nwg = r.gang * r.seq_len * d.B * d.Hkv;
    *gang = r.gang;
    for (int x = 0; x < nwg && x < cap; ++x) {
        spa::DealtRow at;
        const bool some = spa::dealt_row(r, d.G / nh, d.NB, x, at);
        out[3 * x] = some ? at.head_slot : -1;
        out[3 * x + 1] = some ? at.i : -1;
        out[3 * x + 2] = some ? at.turn : -1;
    }
    return nwg;
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    lib = compile_shim(tmp_path_factory.mktemp("deal"), SHIM)

    def rows(nh=1, ragged=False, head_budgets=False, mass=False, row_budgets=False, **kw):
        """gang, [workgroups, 3]"""
        base = dict(batch=1, n_q_heads=8, n_kv_heads=2, seq_len=2048, head_dim=128, block_size=128, n_sink_blocks=1,
                    n_local_blocks=4, top_k_blocks=64)
        base.update(kw)
        p = binding.make_params(**base)
        p.seq_lens = 1 if ragged else None              # only asked whether there is one
        lib.lists_by(head_budgets, mass, row_budgets)
        gang = ctypes.c_int()
        n = lib.deal(ctypes.byref(p), nh, ctypes.byref(gang), None, 0)
        out = np.empty((n, 3), dtype=np.int32)
        assert lib.deal(ctypes.byref(p), nh, ctypes.byref(gang), ctypes.c_void_p(out.ctypes.data), n) == n
        return gang.value, out
    return rows


# Entries of a ragged batch differ in length, so heads of different entries must not sit side by side on the XCDs: the XCDs
# of the short ones would idle while one of them serves the longest entry alone.
@pytest.mark.parametrize("block_size", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (8, 1), (8, 2), (16, 2), (28, 4), (32, 8), (12, 3)])
@pytest.mark.parametrize("S", [100, 900, 1900, 3900, 9000])
def test_the_xcds_serve_one_entry_of_a_ragged_batch_at_a_time(deal, block_size, Hq, Hkv, S):
    _, wg = deal(ragged=True, batch=8, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, block_size=block_size)
    entry = np.where(wg[:, 0] >= 0, wg[:, 0] // Hkv, -1).reshape(-1, 8)      # workgroups 8 s .. 8 s + 7: one for each XCD
    for at_once in entry:
        assert len(set(at_once[at_once >= 0])) <= 1


# One long entry among short ones: the XCD with the most key blocks to visit has at most one row (of all query
# heads of its group) more than its share, where one XCD serving an entry alone has up to eight times it.
@pytest.mark.parametrize("block_size", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (8, 1), (8, 2), (16, 2)])
@pytest.mark.parametrize("S", [1900, 3900])
def test_a_long_entry_of_a_ragged_batch_is_spread_over_the_xcds(deal, block_size, Hq, Hkv, S):
    lens = [S] + [S // 12] * 7
    _, wg = deal(ragged=True, batch=8, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, block_size=block_size)
    work = np.zeros(8)
    for x, (head_slot, i, _) in enumerate(wg):
        if head_slot >= 0 and i * block_size < lens[head_slot // Hkv]:
            work[x % 8] += i + 1                                     # every causal block: T is larger here
    longest_row = -(-S // block_size) * (Hq // Hkv)
    assert work.max() <= work.mean() + longest_row


# Whatever the gang, the runs and the snake: every workgroup of every row of every head is dealt once.
@pytest.mark.parametrize("D,Bs,nh", [(128, 64, 1), (64, 64, 2), (128, 128, 1), (128, 128, 2), (64, 128, 1)])
@pytest.mark.parametrize("B,Hkv,ragged", [(1, 3, False), (1, 8, False), (2, 2, False), (2, 2, True), (8, 1, False), (8, 1, True), (3, 4, True)])
def test_every_row_is_dealt_once(deal, D, Bs, nh, B, Hkv, ragged):
    seen = set()
    for NB, P, kw in ((1, 0, {}), (2, 0, {}), (9, 0, {}), (16, 72, {}), (17, 72, {}), (46, 72, {}), (92, 144, {}), (64, 288, {}), (23, 0, dict(n_dense_q_blocks=3)),
                      (23, 288, dict(n_dense_q_blocks=11)), (11, 0, dict(n_dense_q_blocks=40)), (130, 0, dict(stride_blocks=7)), (520, 0, {}),
                      (1024, 0, {}), (1100, 500, dict(top_k_blocks=700))):
        for G in (2, 8):
            gang, wg = deal(nh=nh, ragged=ragged, batch=B, n_q_heads=G * Hkv, n_kv_heads=Hkv, seq_len=NB * Bs - 5, head_dim=D, block_size=Bs,
                            kv_prefix_len=P * Bs, **kw)
            seen.add(gang)
            served = wg[wg[:, 0] >= 0]
            assert (wg[wg[:, 0] < 0] == -1).all()
            code = (served[:, 0].astype(np.int64) * NB + served[:, 1]) * (G // nh) + served[:, 2]
            assert served[:, 0].max() < B * Hkv and 0 <= served[:, 1].min() and served[:, 1].max() < NB and served[:, 2].max() < G // nh
            assert np.array_equal(np.sort(code), np.arange(B * Hkv * NB * (G // nh))), (NB, P, kw, G)
    divides = Hkv if ragged else B * Hkv                   # a head for each XCD of 8, 4 or 2, where so many heads divide
    assert seen == {8} | {8 // x for x in (2, 4, 8) if divides % x == 0}


# Long calls: as many heads in flight as half of the memory-side cache holds K and V^T of, one beyond 32 MB a head, and
# each XCD serves the rows of all heads alike, to within a few pieces (what an XCD has in flight).
@pytest.mark.parametrize("D,Bs", [(128, 128), (128, 64), (64, 128)])
@pytest.mark.parametrize("B,Hkv", [(1, 8), (2, 4), (1, 4), (1, 2), (1, 3)])
@pytest.mark.parametrize("S", [16384, 50001, 131072, 262143])
def test_heads_side_by_side_fit_the_cache_and_every_xcd_serves_them_alike(deal, D, Bs, B, Hkv, S):
    G, NB = 4, -(-S // Bs)
    if NB > 4096:
        pytest.skip("more than 4096 key blocks")
    gang, wg = deal(batch=B, n_q_heads=G * Hkv, n_kv_heads=Hkv, seq_len=S, head_dim=D, block_size=Bs)
    if gang < 8:
        pytest.skip("a short call")
    in_flight = 8 * 32 * (4 if Bs == 64 else 2)
    first = wg[:in_flight, 0]
    side = len(set(first[first >= 0]))
    assert side == 1 or side * S * D * 4 <= 128 << 20
    if S * D * 4 > 32 << 20:
        assert side == 1                                   # 98304 tokens 12.16 ms, with two heads side by side 12.28
    elif (B * Hkv) % (2 * side) == 0 and side < 8:
        assert 2 * side * S * D * 4 > 128 << 20
    if (B * Hkv) % 2 == 0 and 32 << 20 < S * D * 4 <= 64 << 20:    # a Tri-shape strip: two heads, 131072 tokens 8.73 -> 8.08 ms
        _, wg = deal(batch=B, n_q_heads=G * Hkv, n_kv_heads=Hkv, seq_len=S, head_dim=D, block_size=Bs, n_dense_q_blocks=8)
        assert len(set(wg[:in_flight, 0])) - (wg[:in_flight, 0].min() < 0) == 2
    rows = np.zeros((8, B * Hkv), dtype=np.int64)
    for x in range(8):
        served = wg[x::8, 0]
        rows[x] = np.bincount(served[served >= 0], minlength=B * Hkv)
    piece = in_flight // 8
    assert abs(rows - NB * G / 8).max() <= 2 * piece


# All rows in flight at once, two workgroups to a CU (workgroups k and k + 32 of an XCD): the longest
# row shares its CU with the shortest, and no CU has more than these two (a block more where GH does not divide 32).
@pytest.mark.parametrize("B,Hq,Hkv,S,Bs", [(1, 32, 8, 1999, 128), (1, 32, 8, 1500, 128), (2, 32, 8, 1024, 128), (1, 40, 8, 1024, 128),
                                           (1, 8, 8, 8000, 128), (1, 32, 8, 1024, 64), (1, 16, 2, 4000, 128)])
def test_the_cu_with_the_longest_row_gets_the_shortest_beside_it(deal, B, Hq, Hkv, S, Bs):
    _, wg = deal(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, block_size=Bs)
    blocks = np.where(wg[:, 0] >= 0, wg[:, 1] + 1, 0).reshape(-1, 8)         # causal blocks; [workgroup of the XCD, XCD]
    assert 32 < len(blocks) <= 64
    load = blocks[:32].copy()
    load[: len(blocks) - 32] += blocks[32:]
    assert load.max() <= blocks.max() + blocks[32:][blocks[32:] > 0].min() + (32 % (Hq // Hkv) != 0)


# Rows as long as their causal blocks allow, up to T, all heads alike: no XCD gets more than a few per cent more key blocks to visit than the
# others, whatever takes turns: the heads that an XCD serves and the direction of its rounds (which had cancelled each
# other: 16 / 2 heads of 12288 tokens, 18 % more for one XCD, 502 -> 589 us).  One round of rows is what a head's last, partial round can add.
@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (40, 8), (16, 4), (32, 4), (28, 4), (16, 2), (8, 2), (32, 2)])
@pytest.mark.parametrize("Bs", [64, 128])
@pytest.mark.parametrize("S", [2688, 4096, 8192, 12288, 16384, 20000, 24576, 32768, 50001, 65536])
def test_every_xcd_gets_as_many_key_blocks_as_the_others(deal, Hq, Hkv, Bs, S):
    T = 69
    _, wg = deal(n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, block_size=Bs)
    work = np.array([np.minimum(wg[x::8, 1] + 1, T)[wg[x::8, 0] >= 0].sum() for x in range(8)])
    assert work.max() <= 1.02 * work.mean() + 8 * (Hq // Hkv)


# Where no more heads are in flight than the gangs have, every XCD stays at its head: with all heads alike a change of heads only
# makes more L2s fetch a head's K and V^T (5312 queries over 30464 tokens, blocks of 64, 389 -> 398 us).
@pytest.mark.parametrize("Hq,Hkv,S,Bs,P", [(32, 8, 2688, 128, 0), (32, 8, 2763, 64, 0), (40, 8, 3100, 128, 0), (8, 8, 8000, 128, 0), (32, 8, 5312, 64, 30464)])
def test_an_xcd_of_a_short_call_serves_a_head_to_its_end(deal, Hq, Hkv, S, Bs, P):
    gang, wg = deal(n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, block_size=Bs, kv_prefix_len=P)
    assert gang < 8
    for x in range(8):
        heads = wg[x::8, 0]
        heads = heads[heads >= 0]
        assert (heads[1:] != heads[:-1]).sum() == len(set(heads)) - 1 == Hkv * gang // 8 - 1


# Heads whose lists differ in length (budgets per head, a mass budget) sit side by side only as the gangs do: with all XCDs at one head
# where the rows fill them (16384 tokens, one KV head of 8 with a large budget, 949 -> 789 us).
@pytest.mark.parametrize("why", ["head_budgets", "mass"])
@pytest.mark.parametrize("D,Bs", [(128, 128), (128, 64), (64, 128)])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 32, 8), (2, 16, 4), (1, 16, 4), (1, 40, 8), (1, 12, 2)])
@pytest.mark.parametrize("S", [1999, 6000, 16384, 50001])
def test_heads_of_their_own_budgets_are_not_put_side_by_side(deal, why, D, Bs, B, Hq, Hkv, S):
    gang, wg = deal(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=S, head_dim=D, block_size=Bs, **{why: True})
    head = wg[:, 0].reshape(-1, 8)                         # workgroups 8 s .. 8 s + 7: one for each XCD
    for at_once in head:
        assert len(set(at_once[at_once >= 0])) <= 8 // gang


# ... but only where the longest rows are the last ones for sure: not with a budget per row that may cut them (2000 tokens, 12 falling to 3
# blocks, 35.5 -> 36.6 us), not in a ragged batch (entries of 166 and 1000 tokens, 21.1 -> 24.1).  With a Tri-shape strip they are
# (2000 tokens, 43.8 -> 41.1 us).
@pytest.mark.parametrize("want,kw", [
    (True, dict(seq_len=2000)), (True, dict(seq_len=2000, row_budgets=True)), (True, dict(seq_len=2000, top_k_blocks=4, n_dense_q_blocks=2)),
    (True, dict(seq_len=2000, head_budgets=True)), (True, dict(seq_len=1000, batch=2)), (True, dict(seq_len=8000, n_q_heads=8)),
    (False, dict(seq_len=2000, top_k_blocks=12, row_budgets=True)), (False, dict(seq_len=8000, n_q_heads=8, row_budgets=True)),
    (False, dict(seq_len=2000, top_k_blocks=4, n_dense_q_blocks=2, row_budgets=True)), (False, dict(seq_len=2000, top_k_blocks=4)),
    (False, dict(seq_len=1000, batch=2, ragged=True)), (False, dict(seq_len=1000, batch=2, ragged=True, n_q_heads=16, n_kv_heads=4, block_size=64)),
    (False, dict(seq_len=2000, block_size=64)), (False, dict(seq_len=4096))])
def test_shortest_rows_join_the_longest_only_where_those_are_the_last(deal, want, kw):
    _, wg = deal(**dict(dict(n_q_heads=32, n_kv_heads=8), **kw))
    i = wg[::8, 1]                                         # query blocks of an XCD's workgroups, in their order
    second = i[32:][i[32:] >= 0]
    assert (second[0] < second[-1]) == want


# A gang of two whose rows visit less than a quarter of the blocks keeps the XCDs at its own heads, with blocks of 128 (7680 tokens, lists
# of 11 blocks, 156 -> 154 us).
@pytest.mark.parametrize("kw,side", [
    (dict(seq_len=7680, top_k_blocks=8), 4), (dict(seq_len=7680, top_k_blocks=16), 8), (dict(seq_len=7680, top_k_blocks=9), 4), (dict(seq_len=7680, top_k_blocks=10), 8),
    (dict(seq_len=5000, top_k_blocks=8, block_size=64), 8), (dict(seq_len=5000, top_k_blocks=4), 4), (dict(seq_len=12000, top_k_blocks=8), 8)])
def test_gangs_of_two_with_short_lists_stay_at_their_heads(deal, kw, side):
    gang, wg = deal(n_q_heads=32, n_kv_heads=8, **kw)
    assert gang == (4 if kw["seq_len"] == 12000 else 2)
    head = wg[:, 0].reshape(-1, 8)
    assert max(len(set(at_once[at_once >= 0])) for at_once in head) == side
