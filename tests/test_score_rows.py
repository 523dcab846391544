"""Rows per workgroup of the score kernel (csrc/score_rows.hpp, compiled for the host)."""
import ctypes

import pytest

from host_shim import compile_shim
from paper_2602_21233_amd import binding
from test_gpu_dispatch import SCORE_KERNELS, SCORE_OPTIONS, SHORT_ROWS, score_case

SHIM = r"""
#include "score_rows.hpp"
static spa::Dims lists_of(const spa_params* p, int mass) {
    spa::Dims d = spa::dims_of(*p);
    d.gamma_q16 = mass ? 1 : -1;
    return spa::list_dims(d);
}
extern "C" int score_rows(const spa_params* p, int mass) { return spa::score_rows(lists_of(p, mass)); }
extern "C" int pooled_in_kernel(const spa_params* p, int mass) { return spa::group_pooled_in_kernel(lists_of(p, mass)); }
extern "C" int one_launch(const spa_params* p, int mass) { return spa::small_call(lists_of(p, mass), false); }
extern "C" int one_launch_by_values(const spa_params* p, int mass) { return spa::small_call(lists_of(p, mass), true); }
extern "C" int most_small_blocks(const spa_params* p, int) { return spa::most_small_blocks(p->head_dim, p->block_size); }
extern "C" int lists_by_bound(const spa_params* p, int mass) { return spa::lists_by_bound(lists_of(p, mass)); }
extern "C" int sixteen_row_tiles(const spa_params* p, int mass) { return spa::key_layout(lists_of(p, mass)) == spa::kKeyTiles16; }
"""


@pytest.fixture(scope="module")
def rows_of(tmp_path_factory):
    lib = compile_shim(tmp_path_factory.mktemp("score_rows"), SHIM)

    def ask(NB, NBk, heads, Bs=64, D=128, mass=False, what="score_rows", group=None, **kw):
        """heads: lists; group: query heads that share one (None: a list for each)"""
        p = binding.make_params(**dict(dict(batch=1, n_q_heads=heads * (group or 1), n_kv_heads=heads if group else 1, seq_len=NB * Bs - 3,
                                            head_dim=D, block_size=Bs, n_sink_blocks=1, n_local_blocks=4, top_k_blocks=64,
                                            kv_prefix_len=(NBk - NB) * Bs, lists_per_kv_head=group is not None), **kw))
        return getattr(lib, what)(ctypes.byref(p), int(mass))
    return ask


# Blocks of 64: calls that 8 rows per workgroup slow down (measured, whole select calls, 16 against 8 rows) keep 16.
@pytest.mark.parametrize("NB,NBk,heads,D", [
    (200, 1000, 32, 128),      # 67 against 77 us
    (200, 2000, 32, 128),      # 101 against 118
    (400, 640, 40, 128),       # 86 against 92
    (400, 2000, 40, 128),      # 149 against 183
    (640, 640, 16, 128),       # 50.4 against 52.4
    (1000, 1000, 32, 128),
    (1771, 1771, 16, 64),      # 121 against 136
    (884, 1247, 32, 128),      # 160 against 183
    (2000, 2000, 16, 64),      # 138 against 156
])
def test_sixteen_rows_where_eight_are_slower(rows_of, NB, NBk, heads, D):
    assert rows_of(NB, NBk, heads, D=D) == 16


# ... and those that gain from them take 8 (or 4).
@pytest.mark.parametrize("NB,NBk,heads,Bs,D,want", [
    (100, 1000, 16, 64, 128, 8), (200, 1000, 40, 64, 128, 8), (640, 640, 8, 64, 128, 8), (819, 819, 8, 64, 128, 8),
    (1500, 1500, 8, 64, 128, 8), (400, 640, 16, 128, 128, 8), (1000, 1000, 16, 128, 128, 8), (2048, 2048, 16, 128, 128, 8),
    (32, 1000, 32, 64, 128, 4), (32, 2048, 32, 128, 64, 4), (33, 2048, 32, 128, 64, 8), (128, 128, 8, 64, 64, 4), (129, 129, 8, 64, 64, 8),
    (512, 512, 40, 128, 128, 8), (1024, 1024, 32, 128, 128, 16), (2048, 2048, 40, 128, 128, 16), (2049, 2049, 40, 128, 128, 4)])
def test_fewer_rows_where_they_are_faster(rows_of, NB, NBk, heads, Bs, D, want):
    assert rows_of(NB, NBk, heads, Bs, D) == want


def test_a_mass_budget_keeps_its_groups(rows_of):
    assert [rows_of(8, n, 4, mass=True) for n in (64, 256, 512, 513, 1024, 1025, 2048, 2049, 4096)] == [8, 8, 8, 16, 16, 8, 8, 4, 4]


# Lists shared by several heads keep 4 rows up to 2048 rows; a list of one head is a list like any other (32 heads, 1400 rows over 32768 tokens
# and their own, 71.5 us with 8, 73.4 with 4).
@pytest.mark.parametrize("rows,group,want", [(1024, 1, 4), (1032, 1, 8), (2040, 1, 8), (1032, 2, 4), (2048, 2, 4), (2048, 4, 4), (2056, 4, 8)])
def test_four_rows_for_more_lists_only_where_heads_share_them(rows_of, rows, group, want):
    assert rows_of(rows // 8, rows // 8, 8, Bs=128, group=group) == want
    assert rows_of(rows // 8, rows // 8, 8, Bs=128) == (4 if rows <= 1024 else 8)


# Queries of a group are pooled by the score kernel from 352 workgroups on (384 with head_dim 64), with K below (40000 tokens of 8 KV
# heads, 320 workgroups, 77.7 us, 80.6 in the kernel; 46000, 360 workgroups, 88.7 and 86.5).
@pytest.mark.parametrize("NB,heads,D,want", [(313, 8, 128, False), (344, 8, 128, False), (345, 8, 128, True), (172, 8, 128, False), (173, 8, 128, True),
                                             (345, 8, 64, False), (376, 8, 64, False), (377, 8, 64, True), (192, 8, 64, True), (16, 1, 128, False), (1250, 2, 128, False)])
def test_group_means_in_the_score_kernel_where_its_workgroups_fill_the_chip(rows_of, NB, heads, D, want):
    assert bool(rows_of(NB, NB, heads, Bs=128, D=D, what="pooled_in_kernel", group=4)) == want


# One launch for a small call up to 64 KB of K a head, or 96 KB in 4 blocks (fused, 32 / 8 heads, 384 tokens with head_dim 128 in 3 blocks 22.7 -> 21.2
# us; up to 128 KB in 6 blocks it would pay as well, the line has not been moved).  (Lengths are three tokens short of whole blocks.)
@pytest.mark.parametrize("NB,NBk,Bs,D,want", [
    (1, 1, 64, 64, True), (8, 8, 64, 64, True), (9, 9, 64, 64, False), (12, 12, 64, 64, False), (1, 11, 64, 64, False), (4, 4, 128, 64, True), (5, 5, 128, 64, False),
    (4, 4, 64, 128, True), (5, 5, 64, 128, False), (6, 6, 64, 128, False), (3, 3, 128, 128, True), (1, 3, 128, 128, True), (4, 4, 128, 128, False)])
def test_one_launch_for_small_calls(rows_of, NB, NBk, Bs, D, want):
    ask = lambda heads=8, **kw: bool(rows_of(NB, NBk, heads, Bs=Bs, D=D, **dict(dict(what="one_launch"), **kw)))
    assert ask() == want
    assert not ask(mass=True) and not ask(group=2) and not ask(what="one_launch_by_values")
    assert not ask(heads=1024 // NB + 1)                   # more than 1024 rows: not 4 per workgroup


# ... whose kernel has registers for as many blocks as such a call may have, and no more: what they cost is workgroups that share a CU.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Bs", [64, 128])
def test_small_calls_have_registers_for_their_blocks(rows_of, D, Bs):
    taken = [n for n in range(1, 40) if rows_of(1, n, 8, Bs=Bs, D=D, what="one_launch")]
    assert rows_of(1, 1, 8, Bs=Bs, D=D, what="most_small_blocks") == max(taken) == len(taken)


# 16-row products, and the pooled K laid out for them, are for 16 rows of head_dim 128: 4 or 8 rows lose 1 to 2.5 % to them or to their
# layout, head_dim 64 up to 3 % (1771 blocks of 16 heads, 133.9 -> 137.9 us).
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("NB,NBk,heads,mass", [(7, 7, 8, False), (200, 1000, 40, False), (500, 500, 32, False), (1000, 1000, 32, False), (1000, 1000, 32, True),
                                               (1771, 1771, 16, False), (2000, 2000, 40, False), (2000, 2000, 40, True), (3000, 3000, 8, False)])
def test_sixteen_row_tiles_only_where_sixteen_rows_of_head_dim_128_read_them(rows_of, NB, NBk, heads, mass, D):
    want = D == 128 and rows_of(NB, NBk, heads, D=D, mass=mass) == 16
    assert rows_of(NB, NBk, heads, D=D, mass=mass, what="sixteen_row_tiles") == want


# The GPU test of group means takes 8 and 16 rows per workgroup, pooled in the kernel, at every number of key registers.
@pytest.mark.parametrize("NB,NBk,heads,group,Bs,D,rows", [(47, 47, 64, 2, 64, 64, 8), (89, 289, 32, 2, 64, 64, 8), (90, 590, 32, 3, 64, 128, 8), (90, 1090, 32, 2, 64, 128, 8),
                                                          (520, 520, 16, 2, 64, 128, 16), (48, 48, 32, 2, 128, 64, 4), (42, 342, 32, 3, 64, 128, 4)])
def test_the_shapes_of_the_gpu_test_of_group_means(rows_of, NB, NBk, heads, group, Bs, D, rows):
    assert rows_of(NB, NBk, heads, Bs=Bs, D=D, group=group) == rows and rows_of(NB, NBk, heads, Bs=Bs, D=D, group=group, what="pooled_in_kernel")


# Rows are selected from a list of the blocks that reach a bound where enough of them are long enough for the budget.  Measured, select calls, without and
# with lists: 700 blocks from the first on, 8 wanted, 53.1 and 55.2 us; 768 100.4 and 98.6; 826 blocks, 64 wanted, 105.5 and 107.5; rows of 384
# to 768 blocks 64.3 and 61.8, of 260 to 520 80.2 and 82.0; head_dim 128, 799 blocks, 119.7 and 116.6; all 128 wanted of 960 blocks 56.8 and 61.5.
@pytest.mark.parametrize("NB,NBk,heads,D,topk,want", [
    (700, 700, 32, 64, 8, False), (768, 768, 32, 128, 8, True), (826, 826, 40, 64, 64, False), (960, 960, 32, 64, 64, True), (384, 768, 64, 64, 64, True),
    (260, 520, 64, 64, 64, False), (799, 799, 32, 128, 64, True), (652, 652, 32, 128, 64, False), (799, 799, 16, 128, 64, False), (960, 960, 32, 64, 128, False),
    (1024, 1024, 32, 128, 64, True), (200, 1000, 40, 128, 112, False), (512, 512, 40, 128, 8, False), (200, 1000, 32, 64, 112, True),
    (200, 1000, 32, 64, 113, False), (100, 1025, 8, 64, 124, True), (100, 1025, 8, 64, 125, False), (32, 2048, 32, 64, 64, True), (2048, 2048, 40, 128, 128, True),
    (2048, 2048, 40, 64, 128, True), (1700, 1700, 8, 64, 128, False), (2048, 2048, 40, 128, 129, False), (100, 2048, 40, 128, 128, False),
    (100, 1500, 40, 128, 128, False), (2049, 2049, 40, 128, 8, False)])
def test_lists_by_bound_where_they_are_faster(rows_of, NB, NBk, heads, D, topk, want):
    ask = lambda **kw: bool(rows_of(NB, NBk, heads, D=D, what="lists_by_bound", **dict(dict(top_k_blocks=topk), **kw)))
    assert ask() == want and ask(n_dense_q_blocks=3) == want and ask(n_sink_blocks=64) == want
    assert not ask(mass=True) and not ask(group=2) and not ask(stride_blocks=16) and not ask(n_sink_blocks=65)


# The GPU tests of lists by bound take the kernels that they name.
@pytest.mark.parametrize("shape", SHORT_ROWS)
@pytest.mark.parametrize("D", [64, 128])
def test_the_shapes_of_the_gpu_tests_of_lists_by_bound(rows_of, shape, D):
    NB, heads, P = SHORT_ROWS[shape]
    assert rows_of(NB, P + NB, heads, D=D) == (8 if shape.startswith("8") else 16)
    lists = [k for k in (1, 64, 65, 112, 113, 128) if rows_of(NB, P + NB, heads, D=D, what="lists_by_bound", top_k_blocks=k)]
    assert lists == [1, 64, 65, 112] + ([113] if P + NB > 1024 else []) + ([128] if shape.endswith("long") else [])
    for kernel, (NB, heads, P) in SCORE_KERNELS.items():
        assert bool(rows_of(NB, P + NB, heads, D=D, what="lists_by_bound")) == (kernel[1] == 2048 or kernel == (16, 1024))


# The GPU test of every option on every score kernel takes the kernels that it names.
@pytest.mark.parametrize("option", SCORE_OPTIONS)
@pytest.mark.parametrize("kernel", SCORE_KERNELS)
@pytest.mark.parametrize("D", [64, 128])
def test_the_shapes_of_the_gpu_test_take_the_kernels_they_name(rows_of, kernel, option, D):
    B, Hq, Hkv, NB, P = score_case(kernel, option)
    rows, blocks = kernel
    assert blocks // 2 < P + NB <= blocks
    shared = SCORE_OPTIONS[option].get("group_shared")
    assert rows_of(NB, P + NB, B * (Hkv if shared else Hq), D=D, group=Hq // Hkv if shared else None) == rows
