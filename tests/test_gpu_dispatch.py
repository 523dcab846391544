"""Calls at the sizes where a dispatch rule of the library changes its mind: the launch shapes differ, the
results must not."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spa():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_21233_amd as m
    m.load_library()
    return m


def _normal(shape, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(shape, generator=g).to(torch.bfloat16).cuda()


# A fused call may be captured after nothing but selections and attention calls: what a small call's kernel needs for V^T has been asked for by the
# first selection, also if that had the other block size, which is another kernel.  (First of the tests that launch these kernels, one for each head
# size and kind of pattern, so that none of them has asked for it.)
@pytest.mark.parametrize("D,Bs,before,kw", [(128, 128, 128, {}), (64, 64, 64, dict(stride_blocks=3)), (64, 64, 128, {}), (128, 128, 64, dict(stride_blocks=3))])
def test_a_small_fused_call_is_captured_after_selections(spa, D, Bs, before, kw):
    from paper_2602_21233_amd import binding
    S, ns, nl, k = 3 * Bs - 5, 1, 1, 1
    q, kk, v = _normal((1, 4, S, D), 71), _normal((1, 2, S, D), 72), _normal((1, 2, S, D), 73)
    spa.select(q, kk, before, ns, nl, k, **kw)
    p = binding.make_params(batch=1, n_q_heads=4, n_kv_heads=2, seq_len=S, head_dim=D, block_size=Bs, n_sink_blocks=ns, n_local_blocks=nl,
                            top_k_blocks=k, q=q, k=kk, v=v, out=q, **kw)
    ws = torch.empty(spa.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)
    pattern = (ns, nl, k, kw.get("stride_blocks", 0), 0)
    spa.attn(q, kk, v, *_random_lists(1, 4, 3, 0, 3, 3, 74), Bs, pattern=pattern)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        spa.fused(q, kk, v, Bs, ns, nl, k, workspace=ws, out=out, **kw)
    idx, cnt = spa.select(q, kk, Bs, ns, nl, k, **kw)
    want = spa.attn(q, kk, v, idx, cnt, Bs, pattern=pattern)
    for rep in range(3):
        out.zero_()
        ws.random_(0, 255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep
        spa.fused(q.flip(2).contiguous(), kk, v, Bs, ns, nl, k, **kw)      # eager work between replays
        torch.cuda.synchronize()


def _random_lists(B, Hl, NB, off, T, most, seed):
    """Well-formed lists of T places: up to `most` blocks, some earlier ones, ascending, then the diagonal block."""
    g = torch.Generator().manual_seed(seed)
    idx = torch.full((B, Hl, NB, T), -1, dtype=torch.int32)
    cnt = torch.empty((B, Hl, NB), dtype=torch.int32)
    for b in range(B):
        for h in range(Hl):
            for i in range(NB):
                n = int(torch.randint(0, min(most - 1, off + i) + 1, (1,), generator=g))
                row = torch.randperm(off + i, generator=g)[:n].sort().values.tolist() + [off + i] if off + i else [0]
                idx[b, h, i, : len(row)] = torch.tensor(row, dtype=torch.int32)
                cnt[b, h, i] = len(row)
    return idx.cuda(), cnt.cuda()


def _attn_reference(q, k, v, idx, cnt, Bs, most):
    """fp32 attention of every row over the blocks of its list (at most `most`, the last one causal), and the same sum over |v|."""
    B, Hq, S, D = q.shape
    NB, Skv = -(-S // Bs), k.shape[2]
    NBk = -(-Skv // Bs)
    pad = lambda x, n: torch.nn.functional.pad(x.float(), (0, 0, 0, n - x.shape[2]))
    qb = pad(q, NB * Bs).view(B, Hq, NB, Bs, D)
    kb, vb = (pad(x, NBk * Bs).view(B, -1, NBk, Bs, D) for x in (k, v))
    idx, cnt = (x.repeat_interleave(Hq // x.shape[1], 1) for x in (idx[..., :most], cnt))
    bi = torch.arange(B, device=q.device).view(B, 1, 1, 1)
    hi = (torch.arange(Hq, device=q.device) // (Hq // kb.shape[1])).view(1, Hq, 1, 1)
    at = idx.long().clamp(min=0)
    e = torch.arange(idx.shape[-1], device=q.device)
    kg, vg = (x[bi, hi, at].reshape(B, Hq, NB, -1, D) for x in (kb, vb))
    logits = (qb @ kg.transpose(-1, -2)).view(B, Hq, NB, Bs, -1, Bs) / D ** 0.5
    pos = torch.arange(Bs, device=q.device)
    last = (e == cnt.unsqueeze(-1) - 1).view(B, Hq, NB, 1, -1, 1)
    off_list = (e >= cnt.unsqueeze(-1)).view(B, Hq, NB, 1, -1, 1)
    logits = logits.masked_fill(off_list | (last & (pos.view(1, 1, Bs) > pos.view(Bs, 1, 1))), float("-inf"))
    w = logits.view(B, Hq, NB, Bs, -1).softmax(-1)
    return tuple((w @ x).view(B, Hq, NB * Bs, D)[:, :, :S] for x in (vg, vg.abs()))


# A KV head is served by a gang of 8, 4, 2 or 1 XCDs (by how many rows it has, and if the heads divide, in a ragged batch those of
# one entry), its query blocks dealt in runs of 8, 4, 2 or 1 (by how evenly they divide), forwards or in a snake: every row
# of every head is written, with its own head's keys and values and its own list.  That no row is dealt twice is asked of the rule
# itself (test_row_deal.py).  A prefix of 9000-odd tokens makes K and V^T of a head outgrow one L2 (runs), without
# one they fit (single rows).
@pytest.mark.parametrize("D,Bs", [(128, 64), (64, 64), (128, 128), (64, 128)])
@pytest.mark.parametrize("B,Hkv,ragged", [(1, 3, False), (1, 8, False), (2, 2, False), (2, 2, True), (1, 2, False), (8, 1, False), (8, 1, True)])
@pytest.mark.parametrize("NB,P,shared,n_dense", [(1, 0, 0, 0), (9, 0, 0, 0), (16, 9216, 0, 0), (17, 9216, 1, 0), (46, 9216, 0, 0),
                                                 (92, 18432, 0, 0), (64, 18432, 0, 0), (23, 0, 0, 3), (23, 18432, 1, 11)])
def test_every_row_is_dealt_once(spa, D, Bs, B, Hkv, ragged, NB, P, shared, n_dense):
    Hq, S, most = 2 * Hkv, NB * Bs - 5, 5
    q = _normal((B, Hq, S, D), 11)
    k = _normal((B, Hkv, P + S, D), 12)
    v = _normal((B, Hkv, P + S, D), 14)
    lens = [max(1, S - S * x // B - x % 3) for x in range(B)] if ragged else [S] * B
    dl = torch.tensor(lens, dtype=torch.int32).cuda() if ragged else None
    off, NBk = P // Bs, P // Bs + NB
    T = NBk if n_dense else min(NBk, most)
    idx, cnt = _random_lists(B, Hkv if shared else Hq, NB, off, T, most, 13)
    out = torch.full_like(q, float("nan"))
    spa.attn(q, k, v, idx, cnt, Bs, out=out, pattern=(0, 1, T - 1, 0, n_dense), group_shared=bool(shared), seq_lens=dl)
    want, scale = _attn_reference(q, k, v, idx, cnt, Bs, most)
    # weights are rounded to bf16 (2^-9) and divided by their own sum (2^-9 more), the result is rounded to bf16 (2^-9); fp32 logits
    # and sums add far less: 3 * 2^-9 of the sum of |w v|, 2^-7 with room
    for b, n in enumerate(lens):
        diff = (out[b, :, :n].float() - want[b, :, :n]).abs()
        assert (diff <= 2 ** -7 * scale[b, :, :n]).all(), (b, (diff / scale[b, :, :n]).max().item())
        assert out[b, :, n:].isnan().all()                 # rows past the entry's end are left alone


# Rows per workgroup of the score kernel go by the number of rows and of key blocks (test_score_rows.py); 4, 8, 16 or 32 key
# registers per lane by the key blocks alone.  The lists are the caller-score kernel's on the same scores, bit for bit, at the
# last row count of one group and the first of the next, with a row tile that is not full, and on both sides of every limit in
# key blocks.
@pytest.mark.parametrize("NB,Hq,P_blocks,D,kw", [
    (128, 8, 0, 128, {}), (129, 8, 0, 64, {}), (7, 8, 249, 128, {}), (7, 8, 250, 64, dict(stride_blocks=5)), (6, 4, 506, 128, {}),
    (6, 4, 507, 128, dict(n_dense_q_blocks=2)), (5, 8, 1019, 64, {}), (5, 8, 1020, 128, {}), (3, 8, 2045, 128, dict(stride_blocks=7)),
    (257, 4, 256, 64, {}), (258, 4, 256, 64, {}), (513, 32, 30, 64, {}), (512, 32, 30, 64, {}), (1025, 2, 3, 64, {}), (1030, 32, 0, 64, {})])
def test_rows_per_workgroup_of_the_score_kernel(spa, NB, Hq, P_blocks, D, kw):
    Bs, Hkv = 64, Hq // 2
    q = _normal((1, Hq, NB * Bs - 9, D), 31)
    k = _normal((1, Hkv, P_blocks * Bs + NB * Bs - 9, D), 32)
    for shared in (False, True) if Hq * NB <= 2048 else (False,):
        idx, cnt, sp = spa.select(q, k, Bs, 1, 2, 11, return_scores=True, group_shared=shared, **kw)
        w_idx, w_cnt = spa.topk_from_scores(sp, 1, 2, 11, **kw)
        assert torch.equal(idx, w_idx) and torch.equal(cnt, w_cnt)
        # the scores themselves: fp32 means and products of magnitude below 1 (split bf16 products, 2^-17 each)
        pick = torch.arange(0, NB, max(1, NB // 5), device="cuda").tolist() + [NB - 1]
        for h in (0, Hkv - 1):
            S = q.shape[2]
            heads = range(2 * h, 2 * h + 2) if shared else [2 * h + 1]
            kp = torch.stack([x.double().mean(0) for x in k[0, h].split(Bs)])
            for i in pick:
                qp = torch.stack([q[0, x, i * Bs:min(S, (i + 1) * Bs)].double().mean(0) for x in heads]).mean(0)
                want = (kp @ qp) / D ** 0.5
                n = P_blocks + i + 1
                got = sp[0, h if shared else 2 * h + 1, i]
                torch.testing.assert_close(got[:n].double(), want[:n], rtol=1e-4, atol=1e-5)
                assert torch.isneginf(got[n:]).all()


# (rows per workgroup, key blocks) of a kernel -> a shape that takes it: query blocks, lists (query heads, or KV heads where a group shares
# one), prefix blocks
SCORE_KERNELS = {
    (4, 256): (13, 16, 200), (4, 512): (13, 16, 470), (4, 1024): (13, 16, 990), (4, 2048): (13, 16, 1018),
    (8, 256): (37, 32, 200), (8, 512): (37, 32, 470), (8, 1024): (37, 32, 980), (8, 2048): (37, 32, 1000),
    (16, 1024): (200, 32, 820), (16, 2048): (202, 32, 904)}       # the last: rows on both sides of 1024 blocks, where the chunks meet
SCORE_OPTIONS = {
    "plain": {}, "shared": dict(group_shared=True), "strided": dict(stride_blocks=5, stride_reach_blocks=90),
    "dense": dict(n_dense_q_blocks=3), "strided_shared": dict(stride_blocks=7, group_shared=True), "ragged": dict(ragged=True),
    "schedule": dict(schedule=True), "head_pattern": dict(head_pattern=True), "output_aware": dict(output_aware=True),
    "special_values": dict(special=True), "special_output_aware": dict(special=True, output_aware=True),
    "all": dict(stride_blocks=9, ragged=True, schedule=True, head_pattern=True, output_aware=True)}


def score_case(kernel, option):
    """What the call looks like: batch, query heads, KV heads, query blocks, prefix blocks (as many rows whatever the option, except that
    lists shared by a group take 4 rows per workgroup up to 2048 rows)."""
    NB, heads, P = SCORE_KERNELS[kernel]
    o = SCORE_OPTIONS[option]
    B = 2 if o.get("ragged") else 1
    heads //= B
    if o.get("group_shared") and kernel[0] == 8:
        NB, P = 65, P - 28
    return (B, 2 * heads, heads, NB, P) if o.get("group_shared") else (B, heads, heads // 4, NB, P)


# Every kernel of the score stage with every option that changes its control flow: the lists against the rule on the kernel's
# own scores, from the oracle on some heads and from the caller-score kernel on all, the scores against float64 on some rows.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("option", SCORE_OPTIONS)
@pytest.mark.parametrize("kernel", SCORE_KERNELS, ids=lambda k: f"{k[0]}rows{k[1]}")
def test_options_on_every_score_kernel(spa, oracle, kernel, option, D):
    B, Hq, Hkv, NB, P = score_case(kernel, option)
    o = dict(SCORE_OPTIONS[option])
    Bs, ns, nl, topk = 64, 2, 3, 41
    S, off = NB * Bs - 21, P
    g = torch.Generator("cuda").manual_seed(51)
    rand = lambda H, n: torch.randn((B, H, n, D), generator=g, device="cuda").to(torch.bfloat16)
    q, k = rand(Hq, S), rand(Hkv, P * Bs + S)
    v = rand(Hkv, P * Bs + S) * (0.25 + torch.rand((B, Hkv, P * Bs + S, 1), generator=g, device="cuda")).to(torch.bfloat16)
    special = o.pop("special", False)
    if special:
        # by key block: zeros (ties at 0), a NaN, an infinity, huge values of either sign; by query block: zeros, large values
        kind = torch.randint(0, 12, (1, Hkv, off + NB), generator=g, device="cuda").repeat_interleave(Bs, 2)[:, :, :P * Bs + S, None]
        first = (torch.arange(P * Bs + S, device="cuda") % Bs == 5).view(1, 1, -1, 1)
        k = k.where(kind > 1, 0.0).where(~((kind == 2) & first), float("nan")).where(~((kind == 3) & first), float("inf"))
        k = k.where(kind != 4, k.abs() * 1e36).where(kind != 5, -k.abs() * 1e36)
        v = v.where((kind != 6) & (kind != 0), 0.0)
        kind = torch.randint(0, 6, (1, Hq, NB), generator=g, device="cuda").repeat_interleave(Bs, 2)[:, :, :S, None]
        q = q.where(kind > 0, 0.0).where(kind != 1, q.abs() * 1e3)
    shared = o.get("group_shared", False)
    Hl, G = (Hkv if shared else Hq), Hq // Hkv
    lens = [S, S - (NB // 3) * Bs - 7] if o.pop("ragged", False) else [S]
    sched = torch.linspace(topk, topk // 4, NB).round().to(torch.int32) if o.pop("schedule", False) else None
    hp = None
    if o.pop("head_pattern", False):
        hp = torch.tensor([[h % 4, h % 6, (h * 7) % (topk + 3)] for h in range(Hl)], dtype=torch.int32)
    aware = o.pop("output_aware", False)
    dev = lambda t: None if t is None else t.cuda()
    dl = torch.tensor(lens, dtype=torch.int32).cuda() if B > 1 else None
    kw = dict(o, seq_lens=dl, top_k_per_block=dev(sched), head_pattern=dev(hp), v=v if aware else None)
    idx, cnt, sp = spa.select(q, k, Bs, ns, nl, topk, return_scores=True, **kw)
    idx2, cnt2 = spa.select(q, k, Bs, ns, nl, topk, **kw)
    assert torch.equal(idx, idx2) and torch.equal(cnt, cnt2)               # the score output does not change the lists
    if special:
        tail = sp[..., :off]                               # causal for every row
        assert tail.isnan().any() and tail.isposinf().any() and tail.isneginf().any() and (aware or (tail == 0).any())
    rule = dict(stride_blocks=o.get("stride_blocks", 0), n_dense_q_blocks=o.get("n_dense_q_blocks", 0),
                stride_reach_blocks=o.get("stride_reach_blocks", 0))
    for b, n in enumerate(lens):
        nb = -(-n // Bs)
        assert (cnt[b, :, nb:] == 0).all() and (idx[b, :, nb:] == -1).all()
        sp_b = sp[b:b + 1, :, :nb, :off + nb].contiguous()
        sched_b = None if sched is None else sched[:nb].contiguous()
        t_idx, t_cnt = spa.topk_from_scores(sp_b, ns, nl, topk, top_k_per_block=dev(sched_b), head_pattern=dev(hp), **rule)
        Tb = t_idx.shape[-1]
        assert torch.equal(t_cnt[0], cnt[b, :, :nb]) and torch.equal(t_idx[0], idx[b, :, :nb, :Tb]) and (idx[b, :, :nb, Tb:] == -1).all()
        for h in (0, Hl // 2 + 1):
            w_idx, w_cnt = oracle.topk(sp_b[:, h:h + 1].cpu(), ns, nl, topk, sched_b, stride=rule["stride_blocks"],
                                       n_dense=rule["n_dense_q_blocks"], reach=rule["stride_reach_blocks"],
                                       head_pattern=None if hp is None else hp[h:h + 1].contiguous())
            assert torch.equal(cnt[b, h, :nb].cpu(), w_cnt[0, 0]) and torch.equal(idx[b, h, :nb, :Tb].cpu(), w_idx[0, 0])
            if special:
                continue
            # fp32 means and products of split bf16 operands, magnitude below 1 (2^-17 each); ln of a mean of fp32 norms
            kvh = h if shared else h // G
            keys = k[b, kvh, :P * Bs + n].double()
            kp = torch.stack([x.mean(0) for x in keys.split(Bs)])
            lvn = torch.stack([x.double().norm(dim=1).mean().log() for x in v[b, kvh, :P * Bs + n].split(Bs)]) if aware else 0.0
            for i in sorted({0, 1, nb // 2, nb - 2, nb - 1} | {i for i in (1023 - off, 1024 - off) if 0 <= i < nb}):
                heads = range(G * h, G * h + G) if shared else [h]
                qp = torch.stack([q[b, x, i * Bs:min(n, (i + 1) * Bs)].double().mean(0) for x in heads]).mean(0)
                want = (kp @ qp) / D ** 0.5 + lvn
                m = off + i + 1
                torch.testing.assert_close(sp[b, h, i, :m].double(), want[:m], rtol=1e-4, atol=1e-5)
                assert torch.isneginf(sp[b, h, i, m:off + nb]).all()


# Rows of 1025 to 2048 blocks, and from 513 on in workgroups of 16 rows, are selected from a list of the blocks that reach a bound, up to 112 of
# a budget, 64 sinks and 512 entries, and the general way (the other two kernels here, too) past any of these.  Budgets and sinks on both sides.
# Scores by `keys`: all different; of 40, 2 or 1 distinct values (ties at the threshold inside a list, more equal ones than it holds, all equal);
# "special": NaN, infinities, huge values and zeros in places; "few": most are NaN or -infinity, so that rows have fewer finite ones than wanted.
# The caller-score kernel, which keeps whole rows, is the reference.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kernel", [(4, 1024), (4, 2048), (8, 1024), (8, 2048), (16, 1024), (16, 2048)], ids=lambda k: f"{k[0]}rows{k[1]}")
@pytest.mark.parametrize("keys", [0, 40, 2, 1, "special", "few"])
def test_lists_by_bound(spa, kernel, keys, D):
    NB, Hq, P = SCORE_KERNELS[kernel]
    Hkv, Bs = Hq // 4, 64
    g = torch.Generator("cuda").manual_seed(71)
    q = torch.randn((1, Hq, NB * Bs, D), generator=g, device="cuda").to(torch.bfloat16)
    k = torch.randn((1, Hkv, (P + NB) * Bs, D), generator=g, device="cuda").to(torch.bfloat16)
    if keys in (40, 2, 1):
        which = torch.randint(0, keys, (P + NB,), generator=g, device="cuda")
        k = k.view(1, Hkv, P + NB, Bs, D)[:, :, which].reshape(1, Hkv, -1, D).contiguous()
    elif keys:
        # kinds of block: NaN, and with queries and keys of one sign each scores beyond the largest number
        q = q.abs() * 1e3
        kind = torch.rand((1, Hkv, P + NB), generator=g, device="cuda").repeat_interleave(Bs, 2)[..., None]
        nan, neg, pos, huge, zero = (0.47, 0.94, 0.95, 0.96, 0.97) if keys == "few" else (0.05, 0.1, 0.12, 0.16, 0.2)
        k = k.where(kind >= nan, float("nan")).where((kind < nan) | (kind >= neg), -k.abs() * 1e36).where((kind < neg) | (kind >= pos), k.abs() * 1e36)
        k = k.where((kind < pos) | (kind >= huge), k * 1e30).where((kind < huge) | (kind >= zero), 0.0)
    for ns, nl, topk in ((1, 4, 1), (0, 1, 64), (1, 4, 65), (64, 2, 127), (65, 2, 64), (3, 70, 128), (1, 4, 129), (2, 3, 0), (5, 9, P + NB - 20),
                         (1, 4, 112), (2, 3, 113)):
        idx, cnt, sp = spa.select(q, k, Bs, ns, nl, topk, return_scores=True)
        want_idx, want_cnt = spa.topk_from_scores(sp, ns, nl, topk)
        assert torch.equal(cnt, want_cnt) and torch.equal(idx, want_idx), (ns, nl, topk)
    if keys in ("special", "few"):
        seen = sp[..., :P]                                     # causal for every row
        assert seen.isnan().any() and seen.isposinf().any() and seen.isneginf().any() and (seen == 0).any()
        finite = seen.isfinite().sum(-1)
        assert (finite > 128).all() if keys == "special" else (finite < 127).any() and (finite > 1).all()


# ... and in calls whose first rows have fewer candidates than wanted, or only a few more, or, with budgets above 112, less than the 1024 that these take
# (128 is for the last shape alone).
SHORT_ROWS = {"16rows1024": (700, 32, 230), "8rows2048": (1030, 8, 0), "16rows2048": (1030, 32, 0), "16rows2048long": (600, 32, 950)}


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("shape", SHORT_ROWS)
def test_lists_by_bound_of_short_rows(spa, shape, D):
    NB, Hq, P = SHORT_ROWS[shape]
    g = torch.Generator("cuda").manual_seed(75)
    q = torch.randn((1, Hq, NB * 64, D), generator=g, device="cuda").to(torch.bfloat16)
    k = torch.randn((1, Hq // 4, (P + NB) * 64, D), generator=g, device="cuda").to(torch.bfloat16)
    for ns, nl, topk in ((1, 4, 1), (0, 1, 64), (64, 2, 65), (3, 70, 112), (1, 4, 113), (2, 1, 128)):
        idx, cnt, sp = spa.select(q, k, 64, ns, nl, topk, return_scores=True)
        want_idx, want_cnt = spa.topk_from_scores(sp, ns, nl, topk)
        assert torch.equal(cnt, want_cnt) and torch.equal(idx, want_idx), (ns, nl, topk)


# A mass budget is not searched for where the count budget cannot reach it whatever the scores.  Equal scores weigh 2^19 each, the most there is:
# the rows of one call then lie on both sides of that line and on it.  The caller-score kernel, which always searches, is the reference.
@pytest.mark.parametrize("NB,Bs,D", [(200, 64, 64), (300, 64, 128), (600, 64, 128), (1100, 64, 64)])
@pytest.mark.parametrize("equal", [True, False])
def test_mass_budget_beyond_the_count_budget(spa, NB, Bs, D, equal):
    q, k = _normal((1, 4, NB * Bs, D), 81), _normal((1, 2, NB * Bs, D), 82)
    if equal:
        k.zero_()
    sched = (torch.arange(NB, dtype=torch.int32) % 90).cuda()
    for topk, gamma, kw in ((1, 0.5, {}), (45, 0.25, {}), (89, 0.5, dict(top_k_per_block=sched)), (NB, 1.0, {}), (20, 0.5, dict(n_dense_q_blocks=3))):
        idx, cnt, sp = spa.select(q, k, Bs, 1, 2, topk, return_scores=True, mass_gamma=gamma, **kw)
        want_idx, want_cnt = spa.topk_from_scores(sp, 1, 2, topk, mass_gamma=gamma, **kw)
        assert torch.equal(cnt, want_cnt) and torch.equal(idx, want_idx), (topk, gamma)


# Chunks of the diagonal block that start behind a wavefront's last query (32 queries each) are left out: values there may be
# anything, the wavefront's rows keep their bits.
@pytest.mark.parametrize("D,Bs", [(128, 64), (64, 64), (128, 128), (64, 128)])
@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("NB", [1, 2, 7])
def test_values_behind_a_wavefronts_queries_take_no_part(spa, D, Bs, shared, NB):
    q, k, v = _normal((1, 4, NB * Bs, D), 61), _normal((1, 2, NB * Bs, D), 62), _normal((1, 2, NB * Bs, D), 63)
    idx, cnt = spa.select(q, k, Bs, 1, 2, 3, group_shared=shared)
    pattern = (1, 2, 3, 0, 0)
    want = spa.attn(q, k, v, idx, cnt, Bs, pattern=pattern, group_shared=shared)
    for end in range((NB - 1) * Bs + 32, NB * Bs, 32):     # the first keys behind the wavefronts of the last block
        bad = v.clone()
        bad[:, :, end:] = float("nan")
        got = spa.attn(q, k, bad, idx, cnt, Bs, pattern=pattern, group_shared=shared)
        assert torch.equal(got[:, :, :end], want[:, :, :end])
        vt = spa.transpose_v(bad, Bs)
        assert torch.equal(spa.attn_vt(q, k, vt, idx, cnt, Bs, pattern=pattern, group_shared=shared)[:, :, :end], want[:, :, :end])


# Lists shared by a KV group: the queries of the group's heads are pooled and averaged by the score kernel itself (352 workgroups
# and more, 384 with head_dim 64) or pooled with K and averaged by the score kernel, from a call with V (fused) or without (select).  Either way a row ranks the
# mean of its heads' block means: scores against fp64 (rtol 1e-4, atol 1e-5: fp32 sums of 128 products of magnitude <= 1), lists
# and counts as the rule gives on those scores.
@pytest.mark.parametrize("B,Hq,Hkv,S,D,Bs,P,ragged", [
    (1, 4, 2, 70, 64, 64, 0, False),             # one row and a bit
    (2, 6, 2, 64 * 9 + 1, 128, 64, 64 * 40, True),   # a last block of one token, empty blocks
    (1, 10, 2, 128 * 33 + 77, 128, 128, 0, False),   # groups of five
    (4, 16, 8, 128 * 39 + 5, 64, 128, 0, False),     # 4 x 8 x 10 workgroups of 4 rows: 320
    (4, 16, 8, 128 * 47 + 5, 64, 128, 0, False),     # 4 x 8 x 12: 384
    (4, 24, 8, 64 * 42 - 1, 128, 64, 64 * 300, True),    # groups of three, 352 workgroups, longer rows
    (8, 16, 8, 64 * 39, 64, 64, 0, False),           # 8 rows a workgroup, 320 of them
    (8, 16, 8, 64 * 47, 64, 64, 0, False),           # 384
    (1, 64, 32, 64 * 89 - 3, 64, 64, 64 * 200, False),   # ... over 289 key blocks
    (1, 96, 32, 64 * 90 - 7, 128, 64, 64 * 500, False),  # groups of three, 590
    (1, 64, 32, 64 * 90, 128, 64, 64 * 1000, False),     # 1090
    (1, 32, 16, 64 * 520 - 9, 128, 64, 0, False),        # 16 rows a workgroup, 528 of them
])
def test_group_means_of_pooled_queries(spa, B, Hq, Hkv, S, D, Bs, P, ragged):
    _check_selection(spa, B, Hq, Hkv, S, D, Bs, P, ragged, True)


def _check_selection(spa, B, Hq, Hkv, S, D, Bs, P, ragged, shared, kw=None):
    q, k, v = _normal((B, Hq, S, D), 1), _normal((B, Hkv, P + S, D), 2), _normal((B, Hkv, P + S, D), 3)
    lens = [max(1, S - 37 * b * Bs // 20) for b in range(B)] if ragged else [S] * B
    if ragged and not shared:
        lens[-1] = 0
    kw = dict(kw or {}, **(dict(seq_lens=torch.tensor(lens, dtype=torch.int32, device="cuda")) if ragged else {}))
    idx, cnt, sp = spa.select(q, k, Bs, 1, 2, 6, return_scores=True, group_shared=shared, **kw)
    out, idx2, cnt2 = spa.fused(q, k, v, Bs, 1, 2, 6, return_lists=True, group_shared=shared, **kw)
    if not kw:                                                           # the fused call's V^T is the attention call's
        assert torch.equal(out, spa.attn(q, k, v, idx, cnt, Bs, group_shared=shared))
    mean = lambda x: torch.stack([x[:, i: i + Bs].double().mean(1) for i in range(0, x.shape[1], Bs)], 1)
    for b, n in enumerate(lens):
        nb, off = -(-n // Bs), P // Bs
        assert (cnt[b, :, nb:] == 0).all()
        if n == 0:
            continue
        qp = mean(q[b, :, :n])
        qp = qp.view(Hkv, Hq // Hkv, nb, D)
        kp = mean(k[b, :, : P + n])
        want = ((qp.mean(1) if shared else qp.flatten(1, 2)) @ kp.transpose(1, 2).contiguous() / D ** 0.5).view(-1, nb, off + nb)
        seen = torch.arange(off + nb, device="cuda") <= torch.arange(off, off + nb, device="cuda").unsqueeze(1)
        got = sp[b, :, :nb, : off + nb].double()
        assert torch.allclose(got[:, seen], want[:, seen], rtol=1e-4, atol=1e-5), (b, (got[:, seen] - want[:, seen]).abs().max())
        assert torch.equal(idx[b, :, :nb], idx2[b, :, :nb]) and torch.equal(cnt[b], cnt2[b])
    if ragged:
        kw["seq_lens"] = torch.tensor([-(-n // Bs) * 64 for n in lens], dtype=torch.int32, device="cuda")   # in blocks of 64 there
    again, n_again = spa.topk_from_scores(sp, 1, 2, 6, **kw)
    assert torch.equal(again, idx) and torch.equal(n_again, cnt)


# Calls of up to 64 KB of K a head (96 in 4 blocks): K pooled by the score workgroups, V transposed beside them, in one launch.
@pytest.mark.parametrize("B,Hq,Hkv,S,D,Bs,P,ragged,kw", [
    (1, 1, 1, 1, 64, 64, 0, False, {}),
    (1, 1, 1, 512, 64, 64, 0, False, {}),
    (1, 4, 2, 768, 64, 64, 0, False, dict(stride_blocks=3)),     # 12 blocks: two launches
    (3, 4, 2, 511, 64, 64, 0, False, dict(stride_blocks=3)),     # the largest: 8 blocks
    (1, 6, 2, 383, 128, 128, 0, False, {}),                      # 96 KB in 3 blocks
    (2, 4, 2, 64, 64, 64, 64 * 7, True, {}),                     # a prefix, 8 blocks
    (1, 4, 2, 513, 64, 64, 0, False, {}),                        # just above 64 KB, in 9 blocks
    (2, 6, 2, 767, 64, 128, 0, False, {}),                       # groups of three, an odd number of blocks of V
    (3, 4, 1, 300, 128, 64, 0, True, {}),                        # lengths down to none
    (1, 8, 8, 129, 128, 128, 128, False, {}),                    # a prefix, a block of one token
    (1, 4, 2, 65, 64, 64, 64 * 10, False, dict(n_dense_q_blocks=1)),
    (2, 2, 2, 385, 128, 128, 0, True, {}),                       # just above: the two launches
])
def test_small_calls(spa, B, Hq, Hkv, S, D, Bs, P, ragged, kw):
    _check_selection(spa, B, Hq, Hkv, S, D, Bs, P, ragged, False, kw)


# ... with Q, K and V as views into one projection, each with strides of its own, tokens of other heads in between.
@pytest.mark.parametrize("B,Hq,Hkv,S,D,Bs", [(2, 4, 2, 200, 64, 64), (1, 4, 2, 511, 64, 64), (3, 2, 1, 383, 128, 128), (2, 6, 2, 191, 128, 64)])
def test_small_calls_on_strided_views(spa, B, Hq, Hkv, S, D, Bs):
    qkv = _normal((B, S, Hq + 3 * Hkv + 1, D), 81)
    q, k, v = (qkv[:, :, i: i + n].permute(0, 2, 1, 3) for i, n in ((0, Hq), (Hq, Hkv), (Hq + 2 * Hkv + 1, Hkv)))
    got = spa.fused(q, k, v, Bs, 1, 2, 1, return_lists=True)
    want = spa.fused(q.contiguous(), k.contiguous(), v.contiguous(), Bs, 1, 2, 1, return_lists=True)
    assert not v.is_contiguous() and v.stride() != k.contiguous().stride()
    assert all(torch.equal(x, y) for x, y in zip(got, want))
    idx, cnt = spa.select(q, k, Bs, 1, 2, 1)
    assert torch.equal(idx, got[1]) and torch.equal(cnt, got[2])
    assert torch.equal(got[0], spa.attn(q.contiguous(), k.contiguous(), v.contiguous(), idx, cnt, Bs, pattern=(1, 2, 1, 0, 0)))
