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


# Rows per workgroup of the score kernel go by the number of rows and of key blocks: 4 up to 1024 rows, 8 up to 16384
# (1025 - 2048 key blocks: 32768), then 16; 4, 8, 16 or 32 key registers per lane.  The lists are the caller-score kernel's
# on the same scores, bit for bit, at the last row count of one group and the first of the next, with a row tile that
# is not full, and on both sides of every limit in key blocks.
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
