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


def _random_lists(B, Hl, NB, off, T, seed):
    """Well-formed lists: a random number of earlier blocks, ascending, then the diagonal block."""
    g = torch.Generator().manual_seed(seed)
    idx = torch.full((B, Hl, NB, T), -1, dtype=torch.int32)
    cnt = torch.empty((B, Hl, NB), dtype=torch.int32)
    for b in range(B):
        for h in range(Hl):
            for i in range(NB):
                n = int(torch.randint(0, min(T - 1, off + i) + 1, (1,), generator=g))
                row = torch.randperm(off + i, generator=g)[:n].sort().values.tolist() + [off + i] if off + i else [0]
                idx[b, h, i, : len(row)] = torch.tensor(row, dtype=torch.int32)
                cnt[b, h, i] = len(row)
    return idx.cuda(), cnt.cuda()


# A KV head is served by a gang of 8, 4, 2 or 1 XCDs (by how many rows it has, and if the heads divide), its query blocks dealt in
# runs of 8, 4, 2 or 1 (by how evenly they divide), forwards or in a snake: every row of every head is served exactly once.
# A prefix of 9000-odd tokens makes K and V^T of a head outgrow one L2 (runs), without one they fit (single rows).
@pytest.mark.parametrize("D,Bs", [(128, 64), (64, 64), (128, 128)])
@pytest.mark.parametrize("B,Hkv", [(1, 3), (1, 8), (2, 2), (1, 2)])
@pytest.mark.parametrize("NB,P,shared,n_dense", [(1, 0, 0, 0), (9, 0, 0, 0), (16, 9216, 0, 0), (17, 9216, 1, 0), (46, 9216, 0, 0),
                                                 (92, 18432, 0, 0), (64, 18432, 0, 0), (23, 0, 0, 3), (23, 18432, 1, 11)])
def test_every_row_is_dealt_once(spa, D, Bs, B, Hkv, NB, P, shared, n_dense):
    Hq, S = 2 * Hkv, NB * Bs - 5
    q = _normal((B, Hq, S, D), 11)
    k = _normal((B, Hkv, P + S, D), 12)
    v = torch.ones_like(k)
    off, NBk = P // Bs, P // Bs + NB
    T = NBk if n_dense else min(NBk, 5)
    idx, cnt = _random_lists(B, Hkv if shared else Hq, NB, off, T, 13)
    cnt.clamp_(max=5)                                    # long rows add nothing here (their last entry is then not the diagonal block)
    out = torch.full_like(q, float("nan"))
    spa.attn(q, k, v, idx, cnt, Bs, out=out, pattern=(0, 1, T - 1, 0, n_dense), group_shared=bool(shared))
    # weights are normalised by the sum of the very weights that are used, values are 1: the result is 1 up to the
    # rounding of fp32 sums and one bf16 rounding (2^-8)
    assert torch.isfinite(out).all()
    assert (out.float() - 1).abs().max().item() <= 2 ** -8
