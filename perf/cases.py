"""The sparse-prefill calls that a serving program makes, as timed cases.

A case is a dict of plain values.  `call` says which entry points a pass goes through:

  fused   one prompt (or a padded batch of prompts, `ragged`) through the one-call entry point
  chunk   chunked prefill: the last `tokens` queries over a KV cache of `prefix` + `tokens` tokens whose
          transposed V is kept beside it: select, transposition of the chunk's own V blocks, attention
  select  the pattern stage alone, for programs that hand the block lists to an attention of their own

and `rule` how blocks are chosen: "topk" (uniform budget), "decay" (position-dependent budget), "stem" (that
plus the output-aware score), "mass" (cumulative-mass budget under the count cap), "strided" (static columns every 16
blocks) and "trishape" (the last 8 query blocks attend to everything).  `keys` names the key recipe: "hot" (planted
blocks that attract queries), "drift" (hot plus a trend along the sequence), "heavy" (hot on Student-t(3) keys).
Shapes are the package's own workloads and the sizes of its tests; 32 query / 8 KV heads of 128 are the 8B-class GQA
models that the path serves.
"""
import math

import torch

import paper_2602_21233_amd as spa
from paper_2602_21233_amd import binding

GAMMA = 0.9               # share of the softmax mass that a "mass" row keeps
STRIDE, DENSE_ROWS = 16, 8


def _case(name=None, *, call="fused", tokens, block=128, head_dim=128, q_heads=32, kv_heads=8, batch=1, prefix=0, sink=1,
          local=4, topk=64, rule="topk", shared=False, ragged=False, lse=False, keys="hot"):
    c = dict(call=call, tokens=tokens, block=block, head_dim=head_dim, q_heads=q_heads, kv_heads=kv_heads, batch=batch,
             prefix=prefix, sink=sink, local=local, topk=topk, rule=rule, shared=shared, ragged=ragged, lse=lse, keys=keys)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one head, 8 blocks; launches and latency are all there is
        _case("tiny_512", tokens=512, block=64, head_dim=64, q_heads=1, kv_heads=1, local=2, topk=2),
        # a short prompt of odd length under the settings of the long ones: every causal block is taken
        _case("short_prompt_1999", tokens=1999),
        # an ordinary prompt with small blocks
        _case("prompt_16k_b64", tokens=16384, block=64, topk=16),
        # an ordinary prompt; the log-sum-exp is kept, as a program does that merges partial attention
        _case("prompt_32k", tokens=32768, local=2, topk=32, lse=True),
        # the long prompt that the path is made for
        _case("prompt_128k", tokens=131072, keys="drift"),
        # the longest one: 40 heads, heavy-tailed keys
        _case("prompt_256k", tokens=262144, q_heads=40, sink=2, local=8, topk=96, keys="heavy"),
        # serving: a chunk of a long prompt goes over the KV cache that holds the rest
        _case("chunk_2k_at_96k", call="chunk", tokens=2048, prefix=98304),
        # serving: a padded batch of prompts of different, mostly odd lengths
        _case("ragged_batch_6k", tokens=6000, block=64, batch=6, topk=16, ragged=True),
        # output-aware ranking under a decaying budget, a length that is no multiple of the block
        _case("stem_49k", tokens=49000, rule="stem"),
        # one list per KV head, the smaller head size
        _case("shared_16k_d64", tokens=16384, head_dim=64, local=2, topk=32, shared=True),
        # the pattern stage alone, longest rows
        _case("select_256k", call="select", tokens=262144, q_heads=40, sink=2, local=8, topk=96, keys="heavy"),
        # the pattern stage alone under a cumulative-mass budget
        _case("select_mass_64k", call="select", tokens=65536, rule="mass"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    call = rng.choice(("fused", "fused", "fused", "chunk", "ragged", "select"))
    q_heads, kv_heads = rng.choice(((32, 8), (32, 8), (40, 8), (16, 2), (8, 8)))
    c = dict(block=rng.choice((64, 128, 128)), head_dim=rng.choice((64, 128, 128, 128)), q_heads=q_heads, kv_heads=kv_heads,
             sink=rng.randint(0, 2), local=rng.randint(1, 8), topk=_log_uniform(rng, 4, 96), keys=rng.choice(("hot", "drift", "heavy")),
             rule=rng.choice(("topk", "topk", "topk", "decay", "stem", "strided", "trishape")),
             shared=rng.random() < 0.2, lse=rng.random() < 0.3)
    if call == "fused":
        c["tokens"] = _log_uniform(rng, 300, 131072)
    elif call == "select":
        c.update(call="select", tokens=_log_uniform(rng, 4096, 262144), lse=False)
        if rng.random() < 0.3:
            c["rule"] = "mass"
    elif call == "chunk":
        c.update(call="chunk", tokens=_log_uniform(rng, 256, 8192), prefix=_log_uniform(rng, 2048, 131072) // 128 * 128,
                 rule=rng.choice(("topk", "decay")))
    else:
        c.update(tokens=_log_uniform(rng, 500, 12000), batch=rng.randint(2, 8), ragged=True, lse=False)
    if rng.random() < 0.5:      # half of the drawn lengths are whole blocks
        c["tokens"] = max(c["block"], c["tokens"] // c["block"] * c["block"])
    return _case(**c)


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        c = _draw_once(rng)
        if _blocks(c, c["prefix"] + c["tokens"]) <= 4096 and work(c)["flops"] <= most:
            return c


# ---- sizes ------------------------------------------------------------------------------------------------------

def _blocks(case, tokens):
    return -(-tokens // case["block"])


def _lengths(case):
    """Tokens of every batch entry: all of them, or a spread of lengths down from the padded one, mostly odd."""
    n, b = case["tokens"], case["batch"]
    if not case["ragged"]:
        return [n] * b
    return [max(1, n - (n * x) // (b + 1) - (x % 3)) for x in range(b)]


def _schedule(case):
    """Budget per query block, falling linearly from the full one to a quarter of it (the decaying rules)."""
    nb, k = _blocks(case, case["tokens"]), case["topk"]
    if case["rule"] not in ("decay", "stem"):
        return None
    return [int(round(k + (k // 4 - k) * x / max(nb - 1, 1))) for x in range(nb)]


def _static(case, i, nb_k):
    """Static blocks of the query block at block position i."""
    n = i + 1
    if case["rule"] == "trishape" and i >= nb_k - DENSE_ROWS:
        return n
    lo = max(i - case["local"] + 1, min(case["sink"], n))
    found = min(case["sink"], n) + n - lo
    if case["rule"] == "strided":
        found += sum(1 for j in range(i % STRIDE, lo, STRIDE) if j >= case["sink"])
    return found


def _static_mask(case, i, j, nb_k):
    """Which blocks j are static for the query blocks at positions i (tensors that broadcast)."""
    st = (j < case["sink"]) | (j >= i - case["local"] + 1)
    if case["rule"] == "strided":
        st = st | ((i - j) % STRIDE == 0)
    if case["rule"] == "trishape":
        st = st | (i >= nb_k - DENSE_ROWS)
    return st & (j <= i)


def work(case):
    D, Bs, off = case["head_dim"], case["block"], case["prefix"] // case["block"]
    sched = _schedule(case)
    lists = case["kv_heads"] if case["shared"] else case["q_heads"]
    flops, nbytes = 0.0, 0.0
    for n in _lengths(case):
        nb_k = off + _blocks(case, n)
        kv, taken = case["prefix"] + n, 0
        for iq in range(_blocks(case, n)):
            i, rows = iq + off, min(Bs, n - iq * Bs)
            st = _static(case, i, nb_k)
            c = min(i + 1, st + (sched[iq] if sched else case["topk"]))
            taken += c
            flops += 2.0 * lists * (i + 1) * D                                   # pooled scores
            if case["call"] != "select":
                flops += 4.0 * case["q_heads"] * D * (rows * (c - 1) * Bs + rows * (rows + 1) / 2)
        nbytes += 2.0 * D * (case["q_heads"] * n + case["kv_heads"] * kv)       # Q, K
        if case["call"] == "chunk":
            nbytes += 2.0 * D * case["kv_heads"] * (kv + 2 * n)                  # V^T, and the chunk's V turned into it
        elif case["call"] == "fused" or case["rule"] == "stem":
            nbytes += 2.0 * D * case["kv_heads"] * kv                            # V
        if case["call"] != "select":
            nbytes += 2.0 * D * case["q_heads"] * n + (4.0 * case["q_heads"] * n if case["lse"] else 0.0)
        nbytes += 4.0 * lists * taken                                            # the block lists
    return {"bytes": nbytes, "flops": flops}


# ---- inputs ------------------------------------------------------------------------------------------------------

def _inputs(case, seed):
    """Q [B,Hq,S,D], K and V [B,Hkv,P+S,D] in bf16 on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + 17)
    B, D, S, Skv, Bs = case["batch"], case["head_dim"], case["tokens"], case["prefix"] + case["tokens"], case["block"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    q = torch.empty((B, case["q_heads"], S, D), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((B, case["kv_heads"], Skv, D), dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    nb = Skv // Bs                                   # whole blocks: the ones that can be hot
    for b in range(B):
        for h in range(case["q_heads"]):
            q[b, h] = normal(S, D)
        for h in range(case["kv_heads"]):
            v[b, h] = normal(Skv, D)
            x = normal(Skv, D)
            if case["keys"] == "heavy":
                x /= (normal(3, Skv, 1).square().sum(0) / 3.0).sqrt()
            u, w = normal(D), normal(D)
            if nb > case["sink"]:
                hot = torch.randperm(nb - case["sink"], generator=g, device="cuda")[: max(1, nb // 16)] + case["sink"]
                x[: nb * Bs].view(nb, Bs, D)[hot] += 3.0 * u / u.norm()
            if case["keys"] == "drift":
                x += torch.arange(Skv, device="cuda", dtype=torch.float32).unsqueeze(1) / Skv * (w / w.norm())
            k[b, h] = x
    return q, k, v


def _pattern_kw(case):
    return dict(stride_blocks=STRIDE if case["rule"] == "strided" else 0,
                n_dense_q_blocks=DENSE_ROWS if case["rule"] == "trishape" else 0)


def prepare(case, seed):
    """The tensors, the workspace and the output buffer that a program keeps over its calls; for a chunk also the
    transposed V of the prefix."""
    q, k, v = _inputs(case, seed)
    s = dict(case=case, q=q, k=k, v=v, kw=_pattern_kw(case))
    if case["call"] != "select":
        s["out"] = torch.zeros_like(q)
    p = binding.make_params(batch=case["batch"], n_q_heads=case["q_heads"], n_kv_heads=case["kv_heads"], seq_len=case["tokens"],
                            head_dim=case["head_dim"], block_size=case["block"], n_sink_blocks=case["sink"],
                            n_local_blocks=case["local"], top_k_blocks=case["topk"], q=q, k=k, v=v, out=q,
                            lists_per_kv_head=case["shared"], kv_prefix_len=case["prefix"], **s["kw"])
    s["ws"] = torch.empty(spa.workspace_bytes(p), dtype=torch.uint8, device="cuda")
    s["rule"] = {}
    sched = _schedule(case)
    if sched is not None:
        s["rule"]["top_k_per_block"] = torch.tensor(sched, dtype=torch.int32, device="cuda")
    if case["rule"] == "mass":
        s["rule"]["mass_gamma"] = GAMMA
    if case["ragged"]:
        s["rule"]["seq_lens"] = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")
    if case["call"] == "chunk":
        n = case["prefix"] // case["block"]
        s["vt"] = spa.transpose_v(v, case["block"], blocks_per_head=n + _blocks(case, case["tokens"]) + 8, n_blocks=n)
    return s


def run(state):
    c = state["case"]
    q, k, v, kw, rule = state["q"], state["k"], state["v"], state["kw"], state["rule"]
    budget = (c["block"], c["sink"], c["local"], c["topk"])
    if c["call"] == "fused":
        got = spa.fused(q, k, v, *budget, return_lse=c["lse"], return_lists=True, workspace=state["ws"], out=state["out"],
                        output_aware=c["rule"] == "stem", group_shared=c["shared"], **kw, **rule)
        return dict(zip(("out", "lse", "idx", "cnt") if c["lse"] else ("out", "idx", "cnt"), got))
    idx, cnt = spa.select(q, k, *budget, workspace=state["ws"], v=v if c["rule"] == "stem" else None, group_shared=c["shared"],
                          **kw, **rule)
    if c["call"] == "select":
        return dict(idx=idx, cnt=cnt)
    vt = spa.transpose_v(v, c["block"], vt=state["vt"], blocks_per_head=state["vt"].shape[2], first_block=c["prefix"] // c["block"])
    got = spa.attn_vt(q, k, vt, idx, cnt, c["block"], return_lse=c["lse"], out=state["out"], group_shared=c["shared"],
                      pattern=(c["sink"], c["local"], c["topk"], kw["stride_blocks"], kw["n_dense_q_blocks"]))
    out, lse = got if c["lse"] else (got, None)
    return dict(out=out, idx=idx, cnt=cnt, vt=vt, **({"lse": lse} if c["lse"] else {}))


def tolerance(case):
    # Outputs and weights are bf16 (2^-9 each); block lists hold whole numbers that can differ where two pooled scores
    # are equal to within fp32 rounding, and a row of another list gives another output row.
    if case["call"] == "select":
        return {"rel": 0.0, "max": 0.0, "differ": 0.004}
    return {"rel": 1.2e-2, "max": 0.25, "differ": 0.004}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

def _pooled(x, Bs):
    """Block means of x [S, D], fp64."""
    S, D = x.shape
    nb = -(-S // Bs)
    pad = torch.zeros((nb * Bs, D), dtype=torch.float64, device=x.device)
    pad[:S] = x
    n = torch.full((nb, 1), float(Bs), dtype=torch.float64, device=x.device)
    n[-1] = S - (nb - 1) * Bs
    return pad.view(nb, Bs, D).sum(1) / n


def _lists(case, qp, kp, lvn, off, sched, T):
    """Block lists [NB, T] and counts [NB] of one head from its pooled queries and keys."""
    NB, nb_k = qp.shape[0], kp.shape[0]
    i = torch.arange(off, off + NB, device=qp.device).unsqueeze(1)
    j = torch.arange(nb_k, device=qp.device).unsqueeze(0)
    score = (qp @ kp.t()) / math.sqrt(case["head_dim"])
    if lvn is not None:
        score = score + lvn
    st = _static_mask(case, i, j, nb_k)
    cand = (j <= i) & ~st
    ranked, order = score.masked_fill(~cand, -math.inf).sort(dim=1, descending=True, stable=True)
    n_cand = cand.sum(1)
    budget = torch.full_like(n_cand, case["topk"]) if sched is None else torch.tensor(sched[:NB], device=qp.device)
    if case["rule"] == "mass":
        m = score.masked_fill(j > i, -math.inf).amax(1, keepdim=True)

        def weight(x):
            t = (x - m) * math.log2(math.e)
            return torch.where(t >= -40.0, torch.floor(torch.exp2(t) * 524288.0 + 0.5), torch.zeros_like(t))

        w = weight(score)
        target = torch.ceil(math.floor(GAMMA * 65536 + 0.5) * (w * (j <= i)).sum(1) / 65536.0)
        got = (w * st).sum(1, keepdim=True) + weight(ranked).cumsum(1)
        first = ((w * st).sum(1) < target).long()           # 0 where the static blocks hold enough
        budget = torch.minimum(budget, first * ((got < target.unsqueeze(1)).sum(1) + 1))
    take = torch.minimum(budget, n_cand)
    chosen = torch.zeros_like(cand).scatter(1, order, j < take.unsqueeze(1)) & cand | st
    cnt = chosen.sum(1)
    at = torch.where(chosen, j.expand_as(chosen), torch.full_like(j, nb_k).expand_as(chosen)).sort(dim=1).values[:, :T]
    return torch.where(at < nb_k, at, torch.full_like(at, -1)).int(), cnt.int()


def _attend(case, q, k, v, idx, cnt, off):
    """Softmax attention of one head over its lists, fp64: out [S, D], lse [S]."""
    S, D = q.shape
    Bs, nb_k = case["block"], -(-k.shape[0] // case["block"])
    NB = idx.shape[0]

    def padded(x, n):
        y = torch.zeros((n * Bs, D), dtype=torch.float64, device=x.device)
        y[: x.shape[0]] = x
        return y.view(n, Bs, D)

    qb, kb, vb = padded(q, NB), padded(k, nb_k), padded(v, nb_k)
    out = torch.empty((NB, Bs, D), dtype=torch.float64, device=q.device)
    lse = torch.empty((NB, Bs), dtype=torch.float64, device=q.device)
    T = int(cnt.max())
    step = max(1, (1 << 27) // (T * Bs * D))
    tok = torch.arange(Bs, device=q.device)
    for r in range(0, NB, step):
        at = idx[r:r + step, :T].long()
        n = at.shape[0]
        blk = at.clamp(min=0)
        s = torch.bmm(qb[r:r + step], kb[blk].view(n, T * Bs, D).transpose(1, 2).contiguous()) / math.sqrt(D)
        pos = (blk.unsqueeze(2) * Bs + tok).view(n, 1, T * Bs)
        qpos = ((torch.arange(r, r + n, device=q.device) + off).unsqueeze(1) * Bs + tok).unsqueeze(2)
        gone = (at < 0).repeat_interleave(Bs, 1).unsqueeze(1)
        s.masked_fill_((pos > qpos) | gone, -math.inf)
        lse[r:r + n] = torch.logsumexp(s, 2)
        out[r:r + n] = torch.bmm(torch.exp_(s.sub_(lse[r:r + n].unsqueeze(2))), vb[blk].view(n, T * Bs, D))
    return out.view(-1, D)[:S], lse.view(-1)[:S]


def exact(case, seed):
    q, k, v = _inputs(case, seed)
    B, Hq, S, D = q.shape
    Bs, Hkv, off = case["block"], case["kv_heads"], case["prefix"] // case["block"]
    G, NB, nb_k = Hq // Hkv, _blocks(case, S), _blocks(case, k.shape[2])
    lists = Hkv if case["shared"] else Hq
    T = min(nb_k, case["sink"] + case["local"] + case["topk"] + ((nb_k - 1) // STRIDE if case["rule"] == "strided" else 0))
    if case["rule"] == "trishape":
        T = nb_k
    idx = torch.full((B, lists, NB, T), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((B, lists, NB), dtype=torch.int32, device="cuda")
    attend = case["call"] != "select"
    out = torch.zeros((B, Hq, S, D), dtype=torch.float64, device="cuda") if attend else None
    lse = torch.zeros((B, Hq, S), dtype=torch.float64, device="cuda")
    sched = _schedule(case)
    for b, n in enumerate(_lengths(case)):
        kv = case["prefix"] + n
        for h in range(Hkv):
            kh, vh = k[b, h, :kv].double(), v[b, h, :kv].double()
            kp = _pooled(kh, Bs)
            lvn = None
            if case["rule"] == "stem":
                lvn = torch.log(_pooled(vh.norm(dim=1, keepdim=True).expand(-1, D), Bs)[:, 0])
            heads = [h * G + g for g in range(G)]
            qps = [_pooled(q[b, x, :n].double(), Bs) for x in heads]
            if case["shared"]:
                qps = [torch.stack(qps).mean(0)]
            for x, qp in enumerate(qps):
                row = h if case["shared"] else heads[x]
                a, c = _lists(case, qp, kp, lvn, off, sched, T)
                idx[b, row, : a.shape[0], : a.shape[1]], cnt[b, row, : c.shape[0]] = a, c
            if attend:
                nb = _blocks(case, n)
                for x in heads:
                    row = h if case["shared"] else x
                    out[b, x, :n], lse[b, x, :n] = _attend(case, q[b, x, :n].double(), kh, vh, idx[b, row, :nb], cnt[b, row, :nb], off)
    if not attend:
        return dict(idx=idx, cnt=cnt)
    got = dict(out=out, idx=idx, cnt=cnt, **({"lse": lse} if case["lse"] else {}))
    if case["call"] == "chunk":
        vt = torch.zeros((B, Hkv, nb_k + 8, D, Bs), dtype=torch.float64, device="cuda")
        full = torch.zeros((B, Hkv, nb_k * Bs, D), dtype=torch.float64, device="cuda")
        full[:, :, : v.shape[2]] = v
        vt[:, :, :nb_k] = full.view(B, Hkv, nb_k, Bs, D).transpose(3, 4)
        got["vt"] = vt
    return got
