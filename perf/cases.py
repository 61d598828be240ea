"""The calls this library is used for, as measurable cases.

A case is one call (or one selector + forward step) of the public entry points
on inputs of a stated shape.  The listed cases follow the repository's own
workloads (synthetic/workloads.py, bench.py and the tests); draw() spreads over
the same ranges.  Inputs are made on the GPU from a seed: keys with a shared
offset per block, queries aligned with a few key blocks, everything else N(0, 1),
rounded to bf16, as the workload generator does.

Operations
  step    selector, then sparse forward on its lists (a layer's whole call)
  noalloc the same for a caller that cannot allocate: static selector scratch,
          single-pass forward without a workspace
  select  the selector alone (scorer: separate kernels, fused or static)
  sparse  the sparse forward on given lists
  dense   the dense forward (the coarse scales)
  mass    the token-wise bound of the retained-mass analysis
"""
import math

import torch

from paper_2608_10519_amd import sparstar as S

DEV = "cuda"


def _case(name, op, **kw):
    c = dict(op=op, batch=1, heads=24, d=128, block=64, lq=72_000, l_ref=72_000, l_text=512, rho=0.25, spread=0.0,
             clip=2, aligned=16, split=True, scorer="separate", rows=8)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # smallest call: launch and host latency of the whole step
        _case("tiny_step", "step", heads=2, d=64, lq=512, l_ref=512, l_text=128, aligned=3),
        # a step in a serving loop that may not allocate: ragged lengths, per-head budgets
        _case("noalloc_step", "noalloc", heads=8, lq=6413, l_ref=44_821, rho=0.275, spread=0.5, aligned=6,
              split=False),
        # head dim 64, two batch elements, the first clip's keep set, nothing a multiple of a block
        _case("d64_ragged_sparse", "sparse", batch=2, heads=12, d=64, block=128, lq=11_001, l_ref=20_517, l_text=300,
              rho=0.4, clip=1, aligned=5),
        # mid pyramid scale: selector and forward
        _case("mid_select", "select", lq=11_520, aligned=8),
        _case("mid_sparse", "sparse", lq=11_520, aligned=8),
        # 720p final scale, the headline shape: selector and forward at 25%
        _case("p720_select", "select"),
        _case("p720_sparse", "sparse"),
        # 720p at 10% with per-head budgets (the density sweep)
        _case("p720_sweep10_sparse", "sparse", rho=0.10, spread=0.5),
        # 720p at the paper's block size and finest-scale density
        _case("p720_b128_sparse", "sparse", block=128, rho=0.09375),
        # coarse pyramid scales run dense: the first (few queries, many keys) and the third
        _case("scale1_dense", "dense", lq=2880),
        _case("scale3_dense", "dense", lq=25_920),
        # retained-mass analysis: the token-wise bound on sampled rows of every head
        _case("p720_mass", "mass"),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    op = rng.choice(["step", "noalloc", "select", "select", "sparse", "sparse", "sparse", "dense", "dense", "mass"])
    d = rng.choice([64, 128, 128, 128])
    block = rng.choice([64, 64, 128])
    lq = _log(rng, 64, 72_000)
    l_ref = _log(rng, 64, 72_000)
    l_text = rng.randint(1, 512)
    heads = _log(rng, 1, 24)
    batch = rng.choice([1, 1, 1, 2])
    rho = math.exp(rng.uniform(math.log(0.05), math.log(0.65)))
    spread = rng.choice([0.0, 0.5])
    clip = rng.choice([1, 2, 2])
    split = op != "noalloc" and rng.random() < 0.85
    scorer = rng.choice(["separate", "separate", "separate", "fused", "static"])
    rows = rng.randint(1, 16)
    while True:
        c = _case(None, op, batch=batch, heads=heads, d=d, block=block, lq=lq, l_ref=l_ref, l_text=l_text, rho=rho,
                  spread=spread, clip=clip, aligned=rng.randint(1, 16), split=split, scorer=scorer, rows=rows)
        # no drawn case costs more than the largest listed one (32 TFLOP at head
        # dim 128); head dim 64 and the single pass do less per second
        cap = 24e12 / (3 if d == 64 else 1) / (1 if split else 2)
        if work(c)["flops"] <= cap and _fits(c):
            return c
        if batch > 1:
            batch = 1
        elif heads > 1:
            heads //= 2
        else:
            lq = max(64, lq // 2)


def _lk(c):
    return c["l_ref"] + c["l_text"] + c["lq"]


def _blocks(c):
    return -(-c["lq"] // c["block"]), -(-_lk(c) // c["block"])


def _fits(c):
    """Whether the scorer takes the case (static scratch, fused row length)."""
    if c["op"] not in ("select", "noalloc"):
        return True
    n_q, n_k = _blocks(c)
    bh = c["batch"] * c["heads"]
    scorer = "static" if c["op"] == "noalloc" else c["scorer"]
    if scorer == "static":
        need = bh * (n_q + n_k) * (4 * c["d"] + 4) + bh * n_q * (n_k + 32) * 4 + 2048
        return need <= S.STATIC_SCRATCH_BYTES
    return scorer != "fused" or n_k <= S.FUSED_MAX_BLOCKS


def _segments(c):
    ref = (0, c["l_ref"])
    text = (c["l_ref"], c["l_ref"] + c["l_text"])
    return text, ref


def _keep_ranges(c):
    text, ref = _segments(c)
    return [text, ref] if c["clip"] == 1 else [text]


def _forced(c):
    n_k = _blocks(c)[1]
    f = [False] * n_k
    for a, e in _keep_ranges(c):
        for j in range(a // c["block"], -(-e // c["block"])):
            f[j] = True
    return f


def _budgets(c):
    """One density per head: the nominal one, or spread evenly around it."""
    h, s = c["heads"], c["spread"]
    if not s:
        return [c["rho"]] * h
    return [min(1.0, c["rho"] * (1 - s + 2 * s * i / max(1, h - 1))) for i in range(h)]


def _counts(c):
    """Listed blocks per row of each head, and how many blocks are forced."""
    forced = sum(_forced(c))
    n_sel = _blocks(c)[1] - forced
    ks = []
    for rho in _budgets(c):
        p = rho * n_sel
        r = round(p)
        k = r if abs(p - r) <= 1e-9 * max(1, n_sel) else math.ceil(p)
        ks.append(min(n_sel, max(1, int(k))))
    return [forced + k for k in ks], forced


def work(c):
    bh, d, lq, lk = c["batch"] * c["heads"], c["d"], c["lq"], _lk(c)
    n_q, n_k = _blocks(c)
    counts, _ = _counts(c)
    lists = 4.0 * c["batch"] * n_q * (sum(counts) + len(counts))
    sel = dict(bytes=2.0 * bh * (lq + lk) * d + lists, flops=2.0 * bh * n_q * n_k * d + 1.0 * bh * (lq + lk) * d)
    listed_keys = c["batch"] * sum(min(lk, n * c["block"]) for n in counts)
    att = dict(bytes=2.0 * bh * (2 * lq + 2 * lk) * d + 4.0 * bh * lq + lists, flops=4.0 * lq * listed_keys * d)
    if c["op"] == "select":
        return sel
    if c["op"] == "sparse":
        return att
    if c["op"] in ("step", "noalloc"):
        # V is the forward's only tensor that the selector has not read already
        return dict(bytes=sel["bytes"] + 2.0 * bh * (lq + lk) * d + 4.0 * bh * lq, flops=sel["flops"] + att["flops"])
    if c["op"] == "dense":
        return dict(bytes=2.0 * bh * (2 * lq + 2 * lk) * d + 4.0 * bh * lq, flops=4.0 * bh * lq * lk * d)
    return dict(bytes=2.0 * bh * lk * d + 2.0 * bh * c["rows"] * d + 12.0 * bh * c["rows"],
                flops=2.0 * bh * c["rows"] * lk * d)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _inputs(c, seed, with_v):
    """q [B,H,Lq,D], k and v [B,H,Lk,D] in bf16 with planted block structure."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    bh, d, lq, lk, b = c["batch"] * c["heads"], c["d"], c["lq"], _lk(c), c["block"]
    n_q, n_k = _blocks(c)
    q = torch.empty(bh, lq, d, dtype=torch.bfloat16, device=DEV)
    k = torch.empty(bh, lk, d, dtype=torch.bfloat16, device=DEV)
    v = torch.empty(bh, lk, d, dtype=torch.bfloat16, device=DEV) if with_v else None

    def randn(*shape):
        return torch.randn(*shape, generator=g, device=DEV)

    # the blocks of each token, so that an offset per block is one gather
    qb = torch.arange(lq, device=DEV) // b
    kb = torch.arange(lk, device=DEV) // b
    for i in range(bh):
        off = randn(n_k, d)
        off = 2.0 * off / off.norm(dim=1, keepdim=True)
        pick = torch.randint(0, n_k, (n_q, c["aligned"]), generator=g, device=DEV)
        qoff = 1.5 * off[pick].sum(dim=1)
        k[i] = (randn(lk, d) + off[kb]).to(torch.bfloat16)
        q[i] = (randn(lq, d) + qoff[qb]).to(torch.bfloat16)
        if with_v:
            v[i] = randn(lk, d).to(torch.bfloat16)
    shape = (c["batch"], c["heads"])
    return q.view(*shape, lq, d), k.view(*shape, lk, d), v.view(*shape, lk, d) if with_v else None


def _pooled(x, b):
    """Block means over the nominal block length, [n, d]."""
    n = -(-x.shape[0] // b)
    pad = torch.zeros(n * b, x.shape[1], dtype=x.dtype, device=x.device)
    pad[: x.shape[0]] = x
    return pad.view(n, b, -1).sum(dim=1) / b


def _lists(c, q, k, dtype):
    """Ascending lists of the forced blocks and the best-scoring others, in plain torch."""
    bs, hs, _, d = q.shape
    n_q, n_k = _blocks(c)
    counts, forced = _counts(c)
    fm = torch.tensor(_forced(c), device=DEV)
    stride = max(counts)
    num = torch.empty(bs, hs, n_q, dtype=torch.int32, device=DEV)
    idx = torch.zeros(bs, hs, n_q, stride, dtype=torch.int32, device=DEV)
    j = torch.arange(n_k, dtype=torch.int32, device=DEV)
    for bi in range(bs):
        for h in range(hs):
            s = _pooled(q[bi, h].to(dtype), c["block"]) @ _pooled(k[bi, h].to(dtype), c["block"]).t().contiguous()
            s[:, fm] = -math.inf
            take = fm.repeat(n_q, 1)
            if counts[h] > forced:
                take.scatter_(1, s.topk(counts[h] - forced, dim=1).indices, True)
            order = torch.where(take, j, n_k).sort(dim=1).values
            idx[bi, h, :, : counts[h]] = order[:, : counts[h]]
            num[bi, h] = counts[h]
    return num, idx


def _rows(c):
    n = c["rows"]
    return [((2 * r + 1) * c["lq"]) // (2 * n) for r in range(n)]


def _row_logits(c, q, k, bi, h, rows):
    return q[bi, h, rows].double() @ k[bi, h].double().t().contiguous() / math.sqrt(c["d"])


def prepare(c, seed):
    c = dict(c)
    op, lq, lk, d, b = c["op"], c["lq"], _lk(c), c["d"], c["block"]
    bs, hs = c["batch"], c["heads"]
    q, k, v = _inputs(c, seed, op not in ("select", "mass"))
    st = dict(case=c, q=q, k=k, v=v)
    n_q, _ = _blocks(c)
    if op in ("step", "noalloc", "select"):
        st["keep"] = S.sparstar_clip_keep_ranges(c["clip"], *_segments(c))
        st["budget"] = _budgets(c) if c["spread"] else c["rho"]
        st["stride"] = S.sparstar_kv_stride(hs, lk, b, st["budget"], st["keep"])
        # the lists' buffers, kept by the caller; entries past a row's count stay as they are
        st["num"] = torch.zeros(bs, hs, n_q, dtype=torch.int32, device=DEV)
        st["idx"] = torch.zeros(bs, hs, n_q, st["stride"], dtype=torch.int32, device=DEV)
        st["ws"] = torch.empty(S.sparstar_score_workspace_bytes(bs, hs, lq, lk, d, b), dtype=torch.uint8, device=DEV)
    if op == "sparse":
        st["num"], st["idx"] = _lists(c, q, k, torch.float32)
    if op in ("step", "noalloc", "sparse", "dense"):
        st["o"] = torch.empty_like(q)
        st["lse"] = torch.empty(bs, hs, lq, dtype=torch.float32, device=DEV)
        n = S.sparstar_attn_workspace_bytes(bs, hs, lq, lk, d, b) if c["split"] else 0
        st["aws"] = torch.empty(max(1, n), dtype=torch.uint8, device=DEV) if c["split"] else None
    if op == "mass":
        rows = _rows(c)
        lse = torch.empty(bs, hs, lq, dtype=torch.float32, device=DEV)
        lse.fill_(math.log(lk))
        counts, _ = _counts(c)
        for bi in range(bs):
            for h in range(hs):
                lse[bi, h, rows] = _row_logits(c, q, k, bi, h, rows).logsumexp(dim=1).float()
        n_tok = torch.tensor([min(lk, n * b) for n in counts], dtype=torch.int32, device=DEV)
        st["n_tok"] = n_tok.view(1, hs, 1).expand(bs, hs, len(rows)).contiguous()
        st["lse_all"], st["rows"] = lse, rows
        st["ws"] = torch.empty(S.sparstar_token_topk_workspace_bytes(bs, hs, lk, len(rows)), dtype=torch.uint8,
                               device=DEV)
    return st


def _select(st, scorer):
    c = st["case"]
    if scorer == "static":
        return S.sparstar_score_blocks_static(st["q"], st["k"], c["block"], st["budget"], st["keep"],
                                              kv_stride=st["stride"], out=(st["num"], st["idx"]))
    return S.sparstar_score_blocks(st["q"], st["k"], c["block"], st["budget"], st["keep"], kv_stride=st["stride"],
                                   workspace=st["ws"], out=(st["num"], st["idx"]), fused=scorer == "fused")


def _sparse(st):
    c = st["case"]
    return S.sparstar_sparse_attn_fwd(st["q"], st["k"], st["v"], st["num"], st["idx"], c["block"], out=st["o"],
                                      lse=st["lse"], split=c["split"], workspace=st["aws"])


def run(st):
    c = st["case"]
    op = c["op"]
    if op == "select":
        return _select(st, c["scorer"])
    if op == "sparse":
        return _sparse(st)
    if op in ("step", "noalloc"):
        num, idx = _select(st, "static" if op == "noalloc" else "separate")
        o, lse = _sparse(st)
        return num, idx, o, lse
    if op == "dense":
        return S.sparstar_dense_attn_fwd(st["q"], st["k"], st["v"], c["block"], out=st["o"], lse=st["lse"],
                                         split=c["split"], workspace=st["aws"])
    return S.sparstar_token_topk_mass(st["q"], st["k"], st["rows"], st["n_tok"], st["lse_all"], workspace=st["ws"])


def tolerance(c):
    if c["op"] == "mass":
        # 32-bit dot products and sums; measured 6e-8 against 64 bits
        return {"rel": 1e-6, "max": 1e-5}
    # scores within fp32 rounding of each other may trade places at a row's
    # boundary, which shifts the rest of that row's ascending list: the fused
    # and the separate scorer, and 64-bit scores, differ in up to 4.1e-5 of the
    # list entries at 720p (four times that, with room for small cases)
    if c["op"] == "select":
        return {"rel": 0.0, "differ": 1e-3}
    # P is rounded to bf16 relative to a running maximum, O to bf16: the split
    # and the single pass differ by rel 3.1e-3 and max 0.036
    return {"rel": 1.2e-2, "max": 0.15, "differ": 1e-3}


# --------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# --------------------------------------------------------------------------
def _attend(q, k, v, mask=None):
    """O and log-sum-exp of q [n, r, d] over k, v [n, m, d] in float64."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if mask is not None:
        s.masked_fill_(mask[:, None, :], -math.inf)
    lse = s.logsumexp(dim=2)
    s.sub_(lse[:, :, None]).exp_()
    return torch.matmul(s, v), lse


def _exact_sparse(c, q, k, v, num, idx):
    bs, hs, lq, d = q.shape
    lk, b = k.shape[2], c["block"]
    n_q, n_k = _blocks(c)
    counts, _ = _counts(c)
    o = torch.empty(bs, hs, lq, d, dtype=torch.float64, device=DEV)
    lse = torch.empty(bs, hs, lq, dtype=torch.float64, device=DEV)
    for bi in range(bs):
        for h in range(hs):
            qd = torch.zeros(n_q * b, d, dtype=torch.float64, device=DEV)
            qd[:lq] = q[bi, h].double()
            qd = qd.view(n_q, b, d)
            kd = torch.zeros(n_k * b, d, dtype=torch.float64, device=DEV)
            vd = torch.zeros_like(kd)
            kd[:lk], vd[:lk] = k[bi, h].double(), v[bi, h].double()
            n = counts[h]
            step = max(1, (1 << 20) // (n * b))
            oh = torch.empty(n_q, b, d, dtype=torch.float64, device=DEV)
            lh = torch.empty(n_q, b, dtype=torch.float64, device=DEV)
            for i in range(0, n_q, step):
                blk = idx[bi, h, i: i + step, :n].long()
                tok = (blk[:, :, None] * b + torch.arange(b, device=DEV)).view(blk.shape[0], n * b)
                oh[i: i + step], lh[i: i + step] = _attend(qd[i: i + step], kd[tok], vd[tok],
                                                           tok >= lk if lk % b else None)
            o[bi, h], lse[bi, h] = oh.view(-1, d)[:lq], lh.view(-1)[:lq]
    return o, lse


def _exact_dense(c, q, k, v):
    bs, hs, lq, d = q.shape
    o = torch.empty(bs, hs, lq, d, dtype=torch.float64, device=DEV)
    lse = torch.empty(bs, hs, lq, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // k.shape[2])
    for bi in range(bs):
        for h in range(hs):
            kd, vd = k[bi, h].double()[None], v[bi, h].double()[None]
            for i in range(0, lq, step):
                r, l = _attend(q[bi, h, i: i + step].double()[None], kd, vd)
                o[bi, h, i: i + step], lse[bi, h, i: i + step] = r[0], l[0]
    return o, lse


def exact(c, seed):
    op = c["op"]
    if op == "select":
        return None  # whole numbers
    q, k, v = _inputs(c, seed, op != "mass")
    if op == "dense":
        return _exact_dense(c, q, k, v)
    if op == "sparse":
        return _exact_sparse(c, q, k, v, *_lists(c, q, k, torch.float32))
    if op in ("step", "noalloc"):
        return (None, None) + _exact_sparse(c, q, k, v, *_lists(c, q, k, torch.float64))
    rows = _rows(c)
    counts, _ = _counts(c)
    out = torch.empty(c["batch"], c["heads"], len(rows), dtype=torch.float64, device=DEV)
    for bi in range(c["batch"]):
        for h in range(c["heads"]):
            z = _row_logits(c, q, k, bi, h, rows)
            w = (z - z.logsumexp(dim=1).float().double()[:, None]).exp()
            out[bi, h] = w.topk(min(_lk(c), counts[h] * c["block"]), dim=1).values.sum(dim=1)
    return out
