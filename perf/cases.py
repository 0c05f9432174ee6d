"""The work a user of this library has it do, as timed cases.

A case is one attention layer of one sequence, prefill, through the public
entry points of paper_2509_24745_amd.proxyattn:

  prefill   the whole path (estimate, select_budget, block_sparse_prefill)
  estimate  block scores and last-block masses alone
  select    budgets and block lists alone
  sparse    block-sparse attention over a caller's lists (K/V copy included)
  dense     the dense causal baseline (K/V copy included)

Inputs follow the recipe of paper_2509_24745_amd/synth.py (a smooth shared
latent per KV head, per-head deviations, a sink, hot blocks, per-head
temperatures), drawn on the GPU.
"""
from __future__ import annotations

import math

import torch

from paper_2509_24745_amd import proxyattn as pa

DEV = "cuda"


def _case(name, kind, n, hq, hkv, d, b, g, s=4, dtype="bf16", gamma=0.95, beta=0, hetero=False,
          layout="thd"):
    return {"name": name, "kind": kind, "n": n, "hq": hq, "hkv": hkv, "d": d, "b": b, "g": g,
            "s": s, "dtype": dtype, "gamma": gamma, "beta": beta, "hetero": hetero,
            "layout": layout}


def listed():
    return [
        # the small fp32 GQA layer (workload gqa8x2_n2048_fp32): launches and
        # latency, fp32 products
        _case("prefill_fp32_2k", "prefill", 2048, 8, 2, 64, 64, 2, dtype="fp32", gamma=0.9),
        # a short prompt of odd length through the Llama-shaped layer
        _case("prefill_4k_ragged", "prefill", 4173, 32, 8, 128, 128, 4),
        # an ordinary long prompt, same layer
        _case("prefill_16k", "prefill", 16384, 32, 8, 128, 128, 4),
        # the layer the benchmark times: 128K tokens
        _case("prefill_128k", "prefill", 131072, 32, 8, 128, 128, 4),
        # the Qwen-shaped layer with heterogeneous heads, groups across KV
        # heads and a minimum budget
        _case("prefill_qwen_64k", "prefill", 65536, 28, 4, 128, 128, 7, beta=2048, hetero=True),
        # block scoring and masses alone at the benchmark's size
        _case("estimate_128k", "estimate", 131072, 32, 8, 128, 128, 4),
        # finer estimation: stride 2, one proxy head per KV head, odd length
        _case("estimate_s2_50k", "estimate", 50001, 32, 8, 128, 128, 8, s=2),
        # budgets and lists at the benchmark's size (lists as long as 1024 blocks)
        _case("select_128k", "select", 131072, 32, 8, 128, 128, 4),
        # attention of a head-dim 64 layer with fine blocks, odd length
        _case("sparse_d64_b64", "sparse", 20011, 32, 8, 64, 64, 8),
        # fine blocks at head dim 128, Q/K/V/O stored head-major
        _case("sparse_b64_hm", "sparse", 12345, 32, 8, 128, 64, 4, layout="htd"),
        # fp32 attention of a full-width layer
        _case("sparse_fp32_8k", "sparse", 8192, 32, 8, 128, 128, 4, dtype="fp32"),
        # the dense baseline of the same layer
        _case("dense_32k", "dense", 32768, 32, 8, 128, 128, 4),
    ]


# Kinds drawn, with their range of lengths (bf16; fp32 lengths end at 12288).
_RANGES = {"prefill": (300, 100000), "estimate": (2000, 131072), "select": (2000, 131072),
           "sparse": (1000, 65536), "dense": (300, 49152)}


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "estimate", "select", "sparse", "sparse",
                       "dense"])
    dtype = "fp32" if rng.random() < 0.25 else "bf16"
    lo, hi = _RANGES[kind]
    if dtype == "fp32":
        hi = 12288
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        n = max(256, n // 256 * 256)
    hq, hkv, groups = rng.choice([(32, 8, (1, 2, 4, 8)), (28, 4, (1, 2, 4, 7)), (16, 4, (1, 4)),
                                  (8, 2, (2, 8)), (8, 8, (4,))])
    d = rng.choice([64, 128, 128])
    b = rng.choice([64, 128, 128])
    s = rng.choice([1, 2, 4, 4, 4])
    return {"kind": kind, "n": n, "hq": hq, "hkv": hkv, "d": d, "b": b, "g": rng.choice(groups),
            "s": s, "dtype": dtype, "gamma": rng.choice([0.9, 0.95, 0.95, 0.99]),
            "beta": rng.choice([0, 0, 1024]), "hetero": rng.random() < 0.25,
            "layout": "htd" if rng.random() < 0.25 else "thd"}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_RANK, _CORR, _NOISE, _IID = 16, 1024.0, 0.3, 0.1
_CONTENT, _SINK, _HOT_BLOCKS, _HOT, _SPREAD = 3.1, 6.0, 4, 4.0, 1.5


def _ar1(gen, procs, n):
    """Unit-variance Gaussian AR(1) processes [procs, n, rank] along the tokens."""
    c = 256
    ch = -(-n // c)
    rho = math.exp(-1.0 / _CORR)
    xi = torch.randn((procs, ch, c, _RANK), generator=gen, device=DEV)
    i = torch.arange(c, device=DEV, dtype=torch.float32)
    lag = i[:, None] - i[None, :]
    t = torch.where(lag >= 0, rho ** lag.clamp(min=0), 0.0) * math.sqrt(1 - rho * rho)
    z = torch.matmul(t, xi)
    # each chunk starts from what the chunks before it left
    j = torch.arange(ch, device=DEV, dtype=torch.float32)
    lag = j[:, None] - 1 - j[None, :]
    carry = torch.where(lag >= 0, rho ** (c * lag.clamp(min=0)), 0.0)
    first = rho ** (c * j)
    start = torch.randn((procs, 1, _RANK), generator=gen, device=DEV)
    prev = torch.matmul(carry, z[:, :, -1, :].contiguous()) + first[:, None] * start
    z += (rho ** (i + 1))[None, None, :, None] * prev[:, :, None, :]
    return z.reshape(procs, ch * c, _RANK)[:, :n].contiguous()


def _qkv(case, seed):
    n, hq, hkv, d, b = (case[x] for x in ("n", "hq", "hkv", "d", "b"))
    r = hq // hkv
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 17)

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device=DEV)

    def unit(x):
        return x / x.norm(dim=-1, keepdim=True)

    e = unit(rnd(hkv, 1, d))
    f = rnd(hkv, 1, d)
    f = unit(f - (f * e).sum(-1, keepdim=True) * e)

    def proj(x, h):  # rows of x without their parts along e_h and f_h
        x = x - (x * e[h]).sum(-1, keepdim=True) * e[h]
        return x - (x * f[h]).sum(-1, keepdim=True) * f[h]

    def basis(h):
        return proj(rnd(_RANK, d) / math.sqrt(_RANK), h)

    if case["hetero"]:
        temps = [0.1 if i % 2 == 0 else 2.0 for i in range(hq)]
    else:
        u = torch.rand(hq, generator=gen, device=DEV).tolist()
        temps = [_SPREAD ** (2 * x - 1) for x in u]
    scale = _CONTENT * math.sqrt(_RANK / d)
    nk = -(-n // b)
    head_major = case["layout"] == "htd"
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def empty(heads):
        x = torch.empty((heads, n, d) if head_major else (n, heads, d), dtype=td, device=DEV)
        return x, (x if head_major else x.transpose(0, 1))

    (q, qh), (k, kh), (v, vh) = empty(hq), empty(hkv), empty(hkv)
    norm = math.sqrt(1 + _NOISE ** 2)
    for h in range(hkv):
        z = _ar1(gen, 2 + r, n)
        x = z[0] @ basis(h)
        key = (x + _NOISE * (z[1] @ basis(h))) / norm + _IID * proj(rnd(n, d), h)
        key[0] += math.sqrt(d) * e[h, 0]
        hot = 0
        if nk > 1:
            hot = min(_HOT_BLOCKS, nk - 1)
            for blk in (1 + torch.randperm(nk - 1, generator=gen, device=DEV)[:hot]).tolist():
                key[blk * b:(blk + 1) * b] += math.sqrt(d) * f[h, 0]
        kh[h].copy_(key)
        vh[h].copy_(rnd(n, d))
        for j in range(r):
            i = h * r + j
            t = temps[i]
            gain = 3.0 if case["hetero"] and i % 2 == 1 else 1.0
            qi = (x + _NOISE * (z[2 + j] @ basis(h))) * (scale * t / norm)
            qi += (_IID * scale * t) * proj(rnd(n, d), h) + (t * gain * _SINK) * e[h]
            if hot:
                qi += (t * _HOT) * f[h]
            qh[i].copy_(qi)
    return q, k, v


def _problem(case):
    n, hq, hkv, d = (case[x] for x in ("n", "hq", "hkv", "d"))
    strides = {}
    if case["layout"] == "htd":
        strides = dict(q_tok_stride=d, q_head_stride=n * d, kv_tok_stride=d,
                       kv_head_stride=n * d)
        if case["kind"] != "prefill":  # whose output buffer is token-major
            strides.update(o_tok_stride=d, o_head_stride=n * d)
    return pa.Problem(seq_len=n, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                      block_size=case["b"], num_proxy_groups=case["g"], stride=case["s"],
                      dtype=case["dtype"], **strides)


# Mean share of the causal blocks that lists of this library keep at each
# threshold (a length of 8K to 128K, the recipe above).
_KEEP = {0.9: 0.2, 0.95: 0.3, 0.99: 0.55}


def _scores(case, gen):
    """Block log-scores [G][Mq][Nk] as the estimation gives them: a recent
    band, a sink block, and rows that change slowly down the sequence."""
    g, mq = case["g"], -(-case["n"] // case["b"])
    fine = torch.randn((g, mq, mq), generator=gen, device=DEV)
    rows = -(-mq // 16)
    slow = torch.randn((g, rows, mq), generator=gen, device=DEV).repeat_interleave(16, dim=1)
    m = torch.arange(mq, device=DEV)
    gap = (m[:, None] - m[None, :]).float()
    a = 2.0 * slow[:, :mq] + 0.5 * fine - 1.5 * torch.log1p(gap.clamp(min=0)) - 2.0
    a[:, :, 0] += 4.0
    a = torch.where(gap >= 0, a, float("-inf"))
    return a.contiguous()


def _budgets(case):
    """One budget per head, spread as the dynamic budgets are: log-spaced
    over a factor of 16, their mean share of a row as _KEEP says."""
    hq, mq = case["hq"], -(-case["n"] // case["b"])
    order = [(7 * i + 3) % hq for i in range(hq)] if hq % 7 else list(range(hq))
    w = [16.0 ** (o / max(1, hq - 1)) for o in order]
    target = mq * (1 - math.sqrt(1 - min(0.95, _KEEP[case["gamma"]])))
    return [max(1, min(mq, round(target * x * hq / sum(w)))) for x in w]


def _kept_blocks(case):
    mq = -(-case["n"] // case["b"])
    return sum(c * (c + 1) // 2 + (mq - c) * c for c in _budgets(case))


def _lists(case, gen):
    """A caller's lists: per head the highest scores of each row, in rank order."""
    hq, mq = case["hq"], -(-case["n"] // case["b"])
    order = torch.argsort(_scores(case, gen), dim=2, descending=True, stable=True).int()
    counts = torch.tensor(_budgets(case), dtype=torch.int32, device=DEV)
    rows = torch.arange(1, mq + 1, dtype=torch.int32, device=DEV)
    bc = torch.minimum(counts[:, None], rows[None, :]).contiguous()
    idx = order.repeat_interleave(hq // case["g"], dim=0)
    pos = torch.arange(mq, dtype=torch.int32, device=DEV)
    bi = torch.where(pos[None, None, :] < bc[:, :, None], idx, -1).contiguous()
    return bc, bi


def _mass(case, gen):
    """Last-block masses [Hq][Nk]: heavy-tailed rows that sum to min(b, N)."""
    hq, n, b = case["hq"], case["n"], case["b"]
    mq = -(-n // b)
    z = torch.randn((hq, mq), generator=gen, device=DEV)
    width = torch.linspace(1.0, 3.0, hq, device=DEV)[:, None]
    return (torch.softmax(z * width, dim=1) * min(b, n)).contiguous()


def prepare(case, seed):
    prob = _problem(case)
    kind = case["kind"]
    n, hq, d = case["n"], case["hq"], case["d"]
    mq = prob.num_blocks
    st = {"case": case, "prob": prob}
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 104729 + 5)

    def ints(*shape):
        return torch.empty(shape, dtype=torch.int32, device=DEV)

    if kind in ("prefill", "estimate", "sparse", "dense"):
        st["q"], st["k"], st["v"] = _qkv(case, seed)
    if kind == "select":
        st["logscore"], st["mass"] = _scores(case, gen), _mass(case, gen)
        st["head_count"], st["block_count"] = ints(hq), ints(hq, mq)
        st["block_index"] = ints(hq, mq, mq)
        return st
    if kind == "estimate":
        st["logscore"] = torch.empty((case["g"], mq, mq), dtype=torch.float32, device=DEV)
        st["mass"] = torch.empty((hq, mq), dtype=torch.float32, device=DEV)
        st["workspace"] = torch.empty(pa.proxyattn_workspace_size(prob), dtype=torch.uint8,
                                      device=DEV)
        return st
    if kind == "prefill":
        st["bufs"] = pa.Buffers(prob, DEV)
        return st
    st["out"] = torch.empty((hq, n, d) if case["layout"] == "htd" else (n, hq, d),
                            dtype=prob.torch_dtype, device=DEV)
    st["lse"] = torch.empty((hq, n), dtype=torch.float32, device=DEV)
    st["workspace"] = torch.empty(pa.proxyattn_workspace_size(prob), dtype=torch.uint8, device=DEV)
    if kind == "sparse":
        st["block_count"], st["block_index"] = _lists(case, gen)
    return st


def run(st):
    case, prob = st["case"], st["prob"]
    kind = case["kind"]
    if kind == "prefill":
        b = pa.prefill(prob, st["q"], st["k"], st["v"], case["gamma"], case["beta"], st["bufs"])
        return {"out": b.out, "lse": b.lse, "logscore": b.logscore, "mass": b.mass,
                "head_count": b.head_count, "block_count": b.block_count,
                "block_index": b.block_index}
    if kind == "estimate":
        pa.proxyattn_estimate(prob, st["q"], st["k"], st["logscore"], st["mass"], st["workspace"])
        return {"logscore": st["logscore"], "mass": st["mass"]}
    if kind == "select":
        pa.proxyattn_select_budget(prob, st["logscore"], st["mass"], case["gamma"], case["beta"],
                                   st["head_count"], st["block_count"], st["block_index"])
        return {"head_count": st["head_count"], "block_count": st["block_count"],
                "block_index": st["block_index"]}
    if kind == "sparse":
        pa.proxyattn_block_sparse_prefill(prob, st["q"], st["k"], st["v"], st["block_count"],
                                          st["block_index"], st["out"], st["lse"],
                                          st["workspace"])
    else:
        pa.proxyattn_dense_prefill(prob, st["q"], st["k"], st["v"], st["out"], st["lse"],
                                   st["workspace"])
    return {"out": st["out"], "lse": st["lse"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    n, hq, hkv, d, b, g, s = (case[x] for x in ("n", "hq", "hkv", "d", "b", "g", "s"))
    e = 2 if case["dtype"] == "bf16" else 4
    mq, np_ = -(-n // b), -(-n // s)
    kind = case["kind"]
    q, kv, o = n * hq * d * e, n * hkv * d * e, n * hq * d * e + 4 * hq * n
    scores, mass, lists = 4 * g * mq * mq, 4 * hq * mq, 4 * hq * mq * (mq + 1) + 4 * hq
    # strided rows of Q; the masses read every key, the last block's queries
    est_bytes = np_ * hq * d * e + min(b, n) * hq * d * e + kv + scores + mass
    est_flops = 2 * d * g * (np_ * (np_ + 1) // 2) + 2 * d * hq * min(b, n) * n
    causal = mq * (mq + 1) // 2
    kept = hq * causal * _KEEP[case["gamma"]]
    if kind == "prefill":
        return {"bytes": q + 2 * kv + o + scores + mass + lists,
                "flops": est_flops + 4 * b * b * d * kept}
    if kind == "estimate":
        return {"bytes": est_bytes, "flops": est_flops}
    if kind == "select":
        return {"bytes": scores // 2 + mass + lists, "flops": hq * mq + g * causal}
    if kind == "sparse":
        return {"bytes": q + 2 * kv + o + 4 * _kept_blocks(case),
                "flops": 4 * b * b * d * _kept_blocks(case)}
    return {"bytes": q + 2 * kv + o, "flops": 4 * d * hq * (n * (n + 1) // 2)}


def tolerance(case):
    # measured against exact(): scores and masses 2e-7, fp32 attention 1.6e-6,
    # bf16 attention 2e-3 (bf16 probabilities and outputs)
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "estimate":
        return {"rel": 2e-6, "max": 1e-4}
    fp32 = case["dtype"] == "fp32"
    if case["kind"] == "prefill":
        # scores rounded another way swap a near tie here and there: a list
        # entry in ten thousand, and the rows that attend to another block
        return {"rel": 1e-3 if fp32 else 1e-2, "max": 0.5, "differ": 2e-3}
    return {"rel": 7e-6, "max": 1e-3} if fp32 else {"rel": 1e-2, "max": 0.5}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _heads(x, case):
    return x if case["layout"] == "htd" else x.transpose(0, 1)


def _exact_estimate(case, q, k):
    n, hq, hkv, d, b, g, s = (case[x] for x in ("n", "hq", "hkv", "d", "b", "g", "s"))
    r, gs, mq, np_, bp = hq // hkv, hq // g, -(-n // b), -(-n // s), b // s
    c = 1.0 / math.sqrt(d)
    qh, kh = _heads(q, case), _heads(k, case)
    logscore = torch.full((g, mq, mq), float("-inf"), dtype=torch.float64, device=DEV)
    pad = mq * bp - np_
    for j in range(g):
        # the pooled heads are defined as fp32 sums rounded to the input's type
        aq = torch.zeros((np_, d), dtype=torch.float32, device=DEV)
        ak = torch.zeros_like(aq)
        for i in range(j * gs, (j + 1) * gs):
            aq += qh[i, ::s].float()
            ak += kh[i // r, ::s].float()
        inv = torch.tensor(1.0 / gs, dtype=torch.float32, device=DEV)
        qg, kg = (aq * inv).to(q.dtype).double(), (ak * inv).to(q.dtype).double()
        rows = max(1, min(mq, (1 << 28) // max(1, np_ * bp)))
        for m0 in range(0, mq, rows):
            m1 = min(m0 + rows, mq)
            t0, t1 = m0 * bp, min(m1 * bp, np_)
            x = c * (qg[t0:t1] @ kg[:t1].t())
            t = torch.arange(t0, t1, device=DEV)
            x.masked_fill_(torch.arange(t1, device=DEV)[None, :] > t[:, None], float("-inf"))
            x -= torch.logsumexp(x, dim=1, keepdim=True)
            up = (m1 * bp - t1)
            x = torch.nn.functional.pad(x, (0, up, 0, up), value=float("-inf"))
            x = x.reshape(m1 - m0, bp, m1, bp).amax(dim=3).amax(dim=1)
            logscore[j, m0:m1, :m1] = x
    rows = min(b, n)
    mass = torch.zeros((hq, mq), dtype=torch.float64, device=DEV)
    t = torch.arange(n - rows, n, device=DEV)
    u = torch.arange(n, device=DEV)
    for i in range(hq):
        x = c * (qh[i, n - rows:].double() @ kh[i // r].double().t())
        x.masked_fill_(u[None, :] > t[:, None], float("-inf"))
        p = torch.softmax(x, dim=1).sum(dim=0)
        mass[i] = torch.nn.functional.pad(p, (0, mq * b - n)).reshape(mq, b).sum(dim=1)
    return logscore, mass


def _exact_select(case, logscore, mass):
    hq, b = case["hq"], case["b"]
    mq = mass.shape[1]
    share = torch.sort(mass / mass.sum(dim=1, keepdim=True), dim=1, descending=True).values
    reach = share.cumsum(dim=1) >= case["gamma"]
    count = torch.where(reach.any(dim=1), reach.int().argmax(dim=1) + 1, mq)
    if case["gamma"] >= 1:
        count = torch.full_like(count, mq)
    count = count.clamp(min=-(-case["beta"] // b), max=mq)
    rank = torch.argsort(torch.argsort(logscore, dim=2, descending=True, stable=True), dim=2)
    return count, rank


def _exact_attention(case, q, k, v, keep):
    """keep(i): [Mq][Nk] bool of head i's blocks, or None for all."""
    n, hq, hkv, d, b = (case[x] for x in ("n", "hq", "hkv", "d", "b"))
    r, c = hq // hkv, 1.0 / math.sqrt(d)
    qh, kh, vh = (_heads(x, case) for x in (q, k, v))
    out = torch.empty((hq, n, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((hq, n), dtype=torch.float64, device=DEV)
    step = max(b, (1 << 28) // n // b * b)
    u = torch.arange(n, device=DEV)
    for i in range(hq):
        kk, vv = kh[i // r].double(), vh[i // r].double()
        blocks = keep(i)
        for t0 in range(0, n, step):
            t1 = min(t0 + step, n)
            x = c * (qh[i, t0:t1].double() @ kk[:t1].t())
            t = torch.arange(t0, t1, device=DEV)
            drop = u[None, :t1] > t[:, None]
            if blocks is not None:
                drop |= ~blocks[t // b][:, u[:t1] // b]
            x.masked_fill_(drop, float("-inf"))
            z = torch.logsumexp(x, dim=1, keepdim=True)
            out[i, t0:t1] = torch.exp(x - z) @ vv[:t1]
            lse[i, t0:t1] = z[:, 0]
    if case["layout"] == "thd" or case["kind"] == "prefill":
        out = out.transpose(0, 1).contiguous()
    return out, lse


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        return None
    if kind != "estimate" and case["hq"] * case["n"] ** 2 > 32 * 70000 ** 2:
        return None
    st = prepare(case, seed)
    if kind == "estimate":
        a, mass = _exact_estimate(case, st["q"], st["k"])
        return {"logscore": a, "mass": mass}
    if kind == "dense":
        o, lse = _exact_attention(case, st["q"], st["k"], st["v"], lambda i: None)
        return {"out": o, "lse": lse}
    mq = st["prob"].num_blocks
    pos = torch.arange(mq, device=DEV)
    if kind == "sparse":
        bc, bi = st["block_count"], st["block_index"]

        def keep(i):
            on = torch.zeros((mq, mq + 1), dtype=torch.bool, device=DEV)
            on.scatter_(1, torch.where(bi[i] < 0, mq, bi[i]).long(), True)
            return on[:, :mq]

        o, lse = _exact_attention(case, st["q"], st["k"], st["v"], keep)
        return {"out": o, "lse": lse}
    a, mass = _exact_estimate(case, st["q"], st["k"])
    count, rank = _exact_select(case, a, mass)
    gs = case["hq"] // case["g"]

    def kept(i):
        return (rank[i // gs] < count[i]) & (pos[None, :] <= pos[:, None])

    o, lse = _exact_attention(case, st["q"], st["k"], st["v"], kept)
    return {"out": o, "lse": lse, "logscore": a, "mass": mass, "head_count": None,
            "block_count": None, "block_index": None}
