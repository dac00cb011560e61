"""Timed cases of the public entry points, over the range a serving program uses.

A case names a batch (how many requests, how long, which block length and head
shape) and the call that works on it: one fused denoising step, the block
attention of one layer, the output head with its decode, the dual-cache refresh
of one layer, or a block boundary (KV copy, then the step). The request
lengths and the number of masked positions belong to the case; which box row a
request takes, where its masked positions lie and every tensor value come from
the seed. Head shapes are those of LLaDA-8B (32 heads, D = 128) and Dream-7B
(28 query / 4 KV heads, D = 128), or small generic ones.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2607_08930_amd as bs
from paper_2607_08930_amd import step as bstep

LLADA = dict(Hq=32, Hkv=32, D=128, V=126464, d=4096, base=500000.0)
DREAM = dict(Hq=28, Hkv=4, D=128, V=152064, d=3584, base=1000000.0)


def _case(name, kind, shape, n, p, g, L=32, dtype="bf16", mix="uniform", layers=1, batch=0):
    c = dict(kind=kind, n=n, p_lo=p[0], p_hi=p[1], g=g, L=L, dtype=dtype, mix=mix, layers=layers, batch=batch, **shape)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one user's request, the latency of a single denoising step
        _case("step-llada-n1", "step", LLADA, 1, (64, 512), 256),
        # an ordinary MHA batch: the repository's headline step
        _case("step-llada-n32", "step", LLADA, 32, (64, 512), 256),
        # an ordinary GQA batch
        _case("step-dream-n64", "step", DREAM, 64, (128, 1024), 512),
        # a batch admitted under a token budget: mostly short prompts, a fifth long
        _case("step-dream-skewed-n189", "step", DREAM, 189, (32, 2048), 0, mix="skewed"),
        # a few requests in full precision, as a numerics check of a model runs them
        _case("step-llada-fp32-n8", "step", LLADA, 8, (64, 512), 256, dtype="f32"),
        # the longest block length the method's ablation uses
        _case("attention-llada-L64-n32", "attention", LLADA, 32, (64, 512), 256, L=64),
        # one very long prompt among ordinary ones (split rows)
        _case("attention-dream-straggler-n24", "attention", DREAM, 24, (128, 1024), 512, mix="straggler"),
        # output head of a small serving batch: the head matrix is what is read
        _case("head-llada-n8", "head", LLADA, 8, (64, 512), 256),
        # output head of an ordinary GQA batch: the matrix product is what counts
        _case("head-dream-n64", "head", DREAM, 64, (128, 1024), 512),
        # cache refresh / prefill at a block start, MHA and GQA
        _case("refresh-llada-n32", "refresh", LLADA, 32, (64, 512), 256),
        _case("refresh-dream-n64", "refresh", DREAM, 64, (128, 1024), 512),
        # a block boundary: a quarter of the rows is replaced by staged requests,
        # then a step through several layers
        _case("boundary-llada-n64-8layers", "boundary", LLADA, 64, (32, 256), 128, layers=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    shape = dict(rng.choice((LLADA, DREAM)))
    kind = rng.choice(("step", "step", "step", "attention", "attention", "head", "refresh", "boundary"))
    dtype, mix, layers = "bf16", "uniform", 1
    L = rng.choice((8, 16, 24, 32, 32, 32, 48, 64))
    g = rng.choice((128, 256, 512, rng.randint(1, 512)))
    p_hi = _log(rng, 16, 2048)
    p_lo = rng.randint(0, p_hi)
    # rows of the box that the drawn lengths fill with at most 32768 tokens
    n = _log(rng, 1, max(1, min(192, 32768 // (p_hi + g))))
    if kind in ("step", "attention"):
        mix = rng.choice(("uniform", "uniform", "skewed", "straggler")) if n >= 4 else "uniform"
        if mix == "straggler":
            n = min(n, 48)
        if rng.random() < 0.15:   # other head shapes the bf16 kernels serve
            Hkv = rng.choice((1, 2, 4, 8))
            shape.update(Hq=Hkv * rng.randint(1, 8), Hkv=Hkv, D=rng.choice((64, 128)), V=rng.randint(1000, 65536))
        if kind == "step":
            layers = rng.choice((1, 1, 2, 4))
            if rng.random() < 0.2:
                dtype, layers, n, mix = "f32", 1, min(n, 8), "uniform"
    elif kind == "boundary":
        layers = rng.randint(1, 8)
        n = max(4, min(n, 64))
        p_hi = min(p_hi, 512)
        p_lo = min(p_lo, p_hi)
    elif kind == "head":
        n = min(n, 64)
        L = min(L, 32)
    elif kind == "refresh":
        n = max(1, min(n, 32768 // (p_hi + g)))
    return _case(None, kind, shape, n, (p_lo, p_hi), g, L=L, dtype=dtype, mix=mix, layers=layers, batch=rng.randint(1, 1 << 20))


# ---------------------------------------------------------------- geometry of a case
def _lengths(c):
    """(p, g, k, masked positions) of each request: the case's own, not the seed's."""
    rng = random.Random("%s %d %d %d %d %d" % (c["mix"], c["n"], c["p_lo"], c["p_hi"], c["g"], c["batch"]))
    rows = []
    for i in range(c["n"]):
        p, g = rng.randint(c["p_lo"], c["p_hi"]), c["g"]
        if c["mix"] == "skewed":
            p = rng.randint(1024, 2048) if rng.random() < 0.2 else rng.randint(32, 128)
            g = rng.choice((128, 256, 512))
        elif c["mix"] == "straggler" and i == 0:
            p = 8000
        k = rng.randrange(-(-g // c["L"])) if c["kind"] != "boundary" else rng.randrange(max(1, g // c["L"] - 1))
        B = min(c["L"], g - k * c["L"])
        m = max(1, sum(rng.random() < 0.5 for _ in range(B)))
        rows.append((p, g, k, B, m))
    return rows


def _geometry(c, seed):
    """Descriptors (right-aligned rows), their block lengths and masked positions for this seed."""
    rng = random.Random("%d %s" % (seed, sorted((k, v) for k, v in c.items() if k != "name")))
    rows = _lengths(c)
    rng.shuffle(rows)
    n = len(rows)
    W = max(p + g for p, g, *_ in rows)
    place = list(range(n))
    rng.shuffle(place)
    reqs = np.zeros(n, bs.REQ_DTYPE)
    masked = np.zeros((n, c["L"]), np.uint8)
    for i, (p, g, k, B, m) in enumerate(rows):
        reqs[i] = (p, g, k, place[i], W - p - g)
        masked[i, rng.sample(range(B), m)] = 1
    return reqs, n, W, masked


_contexts = {}


def _context():
    """One library context per process, as a serving program keeps it."""
    if "ctx" not in _contexts:
        _contexts["ctx"] = bs.Context(0)
    return _contexts["ctx"]


def _tensors(c, seed):
    """Everything a call reads, on the GPU, from the seed (also what exact() starts from)."""
    reqs, n, W, masked = _geometry(c, seed)
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 17)
    td = bstep.torch_dtype(c["dtype"])
    L, Hq, Hkv, D, V = c["L"], c["Hq"], c["Hkv"], c["D"], c["V"]

    def normal(shape, sigma=1.0):
        x = torch.empty(shape, dtype=td, device=dev).normal_(generator=gen)
        return x if sigma == 1.0 else x.mul_(sigma)

    def ids(shape):
        return torch.randint(1, V, shape, device=dev, dtype=torch.int32, generator=gen)

    kv = 1.0 / math.sqrt(D)
    t = dict(reqs=reqs, n=n, W=W, masked=torch.from_numpy(masked).to(dev))
    if c["kind"] == "refresh":
        t.update(q=normal((n, W, Hq, D)), k=normal((n, W, Hkv, D), kv), v=normal((n, W, Hkv, D), kv))
        return t
    if c["kind"] in ("step", "attention", "boundary"):
        t["layers"] = []
        t["k_box"] = normal((c["layers"], n, Hkv, W, D), kv)
        t["v_box"] = normal((c["layers"], n, Hkv, W, D), kv)
        for l in range(c["layers"]):
            t["layers"].append(dict(q=normal((n, L, Hq, D)), k_new=normal((n, L, Hkv, D), kv),
                                    v_new=normal((n, L, Hkv, D), kv), k_cache=t["k_box"][l], v_cache=t["v_box"][l]))
        if c["kind"] == "boundary":
            # a quarter of the requests was prefilled into a staging box, left-aligned
            a = max(1, n // 4)
            segs = np.zeros(a, bs.SEG_DTYPE)
            for i in range(a):
                r = reqs[i]
                segs[i] = (1, i, 0, r["row"], r["off"], r["p"] + r["g"])
            t.update(segs=segs, k_stage=normal((c["layers"], a, Hkv, W, D), kv),
                     v_stage=normal((c["layers"], a, Hkv, W, D), kv))
    if c["kind"] in ("step", "boundary"):
        # logits of a confident model: one id stands out by a margin that puts
        # the confidences around the threshold
        x = normal((n, L, (V + 7) // 8 * 8))
        top = math.log(V) + 0.5 + 8.0 * torch.rand((n, L, 1), device=dev, generator=gen)
        x.scatter_(2, ids((n, L, 1)).long(), top.to(td))
        t["logits"] = x
        tokens = ids((n, W))
        box = torch.zeros((n, W), dtype=torch.uint8, device=dev)
        for i, r in enumerate(reqs):
            s = int(r["off"] + r["p"] + r["k"] * L)
            B = min(L, int(r["g"] - r["k"] * L))
            box[int(r["row"]), s + B:] = 1
            box[int(r["row"]), s:s + B] = t["masked"][i, :B]
        t.update(tokens=tokens, mask=box)
    if c["kind"] == "head":
        d = c["d"]
        w = normal((V, d), 1.0 / math.sqrt(d))
        h = normal((n * L, d)).float()
        pick = ids((n * L,)).long()
        m = math.log(V) + 0.5 - 2.0 + 8.0 * torch.rand((n * L, 1), device=dev, generator=gen)
        wt = w[pick].float()
        h += m * wt / wt.square().sum(1, keepdim=True)
        t.update(w=w, hidden=h.to(td).view(n, L, d), tokens=ids((n, L)))
    return t


class _State:
    pass


def prepare(case, seed):
    c, t = case, _tensors(case, seed)
    s = _State()
    s.c, s.t, s.ctx = c, t, _context()
    dev = torch.device("cuda")
    td = bstep.torch_dtype(c["dtype"])
    n, W, L, Hq, Hkv, D, V = t["n"], t["W"], c["L"], c["Hq"], c["Hkv"], c["D"], c["V"]
    if c["kind"] == "refresh":
        s.k_cache = torch.zeros((n, Hkv, W, D), dtype=td, device=dev)
        s.v_cache = torch.zeros_like(s.k_cache)
        s.out = torch.zeros((n, W, Hq, D), dtype=td, device=dev)
    if c["kind"] == "attention":
        s.out = torch.empty((n, L, Hq, D), dtype=td, device=dev)
        need = bs.bs_attention_workspace_bytes(t["reqs"], L, Hq, Hkv, D, bstep.dt_code(c["dtype"]))
        s.ws = torch.empty(need, dtype=torch.uint8, device=dev) if need else None
    if c["kind"] in ("step", "boundary"):
        # tokens and mask lie side by side so that one copy sets the state of the next pass
        s.fresh = torch.cat([t["tokens"].view(torch.uint8).flatten(), t["mask"].flatten()])
        s.now = s.fresh.clone()
        tokens = s.now[: 4 * n * W].view(torch.int32).view(n, W)
        mask = s.now[4 * n * W:].view(n, W)
        layers = [bstep.Layer(out=torch.empty((n, L, Hq, D), dtype=td, device=dev), **x) for x in t["layers"]]
        s.st = bstep.StepState(L, Hq, Hkv, D, V, c["dtype"], n, W, tokens, mask, layers, t["logits"], n).alloc()
    if c["kind"] == "head":
        s.packed = torch.empty(bs.bs_lm_head_pack_bytes(V, c["d"]), dtype=torch.uint8, device=dev)
        bs.bs_lm_head_pack(s.ctx, t["w"], c["d"], V, c["d"], bs.BS_BF16, s.packed, s.packed.numel())
        s.fresh = torch.cat([t["tokens"].view(torch.uint8).flatten(), t["masked"].flatten()])
        s.now = s.fresh.clone()
        s.tokens = s.now[: 4 * n * L].view(torch.int32).view(n, L)
        s.masked = s.now[4 * n * L:].view(n, L)
        s.n_unmasked = torch.empty(n, dtype=torch.int32, device=dev)
        s.done = torch.empty(n, dtype=torch.uint8, device=dev)
        s.eos = torch.empty(n, dtype=torch.uint8, device=dev)
        s.conf = torch.empty((n, L), dtype=torch.float32, device=dev)
        s.ws = torch.empty(bs.bs_lm_head_workspace_bytes(n, L, V), dtype=torch.uint8, device=dev)
        del t["w"]
    return s


def run(s):
    c, t = s.c, s.t
    if c["kind"] == "refresh":
        bs.bs_dual_cache_refresh(s.ctx, t["reqs"], c["L"], c["Hq"], c["Hkv"], c["D"], bs.BS_BF16, 0.0, c["base"],
                                 t["q"], t["k"], t["v"], t["n"], t["W"], s.k_cache, s.v_cache, s.out)
        return dict(out=s.out, k_cache=s.k_cache, v_cache=s.v_cache)
    if c["kind"] == "attention":
        x = t["layers"][0]
        bs.bs_dual_cache_block_attention(s.ctx, t["reqs"], c["L"], c["Hq"], c["Hkv"], c["D"],
                                         bstep.dt_code(c["dtype"]), 0.0, x["q"], x["k_new"], x["v_new"],
                                         x["k_cache"], x["v_cache"], t["n"], t["W"], True, s.out, s.ws,
                                         s.ws.numel() if s.ws is not None else 0)
        return dict(out=s.out, k_cache=x["k_cache"], v_cache=x["v_cache"])
    s.now.copy_(s.fresh)
    if c["kind"] == "head":
        bs.bs_lm_head_decode(s.ctx, t["reqs"], c["L"], c["d"], c["V"], bs.BS_BF16, t["hidden"], s.packed, s.tokens,
                             s.masked, 0.9, 1, -1, s.n_unmasked, s.done, s.eos, s.conf, s.ws, s.ws.numel())
        return dict(tokens=s.tokens, masked=s.masked, n_unmasked=s.n_unmasked, done=s.done, eos=s.eos, conf=s.conf)
    if c["kind"] == "boundary":
        bstep.compact(s.ctx, t["segs"], c["layers"], c["Hkv"], c["D"], c["dtype"], t["k_box"], t["v_box"],
                      t["k_stage"], t["v_stage"], t["k_box"], t["v_box"])
    st = s.st
    bstep.run_step(s.ctx, st, t["reqs"], want_conf=True)
    return dict(out=[x.out for x in st.layers], tokens=st.tokens, mask=st.mask, n_unmasked=st.n_unmasked, done=st.done,
                eos=st.eos_seen, conf=st.conf, pos=st.pos, k_box=t["k_box"], v_box=t["v_box"])


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c = case
    rows = _lengths(c)
    eb = 4 if c["dtype"] == "f32" else 2
    Hq, Hkv, D, V = c["Hq"], c["Hkv"], c["D"], c["V"]
    by = fl = 0
    masked = sum(m for *_, m in rows)
    for p, g, k, B, m in rows:
        ln = p + g
        if c["kind"] == "refresh":
            by += ln * (2 * Hq + 4 * Hkv) * D * eb
            fl += 4 * ln * ln * Hq * D
        elif c["kind"] != "head":
            # cached keys and values outside the block, the block's own, queries and
            # outputs, and the block's keys and values written into the cache
            by += c["layers"] * (2 * ln * Hkv + 2 * B * Hq + 2 * B * Hkv) * D * eb
            fl += c["layers"] * 4 * B * ln * Hq * D
    if c["kind"] in ("step", "boundary"):
        by += masked * V * eb
        fl += masked * V * 4
    if c["kind"] == "head":
        by += V * c["d"] * eb + masked * c["d"] * eb
        fl += 2 * masked * V * c["d"]
    if c["kind"] == "boundary":
        a = max(1, c["n"] // 4)
        mean = sum(p + g for p, g, *_ in rows) / len(rows)
        by += c["layers"] * 2 * 2 * a * mean * Hkv * D * eb
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "head":
        # fp32 sums of bf16 products on logits near 20, through an exponential
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    # bf16 outputs, probabilities rounded to bf16 before the second product
    return {"rel": 1e-2, "max": 4e-2, "differ": 2e-3}


# ---------------------------------------------------------------- the same in 64 bits
def _softmax_attention(q, k, v, scale):
    """q [Hq, m, D], k and v [Hkv, len, D], all in 64 bits -> [Hq, m, D]."""
    Hq, m, D = q.shape
    Hkv, ln, _ = k.shape
    qs = q.reshape(Hkv, Hq // Hkv * m, D).contiguous()
    s = torch.bmm(qs, k.transpose(1, 2).contiguous()) * scale
    return torch.bmm(torch.softmax(s, dim=2), v.contiguous()).reshape(Hq, m, D)


def _exact_layers(c, t):
    L, Hq, D = c["L"], c["Hq"], c["D"]
    outs = []
    if c["kind"] == "boundary":
        for sg in t["segs"]:
            ln = int(sg["len"])
            dst = slice(int(sg["dst_col"]), int(sg["dst_col"]) + ln)
            for box, stage in ((t["k_box"], t["k_stage"]), (t["v_box"], t["v_stage"])):
                box[:, int(sg["dst_row"]), :, dst] = stage[:, int(sg["src_row"]), :, :ln]
    for x in t["layers"]:
        out = torch.zeros((t["n"], L, Hq, D), dtype=torch.float64, device="cuda")
        for i, r in enumerate(t["reqs"]):
            row, off, ln = int(r["row"]), int(r["off"]), int(r["p"] + r["g"])
            s = int(r["p"] + r["k"] * L)
            B = min(L, int(r["g"] - r["k"] * L))
            k = x["k_cache"][row, :, off:off + ln].double()
            v = x["v_cache"][row, :, off:off + ln].double()
            k[:, s:s + B] = x["k_new"][i, :B].double().transpose(0, 1)
            v[:, s:s + B] = x["v_new"][i, :B].double().transpose(0, 1)
            q = x["q"][i, :B].double().transpose(0, 1)
            out[i, :B] = _softmax_attention(q, k, v, 1.0 / math.sqrt(D)).transpose(0, 1)
        outs.append(out)
    return outs


def _rope(x, base):
    """Rotate-half rotary embedding of x [len, H, D] at positions 0 .. len - 1, in 64 bits."""
    ln, _, D = x.shape
    f = torch.arange(D // 2, dtype=torch.float64, device=x.device)
    a = torch.arange(ln, dtype=torch.float64, device=x.device)[:, None] * base ** (-2.0 * f / D)
    cs, sn = torch.cos(a)[:, None], torch.sin(a)[:, None]
    x1, x2 = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([x1 * cs - x2 * sn, x2 * cs + x1 * sn], dim=-1)


def _exact_refresh(c, t):
    n, W, Hq, Hkv, D = t["n"], t["W"], c["Hq"], c["Hkv"], c["D"]
    out = torch.zeros((n, W, Hq, D), dtype=torch.float64, device="cuda")
    kc = torch.zeros((n, Hkv, W, D), dtype=torch.float64, device="cuda")
    vc = torch.zeros_like(kc)
    for r in t["reqs"]:
        row, off, ln = int(r["row"]), int(r["off"]), int(r["p"] + r["g"])
        cells = slice(off, off + ln)
        q = _rope(t["q"][row, cells].double(), c["base"]).transpose(0, 1)
        k = _rope(t["k"][row, cells].double(), c["base"]).transpose(0, 1)
        v = t["v"][row, cells].double().transpose(0, 1)
        kc[row, :, cells], vc[row, :, cells] = k, v
        for h in range(0, Hkv):   # one KV head at a time: the scores of a long row are large
            G = Hq // Hkv
            o = _softmax_attention(q[h * G:(h + 1) * G], k[h:h + 1], v[h:h + 1], 1.0 / math.sqrt(D))
            out[row, cells, h * G:(h + 1) * G] = o.transpose(0, 1)
    return dict(out=out, k_cache=kc, v_cache=vc)


def _exact_confidence(masked, rows_of):
    """conf [n, L]: 1 / sum exp(x - max) of the masked rows, -1 elsewhere; rows_of(i, j) gives 64-bit logits."""
    conf = torch.full(masked.shape, -1.0, dtype=torch.float64, device="cuda")
    for i in range(masked.shape[0]):
        j = torch.nonzero(masked[i]).flatten()
        x = rows_of(i, j)
        conf[i, j] = 1.0 / torch.exp(x - x.max(1, keepdim=True).values).sum(1)
    return conf


def exact(case, seed):
    c, t = case, _tensors(case, seed)
    if c["kind"] == "refresh":
        return _exact_refresh(c, t)
    if c["kind"] == "head":
        w = t["w"].double().t().contiguous()
        conf = _exact_confidence(t["masked"], lambda i, j: t["hidden"][i, j].double() @ w)
        return dict(tokens=None, masked=None, n_unmasked=None, done=None, eos=None, conf=conf)
    outs = _exact_layers(c, t)
    if c["kind"] == "attention":
        return dict(out=outs[0], k_cache=None, v_cache=None)
    conf = _exact_confidence(t["masked"], lambda i, j: t["logits"][i, j, : c["V"]].double())
    return dict(out=outs, tokens=None, mask=None, n_unmasked=None, done=None, eos=None, conf=conf, pos=None,
                k_box=None, v_box=None)
