"""The memory layer's work as a program gives it: the cases that its speed and accuracy are measured on.

Every case goes through the binding's public calls (``paper_2607_07386_amd.sdm``): prefill and decode, the
long-context schedule, training steps, the whole layer and the element-wise steps on either side of the
recurrence.  Shapes are those of the benchmark, the tests and the paper's layers, and generic ones beside them.
"""
from __future__ import annotations

import math

import torch

from paper_2607_07386_amd import sdm

EPS = 1e-5
SILU = 1


# ------------------------------------------------------------------------------------------------ cases
def _case(name, do, B, H, T, s, W, R, d_k, d_v, bf16=True, direct=False, clustered=False, chunk=0):
    return dict(name=name, do=do, B=B, H=H, T=T, s=s, W=W, R=R, d_k=d_k, d_v=d_v, bf16=bf16, direct=direct,
                clustered=clustered, chunk=chunk)


def listed():
    return [
        # The smallest call: a toy layer in fp32, as a first script or a unit test runs it.  Latency only.
        _case("tiny_forward_f32", "forward", 1, 2, 256, 32, 8, 8, 32, 32, bf16=False),
        # Serving: one token for each of 16 sequences, the benchmark's decode step.
        _case("decode_top32", "decode", 16, 16, 1, 256, 32, 32, 128, 128),
        # Serving the paper's 1.4B layer: one token for 16 sequences through the whole layer (gates, norm, gate).
        _case("decode_paper_1p4b", "decode_layer", 16, 2, 1, 240, 64, 64, 480, 960, direct=True),
        # A short prompt of two sequences, of a length that nobody chose.
        _case("prefill_short", "forward", 2, 16, 509, 256, 32, 32, 128, 128),
        # The benchmark's step: eight sequences of 4096 tokens, 65,536 slots per head.
        _case("forward_top32", "forward", 8, 16, 4096, 256, 32, 32, 128, 128, chunk=384),
        # The benchmark's training step: forward with the undo log, then the backward.
        _case("train_top32", "train", 4, 16, 4096, 256, 32, 32, 128, 128),
        # A large learned initial memory (1,048,576 slots per head), few streams of 8192 tokens.
        _case("forward_million_slots", "forward", 4, 8, 8192, 1024, 32, 32, 128, 128, chunk=1280),
        # One document of 65,536 tokens with recurring (clustered) keys: addressing, then the chunked scan.
        _case("long_context", "long", 1, 16, 65536, 512, 32, 32, 128, 128, clustered=True),
        # Training the paper's 1.4B layer: forward and backward of the whole layer, top-64.
        _case("train_layer_paper_1p4b", "train_layer", 8, 2, 4096, 240, 64, 64, 480, 960, direct=True),
        # One prompt through the paper's 8B layer: two heads of wide rows, too few streams for many waves.
        _case("prefill_paper_8b", "layer", 1, 2, 4096, 480, 64, 64, 960, 1920, direct=True),
        # A layer of no one's tuning in fp32: list lengths that differ, sizes that divide nothing.
        _case("train_layer_odd_f32", "train_layer", 3, 5, 777, 100, 48, 24, 72, 100, bf16=False),
        # The element-wise steps on either side of the recurrence, forward and backward, as a program that keeps
        # gates and output gate as tensors calls them.
        _case("gates_and_epilogue", "edges", 4, 16, 4096, 0, 0, 0, 0, 128),
    ]


def _spread(rng, lo, hi):
    """A whole number, uniform in the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["forward", "forward", "forward", "decode", "decode_layer", "train", "train", "layer", "train_layer",
                     "long", "edges"])
    bf16 = rng.random() < 0.7
    if do == "edges":
        return dict(do=do, B=rng.randint(1, 8), H=rng.randint(1, 24), T=_spread(rng, 1, 6000), s=0, W=0, R=0, d_k=0,
                    d_v=4 * _spread(rng, 4, 256), bf16=bf16, direct=False, clustered=False, chunk=0)
    k = rng.choice([8, 16, 32, 32, 32, 64, 64, _spread(rng, 2, 64)])
    W = R = k
    if do in ("layer", "train_layer", "long") and rng.random() < 0.5:
        R = rng.choice([max(1, k // 2), _spread(rng, 2, 64)])
    s = max(W, R, _spread(rng, 32, 512))
    if rng.random() < 0.5:
        s = max(W, R, rng.choice([64, 128, 240, 256, 480, 512]))
    direct = rng.random() < 0.3
    d_k = 2 * s if direct else rng.choice([32, 64, 128, 128, 256, 2 * rng.randint(8, 128)])
    d_v = rng.choice([32, 64, 128, 128, 256, 960, 4 * rng.randint(4, 128)])
    B, H = rng.choice([1, 1, 2, 4, 8, rng.randint(1, 16)]), rng.choice([1, 2, 2, 4, 8, 16, rng.randint(1, 16)])
    if do in ("decode", "decode_layer"):
        T = 1
        B = _spread(rng, 1, 64)
    elif do == "long":
        T = _spread(rng, 2048, 32768)
        B = 1
    else:
        T = _spread(rng, 2, 4096)
        if rng.random() < 0.3:
            T = rng.choice([64, 256, 512, 1024, 2048])
    # tables of at most 4 GiB, and row traffic of at most a tenth of the largest listed case's
    while B * H * s * s * d_v * 4 > 1 << 32 or B * H * T * (W + R) * d_v * 4 > 1 << 33:
        if B > 1:
            B = max(1, B // 2)
        elif H > 1:
            H = max(1, H // 2)
        elif T > 1024:
            T //= 2
        else:
            d_v = max(32, d_v // 8 * 4)
    chunk = rng.choice([0, 0, 0, 384, 64 * rng.randint(2, 20)]) if T > 1 else 0
    return dict(do=do, B=B, H=H, T=T, s=s, W=W, R=R, d_k=d_k, d_v=d_v, bf16=bf16, direct=direct,
                clustered=do == "long" or rng.random() < 0.2, chunk=chunk)


# ------------------------------------------------------------------------------------------------ inputs
def _inputs(c, seed, dev="cuda"):
    """Inputs as the layer meets them: unit-norm queries and keys, unit-norm sub-key rows, normal values, gate
    pre-activations of a fresh model, a learned initial memory of small entries."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    dt = torch.bfloat16 if c["bf16"] else torch.float32
    B, H, T, s, d_k, d_v = (c[n] for n in ("B", "H", "T", "s", "d_k", "d_v"))

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32)

    def unit(x):
        return x / x.norm(dim=-1, keepdim=True)

    x = dict(v=normal(B, H, T, d_v).to(dt))
    if c["do"] != "edges":
        if c["clustered"]:
            centres = unit(normal(H, 4096, d_k))
            heads = torch.arange(H, device=dev)[None, :, None]

            def vectors():
                which = torch.randint(0, 4096, (B, H, T), generator=g, device=dev)
                return unit(centres[heads, which] + 0.1 * normal(B, H, T, d_k)).to(dt)
        else:
            def vectors():
                return unit(normal(B, H, T, d_k)).to(dt)
        x["q"], x["k"] = vectors(), vectors()
        x["cb"] = None if c["direct"] else unit(normal(H, 2, s, d_k // 2)).to(dt)
        x["m0"] = 0.02 * normal(H, s * s, d_v)
    if c["do"] in ("edges", "layer", "train_layer", "decode_layer"):
        x["a"], x["b"], x["g"] = normal(B, H, T).to(dt), normal(B, H, T).to(dt), normal(B, H, T, d_v).to(dt)
        u = torch.rand((3, max(H, d_v)), generator=g, device=dev)
        x["A"] = (16 * u[0, :H]).contiguous()
        x["b_dt"] = torch.log(torch.expm1(0.001 + 0.099 * u[1, :H])).contiguous()
        x["gamma"] = (0.5 + u[2, :d_v]).contiguous()
    else:
        x["alpha"] = torch.sigmoid(-normal(B, H, T)).to(dt)
        x["beta"] = torch.sigmoid(normal(B, H, T)).to(dt)
    if c["do"] in ("train", "train_layer", "edges"):
        x["dy"] = normal(B, H, T, d_v)
    if c["do"] == "edges":
        x["y"] = normal(B, H, T, d_v)
        x["dalpha"], x["dbeta"] = normal(B, H, T), normal(B, H, T)
    return x


def prepare(case, seed):
    """Inputs, the sequences' memory tables and the buffers that a program allocates once."""
    c = case
    x = _inputs(c, seed)
    st = dict(c=c, x=x)
    if c["do"] == "edges":
        return st
    B, H, T, W, R, d_v = (c[n] for n in ("B", "H", "T", "W", "R", "d_v"))
    dev = x["v"].device
    st["mem"] = torch.empty((B, H, c["s"] ** 2, d_v), dtype=torch.float32, device=dev)
    sdm.mem_init(st["mem"], x["m0"])
    if c["do"] == "long":
        st["ws"] = sdm.chunked_workspace(B, H, T, W, R, dev)
    else:
        st["ws"] = sdm.fwd_workspace(B, H, T, W, R, dev)
    if c["do"] in ("train", "train_layer"):
        st["saved"] = sdm.saved_buffer(B, H, T, W, d_v, dev)
    if c["do"] == "train":
        st["ws_b"] = sdm.bwd_workspace(B, H, T, W, R, d_v, dev)
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    c, x, mem = state["c"], state["x"], state.get("mem")
    N, W, R, do = c["s"] ** 2, c["W"], c["R"], c["do"]
    if do in ("forward", "decode"):
        o = sdm.forward(x["q"], x["k"], x["cb"], x["cb"], x["v"], x["alpha"], x["beta"], mem, N, W,
                        workspace=state["ws"], chunk=c["chunk"])
        return dict(o, mem=mem)
    if do == "train":
        o = sdm.forward(x["q"], x["k"], x["cb"], x["cb"], x["v"], x["alpha"], x["beta"], mem, N, W,
                        saved=state["saved"], workspace=state["ws"], chunk=c["chunk"])
        gr = sdm.scan_bwd(o["w_idx"], o["w_val"], o["r_idx"], o["r_val"], x["v"], x["alpha"], x["beta"], mem,
                          state["saved"], x["dy"], cb_q=x["cb"], cb_k=x["cb"], d_k=c["d_k"], workspace=state["ws_b"])
        return dict(o, **gr, mem=mem)
    if do in ("layer", "decode_layer"):
        o = sdm.layer_fwd(x["q"], x["k"], x["cb"], x["cb"], x["v"], x["a"], x["b"], x["g"], x["A"], x["b_dt"],
                          x["gamma"], EPS, SILU, mem, N, W, R, workspace=state["ws"], chunk=c["chunk"])
        return dict(o, mem=mem)
    if do == "train_layer":
        o = sdm.layer_fwd(x["q"], x["k"], x["cb"], x["cb"], x["v"], x["a"], x["b"], x["g"], x["A"], x["b_dt"],
                          x["gamma"], EPS, SILU, mem, N, W, R, saved=state["saved"], workspace=state["ws"],
                          chunk=c["chunk"])
        gr = sdm.layer_bwd(o, x["v"], x["a"], x["b"], x["g"], x["A"], x["b_dt"], x["gamma"], EPS, SILU, mem,
                           state["saved"], x["dy"], cb_q=x["cb"], cb_k=x["cb"], d_k=c["d_k"])
        return dict(o, **gr, mem=mem)
    if do == "long":
        r_idx, r_val = sdm.address(x["q"], x["cb"], N, R)
        w_idx, w_val = sdm.address(x["k"], x["cb"], N, W)
        y = sdm.scan_fwd_chunked(w_idx, w_val, r_idx, r_val, x["v"], x["alpha"], x["beta"], mem,
                                 workspace=state["ws"])
        return dict(y=y, r_idx=r_idx, r_val=r_val, w_idx=w_idx, w_val=w_val, mem=mem)
    alpha, beta = sdm.gates(x["a"], x["b"], x["A"], x["b_dt"])
    o, rstd = sdm.norm_gate(x["y"], x["g"], x["gamma"], EPS, SILU, want_rstd=True)
    dy, dg, dgamma = sdm.norm_gate_bwd(x["y"], x["g"], x["gamma"], EPS, SILU, x["dy"])
    da, db, dA, db_dt = sdm.gates_bwd(x["a"], x["b"], x["A"], x["b_dt"], x["dalpha"], x["dbeta"])
    return dict(alpha=alpha, beta=beta, o=o, rstd=rstd, dy=dy, dg=dg, dgamma=dgamma, da=da, db=db, dA=dA, db_dt=db_dt)


# ------------------------------------------------------------------------------------------------ what it needs
def work(case):
    """Inputs once, outputs once, and of the tables the rows that a sequence's distinct slots take (for slots drawn
    evenly): read once, and written once where the tokens write them.  The undo log goes out and comes back."""
    c = case
    B, H, T, s, W, R, d_k, d_v = (c[n] for n in ("B", "H", "T", "s", "W", "R", "d_k", "d_v"))
    th, e = B * H * T, 2 if c["bf16"] else 4
    if c["do"] == "edges":
        return {"bytes": th * (d_v * (4 + e + 4) + 4 + d_v * (4 + e + 4 + 4 + 4) + 2 * e + 8 + 2 * e + 8 + 8),
                "flops": th * (d_v * 30 + 60)}
    N = s * s

    def distinct(per_token):
        return N * -math.expm1(T * math.log1p(-min(per_token / N, 1 - 1e-12)))

    rows = B * H * d_v * 4
    touched, written = distinct(W + R), distinct(W)
    size = 2 * th * d_k * e + (0 if c["direct"] else H * 2 * s * (d_k // 2) * e) + th * (d_v * e + 2 * e)
    size += th * (W + R) * 8 + th * d_v * 4 + rows * (touched + written)
    score = 0 if c["direct"] else 2 * th * 2 * s * d_k
    flops = score + th * d_v * (2 * W + 3 * W + 2 * R)
    layer = c["do"] in ("layer", "train_layer", "decode_layer")
    if layer:
        size += th * d_v * (e + 4)
        flops += th * d_v * 10
    if c["do"] in ("train", "train_layer"):
        size += 2 * th * W * d_v * 4  # the undo log, out and in
        # the backward: values and gates, lists and the gradient in; the tables' rows undone, the adjoint table out
        size += th * (d_v * e + 2 * e + (W + R) * 8 + d_v * 4) + rows * (touched + written + N)
        size += th * (d_v * 4 + 8 + 2 * d_k * 4) + (0 if layer else th * (W + R) * 4)
        if layer:
            size += th * d_v * (4 + e + 4)
        flops += th * d_v * (12 * W + 4 * R) + (0 if c["direct"] else th * (W + R) * d_k * 2)
    return {"bytes": float(size), "flops": float(flops)}


def tolerance(case):
    """32-bit sums: the outputs are 1e-7 to 9e-7 (the long sum of dgamma) off their values in 64 bits.  Where many
    scores come from sums of products, some of the tokens' k-th and next best differ by less than such a sum's
    rounding, and either choice is right: against the choice from 64-bit sums (about one token in 10^5 falls to the
    other side) y and the tables are up to 1e-3 off and the weights' gradients, whose entries then shift in their
    row, up to 3.2e-3."""
    if case["do"] == "edges" or case["direct"] or case["B"] * case["H"] * case["T"] < 50_000:
        return {"rel": 4e-6, "max": 4e-4}
    return {"rel": 1.2e-2 if case["do"].startswith("train") else 4e-3, "max": 1.0, "differ": 1e-4}


# ------------------------------------------------------------------------------------------------ in 64 bits
def _ordered(score, ids, low):
    """Whole numbers that order by (score descending, id ascending)."""
    bits = (score + 0.0).contiguous().view(torch.int32).to(torch.int64)
    key = torch.where(bits < 0, -(bits & 0x7FFFFFFF), bits)
    return (key << 24) | (low - ids)


def _address(x, cb, s, k):
    """Slots (ascending) and softmax weights of one side.  The choice is between the scores' 32-bit values, as the
    layer defines it; everything after it is in 64 bits."""
    B, H, T, d_k = x.shape
    dev = x.device
    idx = torch.empty((B, H, T, k), dtype=torch.int64, device=dev)
    val = torch.empty((B, H, T, k), dtype=torch.float64, device=dev)
    a, b = torch.meshgrid(torch.arange(k, device=dev), torch.arange(k, device=dev), indexing="ij")
    keep = ((a + 1) * (b + 1) <= k).reshape(-1).nonzero().squeeze(-1)  # the others have k better pairs
    a, b = a.reshape(-1)[keep], b.reshape(-1)[keep]
    step = max(1, (1 << 26) // max(s, len(keep)) // 4)
    for i in range(B):
        for h in range(H):
            for t in range(0, T, step):
                r = x[i, h, t:t + step].double()
                halves = []
                for p in range(2):
                    sub = r[:, p * (d_k // 2):(p + 1) * (d_k // 2)]
                    sc = sub if cb is None else sub @ cb[h, p].double().t()
                    ids = torch.arange(s, device=dev).expand_as(sc)
                    top = _ordered(sc.float(), ids, 0xFFFFFF).topk(k, dim=-1).values
                    at = 0xFFFFFF - (top & 0xFFFFFF)
                    halves.append((sc.gather(1, at), at))
                (s0, a0), (s1, a1) = halves
                ids = a0[:, a] * s + a1[:, b]
                pair = s0[:, a].float() + s1[:, b].float()
                top = _ordered(pair, ids, 0xFFFFFF).topk(k, dim=-1).indices
                ids, at = ids.gather(1, top).sort(dim=-1)
                full = (s0[:, a] + s1[:, b]).gather(1, top.gather(1, at))
                idx[i, h, t:t + step] = ids
                val[i, h, t:t + step] = torch.softmax(full, dim=-1)
    return idx, val


def _scan(wi, wv, ri, rv, v, alpha, beta, mem, save):
    """The recurrence, token by token; mem [streams * N, d_v] in place."""
    S, T, W = wi.shape
    N = mem.shape[0] // S
    base = (torch.arange(S, device=wi.device) * N)[:, None]
    y = torch.empty_like(v)
    saved = torch.empty((T, S, W, v.shape[-1]), dtype=torch.float64, device=v.device) if save else None
    for t in range(T):
        i = (wi[:, t] + base).reshape(-1)
        P = mem.index_select(0, i).view(S, W, -1)
        if save:
            saved[t] = P
        D = P * alpha[:, t, None, None]
        kap = wv[:, t]
        e = beta[:, t, None] * (v[:, t] - torch.bmm(kap[:, None], D)[:, 0])
        mem.index_copy_(0, i, (D + kap[:, :, None] * e[:, None]).view(S * W, -1))
        M = mem.index_select(0, (ri[:, t] + base).reshape(-1)).view(S, ri.shape[-1], -1)
        y[:, t] = torch.bmm(rv[:, t][:, None], M)[:, 0]
    return y, saved


def _scan_bwd(wi, wv, ri, rv, v, alpha, beta, mem, saved, dy):
    """Reverse mode of _scan from the undo log; mem goes back to the start."""
    S, T, W = wi.shape
    N = mem.shape[0] // S
    R = ri.shape[-1]
    base = (torch.arange(S, device=wi.device) * N)[:, None]
    G = torch.zeros_like(mem)
    dv, da, db = torch.empty_like(v), torch.empty_like(alpha), torch.empty_like(beta)
    dw, dr = torch.empty_like(wv), torch.empty_like(rv)
    for t in range(T - 1, -1, -1):
        i, j = (wi[:, t] + base).reshape(-1), (ri[:, t] + base).reshape(-1)
        d = dy[:, t]
        dr[:, t] = torch.bmm(mem.index_select(0, j).view(S, R, -1), d[:, :, None])[:, :, 0]
        G.index_add_(0, j, (rv[:, t, :, None] * d[:, None]).view(S * R, -1))
        g = G.index_select(0, i).view(S, W, -1)
        P = saved[t]
        al, be, kap = alpha[:, t, None, None], beta[:, t, None], wv[:, t]
        D = al * P
        u = torch.bmm(kap[:, None], D)[:, 0]
        e = be * (v[:, t] - u)
        eb = torch.bmm(kap[:, None], g)[:, 0]
        dv[:, t] = be * eb
        db[:, t] = (eb * (v[:, t] - u)).sum(-1)
        dw[:, t] = torch.bmm(g, e[:, :, None])[:, :, 0] - be * torch.bmm(D, eb[:, :, None])[:, :, 0]
        Db = g - be[:, :, None] * kap[:, :, None] * eb[:, None]
        da[:, t] = (Db * P).sum((1, 2))
        G.index_copy_(0, i, (al * Db).view(S * W, -1))
        mem.index_copy_(0, i, P.reshape(S * W, -1))
    return dict(dv=dv, dalpha=da, dbeta=db, dw_val=dw, dr_val=dr, dmem0=G)


def _address_bwd(cb, idx, val, dval, s, d_k):
    """Through the softmax and the sums of sub-scores to the vector."""
    B, H, T, k = idx.shape
    ds = val * (dval - (val * dval).sum(-1, keepdim=True))
    out = torch.empty((B, H, T, d_k), dtype=torch.float64, device=idx.device)
    for p, at in enumerate((idx // s, idx % s)):
        sub = torch.zeros((B, H, T, s), dtype=torch.float64, device=idx.device).scatter_add_(-1, at, ds)
        half = sub if cb is None else torch.matmul(sub, cb[:, p].double().contiguous())
        out[..., p * (d_k // 2):(p + 1) * (d_k // 2)] = half
    return out


def _gates(x):
    z = x["a"].double() + x["b_dt"].double()[:, None]
    return torch.exp(-x["A"].double()[:, None] * torch.nn.functional.softplus(z, threshold=700)), x["b"].double().sigmoid()


def _gates_bwd(x, dalpha, dbeta):
    al, be = _gates(x)
    z = x["a"].double() + x["b_dt"].double()[:, None]
    da = -dalpha * x["A"].double()[:, None] * al * z.sigmoid()
    dA = -(dalpha * torch.nn.functional.softplus(z, threshold=700) * al).sum((0, 2))
    return dict(da=da, db=dbeta * be * (1 - be), dA=dA, db_dt=da.sum((0, 2)))


def _epilogue(y, x, dout):
    y, g, ga = (t.double().requires_grad_(dout is not None) for t in (y, x["g"], x["gamma"]))
    rstd = torch.rsqrt(y.square().mean(-1, keepdim=True) + EPS)
    o = y * rstd * ga * torch.nn.functional.silu(g)
    out = dict(o=o.detach(), rstd=rstd.detach()[..., 0])
    if dout is not None:
        out["dy"], out["dg"], out["dgamma"] = torch.autograd.grad(o, (y, g, ga), dout.double())
    return out


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    if c["do"] == "edges":
        alpha, beta = _gates(x)
        return dict(_epilogue(x["y"], x, x["dy"]), alpha=alpha, beta=beta,
                    **_gates_bwd(x, x["dalpha"].double(), x["dbeta"].double()))
    B, H, T, s, W, R, d_k, d_v = (c[n] for n in ("B", "H", "T", "s", "W", "R", "d_k", "d_v"))
    S, train, layer = B * H, c["do"].startswith("train"), "layer" in c["do"]
    ri, rv = _address(x["q"], x["cb"], s, R)
    wi, wv = _address(x["k"], x["cb"], s, W)
    alpha, beta = _gates(x) if layer else (x["alpha"].double(), x["beta"].double())
    mem = x.pop("m0").double().expand(B, -1, -1, -1).reshape(S * s * s, d_v)
    flat = [t.reshape(S, T, *t.shape[3:]) for t in (wi, wv, ri, rv, x["v"].double(), alpha, beta)]
    y, saved = _scan(*flat, mem, train)
    y = y.view(B, H, T, d_v)
    out = dict(y=y, r_idx=None, w_idx=None, r_val=rv, w_val=wv)
    dy = x.get("dy")
    if layer:
        epi = _epilogue(y, x, dy)
        out["o"] = epi["o"]
        if train:
            dy = epi["dy"]
            out["dg"], out["dgamma"] = epi["dg"], epi["dgamma"]
    if train:
        gr = _scan_bwd(*flat, mem, saved, dy.double().reshape(S, T, d_v))
        gr = {n: t.view(B, H, s * s, d_v) if n == "dmem0" else t.view(B, H, T, *t.shape[2:]) for n, t in gr.items()}
        gr["dq"] = _address_bwd(x["cb"], ri, rv, gr["dr_val"], s, d_k)
        gr["dk"] = _address_bwd(x["cb"], wi, wv, gr["dw_val"], s, d_k)
        if layer:
            gr.update(_gates_bwd(x, gr.pop("dalpha"), gr.pop("dbeta")))
            del gr["dw_val"], gr["dr_val"]
        out.update(gr)
    out["mem"] = mem.view(B, H, s * s, d_v)
    return out
