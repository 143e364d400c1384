"""The workloads this library is timed on, through its public entry points (the ctypes functions of
paper_2404_15159_amd.binding, one per C entry point).

A case is one pass of a user's program: a forward call of a serving step, a forward and a backward
call of a training step, or an optimiser step.  `listed` names the fixed ones, `draw` gives further
ones of the same ranges, `prepare` makes the inputs and everything a program keeps between calls
(weights, transposed frozen copies, workspace, output buffers), `run` is the timed pass, `exact` is
the same result in 64-bit torch.

Model shapes are the LLaMA-2 7B / 13B and LLaMA-3 8B feed-forward blocks and attention projections
(and small generic widths); adapters have 8 or 16 experts, top-2, ranks 2 to 32.  Inputs follow the
recipe of paper_2404_15159_amd/synth.py: x, dy ~ N(0, 1), frozen W ~ N(0, 0.02^2), A uniform within
1/sqrt(fan_in), B ~ N(0, 0.01^2), router ~ N(0, 0.02^2).
"""
import math

import torch

from paper_2404_15159_amd import binding as B

DEV = "cuda:0"
BLOCK = ("A_gate", "B_gate", "A_up", "B_up", "A_down", "B_down", "W_router")
FROZEN = ("W_gate", "W_up", "W_down")
MODELS = {"7b": (4096, 11008), "13b": (5120, 13824), "l3_8b": (4096, 14336)}
ADAMW = dict(lr=2e-4, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=7)


def block(kind, model, T, N=8, k=2, r=16, M=1, structure="uniform", dtype="bf16", shared=0):
    d, f = MODELS[model] if isinstance(model, str) else model
    return dict(kind=kind, T=T, d=d, d_ff=f, N=N, k=k, r=r, M=M, structure=structure, dtype=dtype,
                shared=shared)


def linear(kind, T, d_in, d_out, r=16):
    return dict(kind=kind, T=T, d_in=d_in, d_out=d_out, r=r, dtype="bf16")


def listed():
    cases = {
        # one new token of one sequence: latency of the whole launch chain, weights read once
        "decode_1_token": block("static", "7b", 1),
        # one new token of each of 64 sequences in flight
        "decode_64": block("forward", "7b", 64),
        # a prompt of ragged length before the first decode step
        "prefill_517": block("forward", "7b", 517),
        # one fine-tuning step on a micro-batch of two short sequences
        "train_short": block("train", "7b", 300),
        # the usual fine-tuning step: 8 sequences of 512 tokens (rank 16, 8 experts, top-2)
        "train_7b": block("train", "7b", 4096),
        # the same with the rank the rank study ends on, and an odd number of tokens
        "train_rank32": block("train", "7b", 1999, r=32),
        # the largest step: 16 sequences of 1024 tokens in topic clusters, 16 experts of rank 8
        "train_l3_8b": block("train", "l3_8b", 16384, N=16, r=8, structure="clusters"),
        # two adapters trained together on one frozen base
        "train_two_adapters": block("multi", "7b", 2048, M=2),
        # weight-decomposed experts, magnitudes per expert
        "train_dora": block("dora", "7b", 2048),
        # adapter on a square attention projection, one training step
        "attn_proj_train": linear("linear_train", 4096, 4096, 4096),
        # the optimiser step over the seven tensors of one block's adapter
        "adamw_block": dict(kind="adamw", d=4096, d_ff=11008, N=8, r=16, dtype="f32"),
        # 32-bit storage: the small configuration the numerics are debugged on
        "train_tiny_f32": block("train", (128, 344), 256, r=8, dtype="f32"),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "train", "train", "train", "multi",
                       "dora", "linear", "linear", "adamw", "f32"])
    model = rng.choice(["7b", "7b", "13b", "l3_8b", "small"])
    if model == "small":
        d = 8 * _log(rng, 32, 256)
        model = (d, 8 * int(d * rng.uniform(2.5, 4.0) / 8))
    N, r = rng.choice([(8, 16), (8, 16), (16, 8), (8, 8), (8, 4), (8, 2), (8, 32), (4, 32)])
    k = rng.choice([2, 2, 2, 2, 1, 3])
    structure = rng.choice(["uniform", "uniform", "skew", "clusters"])
    if kind == "decode":
        # the library's own scratch holds decode batches up to rank 16
        kind = rng.choice(["static", "forward"]) if r <= 16 else "forward"
        return block(kind, model, _log(rng, 1, 128), N, 2, r)
    if kind == "prefill":
        return block("forward", model, _log(rng, 129, 4096), N, k, r, structure=structure)
    if kind == "train":
        return block("train", model, _log(rng, 256, 8192), N, k, r, structure=structure)
    if kind == "multi":
        M, N, r = rng.choice([(2, 8, 16), (2, 8, 8), (4, 4, 16), (3, 8, 8)])
        return block("multi", model, _log(rng, 256, 8192), N, 2, r, M=M)
    if kind == "dora":
        return block("dora", model, _log(rng, 256, 4096), N, 2, r, shared=rng.choice([0, 1]))
    if kind == "linear":
        d_in, d_out = rng.choice([(4096, 4096), (5120, 5120), (4096, 1024)])
        if rng.random() < 0.4:
            return linear("linear_forward", _log(rng, 1, 2048), d_in, d_out, r)
        return linear("linear_train", _log(rng, 128, 8192), d_in, d_out, r)
    if kind == "adamw":
        d, f = MODELS[model] if isinstance(model, str) else model
        return dict(kind="adamw", d=d, d_ff=f, N=N, r=r, dtype="f32")
    d = 8 * _log(rng, 8, 32)
    return block("train", (d, 8 * int(d * 2.7 / 8)), _log(rng, 64, 1024), rng.choice([4, 8]), 2,
                 rng.choice([4, 8, 16]), dtype="f32")


# ---- inputs ---------------------------------------------------------------------------------

def _scale(case):
    return 2.0    # alpha = 2 r at every rank of the configurations


def _inputs(case, seed):
    """Every tensor the caller owns, in the storage dtype, from the seed alone."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def nrm(shape, std):
        return (torch.randn(shape, generator=gen, device=DEV) * std).to(td)

    def uni(shape, fan_in):
        return ((torch.rand(shape, generator=gen, device=DEV) * 2 - 1) / math.sqrt(fan_in)).to(td)

    t = {}
    if case["kind"].startswith("linear"):
        T, di, do, r = case["T"], case["d_in"], case["d_out"], case["r"]
        t["x"], t["W"], t["A"] = nrm((T, di), 1.0), nrm((do, di), 0.02), uni((r, di), di)
        t["B"], t["dy"] = nrm((do, r), 0.01), nrm((T, do), 1.0)
        return t
    d, f, r = case["d"], case["d_ff"], case["r"]
    N = case["N"] * case.get("M", 1)
    shapes = dict(A_gate=(N, r, d), B_gate=(N, f, r), A_up=(N, r, d), B_up=(N, f, r),
                  A_down=(N, r, f), B_down=(N, d, r), W_router=(N, d))
    if case["kind"] == "adamw":
        for n, s in shapes.items():
            t["p_" + n], t["g_" + n] = nrm(s, 0.01), nrm(s, 1e-3)
            t["m_" + n], t["v_" + n] = nrm(s, 1e-3), nrm(s, 1e-3).square()
            t["lowp_" + n] = torch.empty(s, dtype=torch.bfloat16, device=DEV)
        return t
    T = case["T"]
    x = torch.randn((T, d), generator=gen, device=DEV)
    router = torch.randn((N, d), generator=gen, device=DEV) * 0.02
    if case["structure"] == "skew":          # expert 0's logit gets +1.5
        x[:, d - 1] = 1.0
        router[0, d - 1] += 1.5
    elif case["structure"] == "clusters":    # sequences of four topics
        sign = torch.randint(0, 2, (4, d), generator=gen, device=DEV).float() * 2 - 1
        x += 0.5 * sign[(torch.arange(T, device=DEV) // max(1, min(1024, T // 8))) % 4]
    t["x"], t["W_router"] = x.to(td), router.to(td)
    t["W_gate"], t["W_up"], t["W_down"] = nrm((f, d), 0.02), nrm((f, d), 0.02), nrm((d, f), 0.02)
    for n, s in shapes.items():
        if n.startswith("A"):
            t[n] = uni(s, s[2])
        elif n.startswith("B"):
            t[n] = nrm(s, 0.01 if case["dtype"] == "bf16" else 0.02)
    if case["kind"] in ("train", "multi", "dora"):
        t["dy"] = nrm((T, d), 1.0)
    if case["kind"] == "multi":              # whole sequences alternate between the adapters
        t["token_model"] = (torch.arange(T, device=DEV) // max(1, T // 7) % case["M"]).to(torch.int32)
    if case["kind"] == "dora":
        E = () if case["shared"] else (N,)
        for n, s, fan in (("m_gate", E + (f,), d), ("m_up", E + (f,), d), ("m_down", E + (d,), f)):
            u = torch.rand(s, generator=gen, device=DEV)
            t[n] = (0.8 + 0.4 * u) * 0.02 * math.sqrt(fan)
    return t


class State:
    """Tensors and handles of one problem, held for its lifetime."""


def prepare(case, seed):
    s = State()
    kind = s.kind = case["kind"]
    t = s.t = _inputs(case, seed)
    code = B.BF16 if case["dtype"] == "bf16" else B.F32
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def empty(shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=DEV)

    def transposed(w):
        out = empty((w.shape[1], w.shape[0]), td)
        B.mixlora_transpose(w, out, w.shape[0], w.shape[1], code)
        return out

    if kind == "adamw":
        s.h = B.AdamW(**ADAMW)
        s.names = [n[2:] for n in t if n.startswith("p_")]
        return s
    if kind.startswith("linear"):
        T, di, do, r = case["T"], case["d_in"], case["d_out"], case["r"]
        back = kind == "linear_train"
        s.dims = B.LinearDims(T, di, do, r, _scale(case), code)
        s.W_T = transposed(t["W"]) if back else None
        s.ws_bytes = B.mixlora_lora_linear_workspace_bytes(s.dims, back)
        s.ws = empty(s.ws_bytes, torch.uint8)
        s.out = {"y": empty((T, do), td)}
        if back:
            s.out.update(dx=empty((T, di), td), dA=empty((r, di)), dB=empty((do, r)))
        return s
    T, d, f, k, r, M = (case[n] for n in ("T", "d", "d_ff", "k", "r", "M"))
    N = case["N"] * M
    s.dims = B.make_dims(T, d, f, case["N"], k, r, _scale(case), dtype=code)
    back = kind in ("train", "multi", "dora")
    w = {n: t[n] for n in FROZEN + BLOCK}
    if back:
        for n in FROZEN:
            w[n + "_T"] = transposed(t[n])
    s.keep, s.weights = w, B.make_weights(w)
    if kind == "multi":
        s.multi = B.make_multi(M, t["token_model"])
        s.ws_bytes = B.mixlora_multi_workspace_bytes(s.dims, M, True)
    elif kind == "dora":
        s.dora = B.make_dora(t, shared=bool(case["shared"]))
        s.ws_bytes = B.mixlora_dora_workspace_bytes(s.dims, True)
    else:
        s.ws_bytes = B.mixlora_workspace_bytes(s.dims, back)
    s.ws = empty(s.ws_bytes if kind != "static" else 0, torch.uint8)
    s.out = dict(y=empty((T, d), td), topk_idx=empty((T, k), torch.int32), topk_w=empty((T, k)),
                 counts=empty((N,), torch.int32), aux_loss=empty((M,)))
    if back:
        s.g = {"d" + n: empty(t[n].shape) for n in BLOCK}
        s.grads = B.make_grads(s.g)
        s.out.update(s.g, dx=empty((T, d), td))
    if kind == "dora":
        gm = {"d" + n: empty(t[n].shape) for n in B.DORA_FIELDS}
        s.dora_grads = B.make_dora_grads(gm)
        s.out.update(gm)
    return s


def run(s):
    t = s.t
    if s.kind == "adamw":
        for n in s.names:
            p = t["p_" + n]
            B.mixlora_adamw_step(s.h, p.numel(), p, t["g_" + n], t["m_" + n], t["v_" + n],
                                 t["lowp_" + n])
        return {q + n: t[q + n] for n in s.names for q in ("p_", "m_", "v_", "lowp_")}
    o = s.out
    if s.kind.startswith("linear"):
        B.mixlora_lora_linear_forward(s.dims, t["W"], t["A"], t["B"], t["x"], o["y"], s.ws,
                                      s.ws_bytes)
        if s.kind == "linear_train":
            B.mixlora_lora_linear_backward(s.dims, t["W"], s.W_T, t["A"], t["B"], t["x"], t["dy"],
                                           s.ws, s.ws_bytes, o["dx"], o["dA"], o["dB"])
        return o
    fwd = (t["x"], o["y"], o["topk_idx"], o["topk_w"], o["counts"], o["aux_loss"])
    if s.kind == "static":
        B.mixlora_ffn_forward_static(s.dims, s.weights, *fwd)
    elif s.kind == "multi":
        B.mixlora_multi_forward(s.dims, s.multi, s.weights, *fwd, s.ws, s.ws_bytes)
        B.mixlora_multi_backward(s.dims, s.multi, s.weights, t["x"], t["dy"], s.ws, s.ws_bytes,
                                 o["dx"], s.grads)
    elif s.kind == "dora":
        B.mixlora_dora_forward(s.dims, s.weights, s.dora, *fwd, s.ws, s.ws_bytes)
        B.mixlora_dora_backward(s.dims, s.weights, s.dora, t["x"], t["dy"], 1.0, s.ws, s.ws_bytes,
                                o["dx"], s.grads, s.dora_grads)
    else:
        B.mixlora_ffn_forward(s.dims, s.weights, *fwd, s.ws, s.ws_bytes)
        if s.kind == "train":
            B.mixlora_ffn_backward(s.dims, s.weights, t["x"], t["dy"], 1.0, s.ws, s.ws_bytes,
                                   o["dx"], s.grads)
    return o


def work(case):
    """Inputs read once, outputs written once; frozen products once per token (gate, up, down),
    their input-gradient counterparts, and the rank-r and router terms."""
    kind, r = case["kind"], case["r"]
    E = 2 if case["dtype"] == "bf16" else 4
    if kind.startswith("linear"):
        T, di, do = case["T"], case["d_in"], case["d_out"]
        by = E * (T * di + di * do + r * (di + do) + T * do)
        fl = 2.0 * T * (di * do + r * (di + do))
        if kind == "linear_train":
            by += E * (T * do + T * di) + 4 * r * (di + do)
            fl += 2.0 * T * (di * do + 2 * r * (di + do))
        return {"bytes": by, "flops": fl}
    d, f, N = case["d"], case["d_ff"], case["N"] * case.get("M", 1)
    banks = 3 * N * r * (d + f) + N * d
    if kind == "adamw":
        return {"bytes": banks * (16 + 12 + 2), "flops": 12.0 * banks}
    T, k = case["T"], case["k"]
    units = 3 if kind != "dora" else 2 + k    # the magnitude of the down projection is per expert
    by = E * (3 * d * f + banks + 2 * T * d) + 12 * T * k
    fl = T * (units * 2.0 * d * f + 6.0 * k * r * (d + f) + 2.0 * d * case["N"])
    if kind in ("train", "multi", "dora"):
        by += 2 * E * T * d + 4 * banks
        fl += T * (units * 2.0 * d * f + 12.0 * k * r * (d + f) + 4.0 * d * case["N"])
    if kind == "dora":
        by += 8 * (1 if case["shared"] else N) * (2 * f + d)
        fl += 2.0 * N * r * 3 * d * f
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """bf16 keeps 8 bits: every stored intermediate adds up to 2^-9 of its size, and four to six of
    them lie between an input and an output or gradient (4e-3 seen against 64 bits).  In 32 bits
    sums over up to a few thousand terms show 1e-6.  Whole values differ only where two experts'
    logits tie within rounding."""
    if case["dtype"] == "bf16":
        return {"rel": 1.6e-2, "differ": 2e-3}
    return {"rel": 1e-5, "differ": 2e-3}


# ---- 64-bit reference -----------------------------------------------------------------------

def _expert(t, e, x, G, U, s, mag):
    """Expert e on rows x, whose frozen gate and up products are G and U."""
    W = {p: t["W_" + p] for p in ("gate", "up", "down")}
    A = {p: t["A_" + p][e] for p in W}
    Bm = {p: t["B_" + p][e] for p in W}
    c = {}
    for p in W:
        c[p] = 1.0
        if mag:
            n = (W[p] + s * Bm[p] @ A[p]).square().sum(1).sqrt()
            m = t["m_" + p]
            c[p] = (m[e] if m.dim() == 2 else m) / n
            c["n_" + p] = n
    pg, pu = x @ A["gate"].T, x @ A["up"].T
    vg, vu = G + s * pg @ Bm["gate"].T, U + s * pu @ Bm["up"].T
    g, u = c["gate"] * vg, c["up"] * vu
    sg = torch.sigmoid(g)
    a = g * sg * u
    q = a @ A["down"].T
    vd = a @ W["down"].T + s * q @ Bm["down"].T
    return dict(A=A, B=Bm, c=c, pg=pg, pu=pu, vg=vg, vu=vu, g=g, u=u, sg=sg, a=a, q=q, vd=vd)


def _exact_block(case, t):
    """One adapter's block, t in float64."""
    k, s, N = case["k"], _scale(case), case["N"]
    mag, back = case["kind"] == "dora", "dy" in t
    x = t["x"]
    T, d = x.shape
    z = x @ t["W_router"].T
    p = torch.softmax(z, 1)
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :k]
    kept = p.gather(1, idx)
    tot = kept.sum(1, keepdim=True)
    w = kept / tot
    F = torch.bincount(idx[:, 0], minlength=N).double() / T
    out = dict(topk_idx=idx.to(torch.int32), topk_w=w, aux_loss=(0.01 * N * (F * p.mean(0)).sum()).reshape(1),
               counts=torch.bincount(idx.reshape(-1), minlength=N).to(torch.int32))
    G, U = x @ t["W_gate"].T, x @ t["W_up"].T
    y = torch.zeros_like(x)
    if back:
        dx = torch.zeros_like(x)
        dw = torch.zeros_like(w)
        sums_g, sums_u = torch.zeros_like(G), torch.zeros_like(G)
        grad = {n: torch.zeros_like(t[n]) for n in BLOCK + (B.DORA_FIELDS if mag else ())}
    for e in range(N):
        rows, slot = (idx == e).nonzero(as_tuple=True)
        if not len(rows):
            continue
        xe, we = x[rows], w[rows, slot][:, None]
        v = _expert(t, e, xe, G[rows], U[rows], s, mag)
        A, Bm, c = v["A"], v["B"], v["c"]
        o = c["down"] * v["vd"]
        y.index_add_(0, rows, we * o)
        if not back:
            continue
        dye = t["dy"][rows]
        dw[rows, slot] = (dye * o).sum(1)
        do = we * dye
        dvd = c["down"] * do
        grad["B_down"][e] = s * dvd.T @ v["q"]
        vb = dvd @ Bm["down"]
        grad["A_down"][e] = s * vb.T @ v["a"]
        da = dvd @ t["W_down"] + s * vb @ A["down"]
        dg = da * v["u"] * v["sg"] * (1 + v["g"] * (1 - v["sg"]))
        du = da * v["g"] * v["sg"]
        if mag:
            for n, val in (("gate", dg * v["vg"]), ("up", du * v["vu"]), ("down", do * v["vd"])):
                term = val.sum(0) / c["n_" + n]
                m = grad["m_" + n]
                if m.dim() == 2:
                    m[e] = term
                else:
                    m += term
        dg, du = c["gate"] * dg, c["up"] * du
        grad["B_gate"][e], grad["B_up"][e] = s * dg.T @ v["pg"], s * du.T @ v["pu"]
        tg, tu = dg @ Bm["gate"], du @ Bm["up"]
        grad["A_gate"][e], grad["A_up"][e] = s * tg.T @ xe, s * tu.T @ xe
        sums_g.index_add_(0, rows, dg)
        sums_u.index_add_(0, rows, du)
        dx.index_add_(0, rows, s * (tg @ A["gate"] + tu @ A["up"]))
    out["y"] = y
    if back:
        dx += sums_g @ t["W_gate"] + sums_u @ t["W_up"]
        dp = torch.zeros_like(p).scatter_(1, idx, (dw - (w * dw).sum(1, keepdim=True)) / tot)
        dp += 0.01 * N * F / T
        dz = p * (dp - (p * dp).sum(1, keepdim=True))
        grad["W_router"] = dz.T @ x
        out["dx"] = dx + dz @ t["W_router"]
        out.update({"d" + n: v for n, v in grad.items()})
    return out


def exact(case, seed):
    t = {n: v.double() if v.is_floating_point() else v for n, v in _inputs(case, seed).items()}
    if case["kind"] == "adamw":
        out, h = {}, ADAMW
        h = {n: torch.tensor(v, dtype=torch.float32).item() if n != "step" else v for n, v in h.items()}
        for n in BLOCK:
            g = t["g_" + n]
            m = h["beta1"] * t["m_" + n] + (1 - h["beta1"]) * g
            v = h["beta2"] * t["v_" + n] + (1 - h["beta2"]) * g * g
            upd = (m / (1 - h["beta1"] ** h["step"])) / ((v / (1 - h["beta2"] ** h["step"])).sqrt() + h["eps"])
            p = t["p_" + n] * (1 - h["lr"] * h["weight_decay"]) - h["lr"] * upd
            out.update({"p_" + n: p, "m_" + n: m, "v_" + n: v, "lowp_" + n: p})
        return out
    if case["kind"].startswith("linear"):
        s = _scale(case)
        x, W, A, Bm, dy = (t[n] for n in ("x", "W", "A", "B", "dy"))
        out = {"y": x @ W.T + s * (x @ A.T) @ Bm.T}
        if case["kind"] == "linear_train":
            v = dy @ Bm
            out.update(dx=dy @ W + s * v @ A, dA=s * v.T @ x, dB=s * dy.T @ (x @ A.T))
        return out
    if case["kind"] != "multi":
        return _exact_block(case, t)
    N, M = case["N"], case["M"]
    parts, rows = [], [(t["token_model"] == m).nonzero()[:, 0] for m in range(M)]
    for m in range(M):
        own = {n: t[n] for n in FROZEN}
        own.update({n: t[n][m * N:(m + 1) * N] for n in BLOCK})
        own.update(x=t["x"][rows[m]], dy=t["dy"][rows[m]])
        parts.append(_exact_block(case, own))
    out = {}
    for n in parts[0]:
        cat = torch.cat([q[n] for q in parts])
        if n in ("y", "dx", "topk_idx", "topk_w"):
            back = torch.empty_like(cat)
            back[torch.cat(rows)] = cat
            cat = back
        out[n] = cat
    return out
