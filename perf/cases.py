"""The timed workloads of the MoE expert-FFN path: what is measured, on which inputs, against which reference.

Every case goes through the public entry points (`MoELayer` and the calls of `binding`).  The layer shapes are the ones
of this repository's benchmark and tests (synth/moe_inputs.py: the Mixtral, fine-grained, skewed and expert-parallel
layers and the tiny fp32 layer) plus generic odd ones; inputs follow the same recipe (N(0,1) tokens and output gradients,
expert weights of std 0.02 or 1/sqrt(d), router weights and per-expert bias that shape the load).

kinds
  forward   forward of one layer (serving, evaluation): few to a few thousand tokens
  train     forward and backward of one layer (one micro-batch of a training step)
  route     gate and row map from given logits, and the gate's backward
  rows      the row movers of the communication path: dispatch, weighted dispatch, combine, gate gradient
  cast      the E4M3 cast of the communication compression, both directions and both groupings

`exact` restates the layer in plain torch with float64 products; nothing of the package is used there.
"""
from __future__ import annotations

import math

import torch

DEV = "cuda:0"
E4M3_MAX = 448.0

# order: "plain" = dispatched copies; "fused" = row selection inside FC1 and the gate weight after SwiGLU;
#        "keep_a" = plain, with the FC2 input kept from the forward.
# bwd8 (dtype "fp8"): 1 = the backward GEMMs on e4m3 operands as well, 0 = bf16 backward (straight-through casts)
_LAYER = dict(dtype="bf16", order="plain", renorm=1, bias="none", gamma=0.0, w_std=0.02, lo=-1, hi=-1, devices=0,
              capacity_factor=0.0, alpha=0.0, bwd8=0)


def _layer(name, kind, T, d, E, k, f, **kw):
    c = dict(name=name, kind=kind, T=T, d=d, E=E, k=k, f=f, wr_std=1.0 / math.sqrt(d), **_LAYER)
    c.update(kw)
    return c


def listed():
    return [
        # a serving step: a handful of tokens in flight, every expert's weights read for a few rows each
        _layer("forward_16_tokens", "forward", 16, 4096, 8, 2, 14336, wr_std=0.02),
        # a small evaluation batch through many narrow experts (odd token count, 32 rows per expert on average)
        _layer("forward_fine_257_tokens", "forward", 257, 2048, 64, 8, 1408, bias="linear", gamma=0.17),
        # the correctness layer that tests and new users start with: launches, not arithmetic
        _layer("train_f32_tiny", "train", 256, 128, 8, 2, 256, dtype="f32", w_std=1.0 / math.sqrt(128), wr_std=0.02),
        # a single-precision layer of ordinary size (reference runs, small models trained in fp32)
        _layer("train_f32_1000_tokens", "train", 1000, 1024, 8, 2, 2816, dtype="f32"),
        # a micro-batch of odd sizes (nothing a multiple of a tile) with token dropping and the balance loss
        _layer("train_ragged_capacity", "train", 1531, 1040, 24, 3, 1424, bias="linear", gamma=0.3, devices=8,
               capacity_factor=1.1, alpha=0.01),
        # the headline layer of bench.py
        _layer("train_mixtral", "train", 8192, 4096, 8, 2, 14336, wr_std=0.02),
        # fine-grained experts: many ragged segments, large row buffers
        _layer("train_finegrained", "train", 16384, 2048, 64, 8, 1408, bias="linear", gamma=0.17),
        # one GPU's share of an expert-parallel layer: all-gathered tokens, four local experts of 32
        _layer("train_ep_share_fused", "train", 8192, 4096, 32, 3, 14336, order="fused", lo=8, hi=12),
        # FP8 training of the headline layer: e4m3 activations, weights and gradients in all six expert GEMMs
        _layer("train_mixtral_fp8", "train", 8192, 4096, 8, 2, 14336, dtype="fp8", wr_std=0.02, bwd8=1),
        # gating alone, as the overlap of communication and computation calls it ahead of the expert work
        dict(name="route_4096_tokens", kind="route", T=4096, E=64, k=8, renorm=1, quantum=0.0),
        # the row movers on buffers larger than the last-level cache
        dict(name="rows_finegrained", kind="rows", T=16384, d=2048, E=64, k=8, dtype="bf16"),
        # communication compression of one micro-batch: activations per token, gradients per channel and 128 tokens
        dict(name="cast_8192_tokens", kind="cast", rows=8192, cols=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _log16(rng, lo, hi):
    return max(1, _log_int(rng, lo // 16, hi // 16)) * 16


def draw(rng):
    kind = rng.choice(["forward", "forward", "train", "train", "train", "train_f32", "train_fp8", "route", "rows", "cast"])
    if kind == "route":
        E = rng.choice([8, 12, 16, 32, 64, 100, 160, 256])
        return dict(kind="route", T=_log_int(rng, 16, 65536), E=E, k=rng.randint(1, min(8, E)), renorm=rng.randint(0, 1),
                    quantum=rng.choice([0.0, 0.0, 0.25]))
    if kind == "cast":
        return dict(kind="cast", rows=_log_int(rng, 64, 16384), cols=_log16(rng, 256, 8192))
    if kind == "rows":
        E = rng.choice([8, 16, 64])
        return dict(kind="rows", T=_log_int(rng, 64, 16384), d=_log16(rng, 256, 4096), E=E, k=rng.randint(1, min(8, E)),
                    dtype=rng.choice(["bf16", "bf16", "f32"]))
    if kind == "train_f32":
        E = rng.choice([4, 6, 8, 16])
        return _layer(None, "train", _log_int(rng, 64, 1500), _log16(rng, 128, 1024), E, rng.randint(1, 3),
                      _log16(rng, 128, 2816), dtype="f32", renorm=rng.randint(0, 1)) | {"name": "drawn"}
    T = _log_int(rng, 1, 1024) if kind == "forward" else _log_int(rng, 64, 16384)
    d, f = _log16(rng, 256, 4096), _log16(rng, 256, 14336)
    E = rng.choice([4, 8, 12, 16, 32, 64])
    k = rng.randint(1, min(8, E))
    while E > 4 and E * d * f > 8 * 4096 * 14336:            # no more weights than the headline layer holds
        E //= 2
    k = min(k, E)
    while T > 64 and T * k * d * f > 8192 * 2 * 4096 * 14336 // 2:
        T = T // 2 + 1
    kw = dict(renorm=rng.randint(0, 1), bias=rng.choice(["none", "linear", "zipf"]))
    kw["gamma"] = {"none": 0.0, "linear": 0.3, "zipf": 0.8}[kw["bias"]]
    if kind == "train_fp8":
        kw.update(dtype="fp8", bwd8=rng.randint(0, 1))
    else:
        kw["order"] = rng.choice(["plain", "plain", "fused", "keep_a"])
        extra = rng.choice(["none", "none", "range", "capacity", "balance"])
        if extra == "range" and E >= 8:
            kw.update(lo=E // 4, hi=E // 2)
        elif extra == "capacity":
            kw.update(devices=4, capacity_factor=1.1)
        elif extra == "balance":
            kw.update(devices=4, alpha=0.01)
    return _layer("drawn", "forward" if kind == "forward" else "train", T, d, E, k, f, **kw)


# ---- inputs ---------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)


def _randn(g, shape, std, dtype):
    t = torch.randn(shape, generator=g, device=DEV, dtype=dtype)
    return t.mul_(std) if std != 1.0 else t


def _router_bias(case, g):
    E = case["E"]
    if case["bias"] == "none":
        return None
    order = torch.randperm(E, generator=g, device=DEV)
    if case["bias"] == "linear":
        u = torch.linspace(1.0, -1.0, E, device=DEV)
        return (case["gamma"] * u[order]).contiguous()
    return (-case["gamma"] * torch.log(1.0 + order.float())).contiguous()


def _layer_inputs(case, seed):
    g = _gen(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    T, d, E, f = case["T"], case["d"], case["E"], case["f"]
    n = E if case["lo"] < 0 else case["hi"] - case["lo"]
    inp = {"x": _randn(g, (T, d), 1.0, dt), "dy": _randn(g, (T, d), 1.0, dt),
           "w_r": _randn(g, (E, d), case["wr_std"], dt), "bias": _router_bias(case, g)}
    inp["w1"] = _randn(g, (n, 2 * f, d), case["w_std"], dt)
    inp["w2"] = _randn(g, (n, d, f), case["w_std"], dt)
    return inp


def _capacity(case):
    return int(math.ceil(case["capacity_factor"] * case["T"] * case["k"] / case["devices"]))


def _logits(case, seed):
    z = torch.randn((case["T"], case["E"]), generator=_gen(seed), device=DEV)
    if case["quantum"]:
        z = (torch.round(z / case["quantum"]) * case["quantum"]).contiguous()    # a coarse grid: many equal logits
    return z


def _d_topk(case, seed):
    return torch.randn((case["T"], case["k"]), generator=_gen(seed + 1), device=DEV)


def _rows_inputs(case, seed):
    g = _gen(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    T, d, E, k = case["T"], case["d"], case["E"], case["k"]
    idx = torch.rand((T, E), generator=g, device=DEV).argsort(dim=1)[:, :k].contiguous()
    order = torch.sort(idx.view(-1), stable=True).indices
    inv_perm = torch.empty((T * k,), dtype=torch.int32, device=DEV)
    inv_perm[order] = torch.arange(T * k, dtype=torch.int32, device=DEV)
    w = torch.rand((T, k), generator=g, device=DEV) + 0.1
    return {"x": _randn(g, (T, d), 1.0, dt), "dy": _randn(g, (T, d), 1.0, dt), "yp": _randn(g, (T * k, d), 1.0, dt),
            "w": (w / w.sum(dim=1, keepdim=True)).contiguous(), "inv_perm": inv_perm}


def _cast_inputs(case, seed):
    g = _gen(seed)
    shape = (case["rows"], case["cols"])
    return _randn(g, shape, 1.0, torch.bfloat16), _randn(g, shape, 1e-3, torch.bfloat16)


# ---- what a program holds before the call -------------------------------------------------------------------------
def prepare(case, seed):
    from paper_2505_11432_amd import binding as B
    kind = case["kind"]
    i32 = dict(dtype=torch.int32, device=DEV)
    if kind == "route":
        T, E, k = case["T"], case["E"], case["k"]
        return {"case": case, "logits": _logits(case, seed), "dw": _d_topk(case, seed),
                "idx": torch.empty((T, k), **i32), "w": torch.empty((T, k), device=DEV),
                "counts": torch.empty((E,), **i32), "offsets": torch.empty((E + 1,), **i32),
                "perm": torch.empty((T * k,), **i32), "inv_perm": torch.empty((T * k,), **i32),
                "d_logits": torch.empty((T, E), device=DEV),
                "ws": torch.empty((max(B.moe_workspace_bytes(T, 16, E, k, 16, B.BF16), 256),), dtype=torch.uint8, device=DEV)}
    if kind == "rows":
        st = _rows_inputs(case, seed)
        st.update(case=case, xp=torch.empty_like(st["yp"]), dyp=torch.empty_like(st["yp"]), y=torch.empty_like(st["x"]),
                  dx=torch.empty_like(st["x"]), dw=torch.empty_like(st["w"]))
        return st
    if kind == "cast":
        x, dy = _cast_inputs(case, seed)
        r, c = case["rows"], case["cols"]
        u8 = dict(dtype=torch.uint8, device=DEV)
        return {"case": case, "x": x, "dy": dy,
                "xc": torch.empty((r, c), **u8), "xs": torch.empty((r,), device=DEV), "xd": torch.empty_like(x),
                "gc": torch.empty((r, c), **u8), "gs": torch.empty(((r + 127) // 128, c), device=DEV),
                "gd": torch.empty_like(dy)}
    from paper_2505_11432_amd.layer import MoELayer
    st = _layer_inputs(case, seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    fp8 = case["dtype"] == "fp8"
    layer = MoELayer(case["T"], case["d"], case["E"], case["k"], case["f"], dtype=dt, renorm=case["renorm"], fp8=fp8,
                     expert_range=None if case["lo"] < 0 else (case["lo"], case["hi"]),
                     capacity=(case["devices"], _capacity(case)) if case["capacity_factor"] > 0 else None,
                     balance=(case["devices"], case["alpha"]) if case["alpha"] > 0 else None,
                     fused=case["order"] == "fused", keep_a=case["order"] == "keep_a")
    if fp8:
        layer.set_fp8_weights(st["w1"], st["w2"])
        if case["bwd8"]:
            layer.set_fp8_backward_weights(st["w1"], st["w2"])
    st.update(case=case, layer=layer)
    return st


def run(st):
    from paper_2505_11432_amd import binding as B
    case = st["case"]
    kind = case["kind"]
    if kind == "route":
        B.moe_route(st["logits"], case["k"], case["renorm"], st["idx"], st["w"], st["counts"], st["offsets"], st["perm"],
                    st["inv_perm"], st["ws"])
        B.moe_route_bwd(st["logits"], st["idx"], st["w"], st["dw"], case["E"], case["renorm"], st["d_logits"])
        return {n: st[n] for n in ("idx", "w", "counts", "offsets", "perm", "inv_perm", "d_logits")}
    if kind == "rows":
        k = case["k"]
        B.moe_dispatch(st["x"], None, st["inv_perm"], None, k, st["xp"], None)
        B.moe_combine(st["yp"], None, st["inv_perm"], st["w"], k, st["y"])
        B.moe_gate_grad(st["dy"], st["yp"], None, st["inv_perm"], k, st["dw"])
        B.moe_dispatch(st["dy"], None, st["inv_perm"], st["w"].view(-1), k, st["dyp"], None)
        B.moe_combine(st["yp"], None, st["inv_perm"], None, k, st["dx"])
        return {n: st[n] for n in ("xp", "y", "dw", "dyp", "dx")}
    if kind == "cast":
        B.moe_quant_fp8(st["x"], B.Q_ROW, st["xc"], st["xs"])
        B.moe_dequant_fp8(st["xc"], st["xs"], B.Q_ROW, st["xd"])
        B.moe_quant_fp8(st["dy"], B.Q_COLGROUP128, st["gc"], st["gs"])
        B.moe_dequant_fp8(st["gc"], st["gs"], B.Q_COLGROUP128, st["gd"])
        return {n: st[n] for n in ("xc", "xs", "xd", "gc", "gs", "gd")}
    layer = st["layer"]
    x, w_r, bias, w1, w2, dy = (st[n] for n in ("x", "w_r", "bias", "w1", "w2", "dy"))
    if case["dtype"] == "fp8":
        layer.forward_fp8(x, w_r, bias)
        if case["bwd8"]:
            layer.backward_fp8_gemm(x, w_r, dy)
        else:
            layer.backward_fp8(x, w_r, w1, w2, dy)
    else:
        layer.forward(x, w_r, bias, w1, w2)
        if kind == "train":
            layer.backward(x, w_r, w1, w2, dy)
    out = {"logits": layer.logits, "y": layer.y}
    if kind == "train":
        out.update(dx=layer.dx, d_w1=layer.d_w1, d_w2=layer.d_w2, d_w_r=layer.d_w_r)
    if case["alpha"] > 0:
        out["aux_loss"] = layer.aux_loss
    return out


# ---- what one pass cannot do without --------------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "route":
        T, E, k = case["T"], case["E"], case["k"]
        # logits in, idx / w / perm / inv_perm out; backward: d_w in, d_logits out
        return {"bytes": 4.0 * (2 * T * E + 5 * T * k + 2 * E), "flops": float(T * E)}
    if kind == "rows":
        T, d, k = case["T"], case["d"], case["k"]
        es = 4 if case["dtype"] == "f32" else 2
        # x, dy, yp in; xp, dyp, y, dx out
        return {"bytes": es * float(4 * T * d + 3 * T * k * d), "flops": 8.0 * T * k * d}
    if kind == "cast":
        n = float(case["rows"]) * case["cols"]
        return {"bytes": 2 * n * (2 + 1 + 2), "flops": 4 * n}          # bf16 in, codes and bf16 out, twice
    T, d, E, k, f = (case[n] for n in ("T", "d", "E", "k", "f"))
    share = 1.0 if case["lo"] < 0 else (case["hi"] - case["lo"]) / E
    n_local = E * share
    rows = T * k * share
    es = 4 if case["dtype"] == "f32" else 2
    wes = 1 if case["dtype"] == "fp8" else es
    touched = n_local * (1.0 - (1.0 - k / E) ** T)                     # experts that get a row
    weights = touched * 3.0 * d * f
    flops = 6.0 * rows * d * f + 2.0 * T * d * E
    nbytes = weights * wes + 2.0 * T * d * es + E * d * es
    if kind == "train":
        flops *= 3
        # the weights again for the backward (e4m3 backward: their transposed copies; straight-through: bf16 masters)
        if case["dtype"] == "fp8":
            nbytes += weights * (1 if case["bwd8"] else 2)
        nbytes += n_local * 3.0 * d * f * 4 + 2.0 * T * d * es + 4.0 * E * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind == "cast":
        return "exact"
    if kind == "route":
        return {"rel": 2e-6, "differ": 0.0}          # fp32 exponentials and sums of at most 256 terms
    if kind == "rows":
        return {"rel": 1e-2 if case["dtype"] == "bf16" else 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5}          # 1.6e-6 seen
    if case["dtype"] == "bf16":
        return {"rel": 2e-2}          # bf16 storage between the GEMMs: 4.4e-3 seen
    return {"rel": 8e-2}          # a changed sum order moves codes by one step: 2.6e-2 seen against exact()


# ---- the same in float64 ----------------------------------------------------------------------------------------------
def _bf16(v):
    return v.to(torch.bfloat16).double()


def _e4m3(v32, amax32):
    """(codes as float8, scale) of fp32 values under a broadcastable amax: scale amax/448, amax = 0 gives scale 1."""
    one = torch.ones_like(amax32)
    inv = torch.where(amax32 > 0, E4M3_MAX / amax32, one)
    scale = torch.where(amax32 > 0, amax32 / E4M3_MAX, one)
    return (v32 * inv).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn), scale


def _q_row(v):
    v = v.float()
    codes, scale = _e4m3(v, v.abs().amax(dim=1, keepdim=True))
    return codes, scale


def _q_group(v):
    """One scale per column inside each group of 128 consecutive rows."""
    v = v.float()
    r, c = v.shape
    groups = (r + 127) // 128
    pad = torch.zeros((groups * 128, c), device=v.device)
    pad[:r] = v
    codes, scale = _e4m3(pad.view(groups, 128, c), pad.view(groups, 128, c).abs().amax(dim=1, keepdim=True))
    return codes.view(groups * 128, c)[:r], scale.view(groups, c)


def _deq_row(v):
    codes, scale = _q_row(v)
    return codes.double() * scale.double()


def _deq_group(v):
    codes, scale = _q_group(v)
    return codes.double() * scale.double().repeat_interleave(128, dim=0)[: v.shape[0]]


def _deq_group_pow2(v):
    """Groups of 128 rows with the smallest power-of-two scale that keeps the group inside +-448."""
    v = v.float()
    r, c = v.shape
    groups = (r + 127) // 128
    pad = torch.zeros((groups * 128, c), device=v.device)
    pad[:r] = v
    pad = pad.view(groups, 128, c)
    amax = pad.abs().amax(dim=1, keepdim=True)
    m, ex = torch.frexp(amax)                                          # amax = m * 2^ex, m in [0.5, 1)
    kk = torch.where(amax > 0, ex - 9 + (m > 0.875).int(), torch.zeros_like(ex)).clamp(-126, 127)
    s = torch.exp2(kk.float())
    codes = (pad / s).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn).double()
    return (codes * s.double()).view(groups * 128, c)[:r]


def _gate(z, k, renorm):
    idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :k]
    sel = torch.gather(z, 1, idx)
    p = torch.softmax(z, dim=1)
    return idx, (torch.softmax(sel, dim=1) if renorm else torch.gather(p, 1, idx)), p


def _gate_bwd(idx, w, p, dw, renorm):
    inner = (w * dw).sum(dim=1, keepdim=True)
    out = torch.zeros_like(p) if renorm else -p * inner
    return out.scatter_add(1, idx, (w * (dw - inner)) if renorm else w * dw)


def _exact_layer(case, seed):
    inp = _layer_inputs(case, seed)
    T, d, E, k, f = (case[n] for n in ("T", "d", "E", "k", "f"))
    lo, hi = (0, E) if case["lo"] < 0 else (case["lo"], case["hi"])
    fp8, train = case["dtype"] == "fp8", case["kind"] == "train"
    x, dy, w_r = inp["x"].double(), inp["dy"].double(), inp["w_r"].double()
    z = x @ w_r.t()
    if inp["bias"] is not None:
        z = z + inp["bias"].double()
    idx, w, p = _gate(z, k, case["renorm"])
    counts = torch.bincount(idx.reshape(-1), minlength=E).double()
    keep = (idx >= lo) & (idx < hi)
    if case["capacity_factor"] > 0:
        score, cap, per = torch.gather(p, 1, idx).reshape(-1), _capacity(case), E // case["devices"]
        dev = idx.reshape(-1) // per
        kept = torch.zeros_like(dev, dtype=torch.bool)
        for g in range(case["devices"]):
            a = torch.nonzero(dev == g).view(-1)
            kept[a[torch.sort(score[a], descending=True, stable=True).indices[:cap]]] = True
        keep = keep & kept.view(T, k)
    out = {"logits": z}
    y, dx, dw = torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(w)
    if train:
        d_w1 = torch.zeros(inp["w1"].shape, dtype=torch.float64, device=DEV)
        d_w2 = torch.zeros(inp["w2"].shape, dtype=torch.float64, device=DEV)
    xin = _deq_row(inp["x"]) if fp8 else x
    dy_in = _bf16(_deq_group(inp["dy"])) if fp8 else dy
    for e in range(lo, hi):
        t, j = torch.nonzero((idx == e) & keep, as_tuple=True)
        if t.numel() == 0:
            continue
        w1b, w2b = inp["w1"][e - lo], inp["w2"][e - lo]
        w1, w2 = (_deq_row(w1b), _deq_row(w2b)) if fp8 else (w1b.double(), w2b.double())
        X = xin[t]
        H = X @ w1.t()
        if fp8:
            H = _bf16(H)
        G, U = H[:, :f], H[:, f:]
        s = torch.sigmoid(G)
        A = G * s * U
        if fp8:
            A = _deq_row(_bf16(A))
        Y = A @ w2.t()
        if fp8:
            Y = _deq_row(_bf16(Y))
        wt = w[t, j][:, None]
        y.index_add_(0, t, wt * Y)
        if not train:
            continue
        g = dy_in[t]
        dw[t, j] = (g * Y).sum(dim=1)
        dY = wt * g
        if not fp8:
            dA = dY @ w2
            dH = torch.cat([dA * U * s * (1 + G * (1 - s)), dA * G * s], dim=1)
            d_w2[e - lo] = dY.t() @ A
            dx.index_add_(0, t, dH @ w1)
            d_w1[e - lo] = dH.t() @ X
            continue
        dY = _bf16(dY)
        if case["bwd8"]:
            dA = _bf16(_deq_row(dY) @ _deq_row(w2b.t()).t())
            dH = _bf16(torch.cat([dA * U * s * (1 + G * (1 - s)), dA * G * s], dim=1))
            d_w2[e - lo] = _deq_group_pow2(dY).t() @ _deq_group_pow2(A)
            dx.index_add_(0, t, _bf16(_deq_row(dH) @ _deq_row(w1b.t()).t()))
            d_w1[e - lo] = _deq_group_pow2(dH).t() @ _deq_group_pow2(X)
        else:
            dA = _bf16(dY @ w2b.double())
            dH = _bf16(torch.cat([dA * U * s * (1 + G * (1 - s)), dA * G * s], dim=1))
            d_w2[e - lo] = dY.t() @ _bf16(A)
            dx.index_add_(0, t, _bf16(dH @ w1b.double()))
            d_w1[e - lo] = dH.t() @ _bf16(X)
    out["y"] = y
    if train:
        dz = _gate_bwd(idx, w, p, dw, case["renorm"])
        if case["alpha"] > 0:
            dz = dz + _balance(case, p, counts)[1]
        out.update(dx=dx + dz @ w_r, d_w1=d_w1, d_w2=d_w2, d_w_r=dz.t() @ x)
    if case["alpha"] > 0:
        out["aux_loss"] = _balance(case, p, counts)[0]
    return out


def _balance(case, p, counts):
    T, E, k, n = case["T"], case["E"], case["k"], case["devices"]
    fg = (counts * (E / (k * T))).view(n, E // n).mean(dim=1)
    loss = case["alpha"] * (fg * p.mean(dim=0).view(n, E // n).sum(dim=1)).sum()
    F = fg.repeat_interleave(E // n)[None, :]
    return loss.view(1), case["alpha"] / T * p * (F - (p * F).sum(dim=1, keepdim=True))


def exact(case, seed):
    kind = case["kind"]
    if kind == "route":
        z = _logits(case, seed)
        E, k = case["E"], case["k"]
        idx = torch.sort(z, dim=1, descending=True, stable=True).indices[:, :k].contiguous()
        z = z.double()
        p = torch.softmax(z, dim=1)
        w = torch.softmax(torch.gather(z, 1, idx), dim=1) if case["renorm"] else torch.gather(p, 1, idx)
        counts = torch.bincount(idx.view(-1), minlength=E)
        perm = torch.sort(idx.view(-1), stable=True).indices
        inv_perm = torch.empty_like(perm)
        inv_perm[perm] = torch.arange(perm.numel(), device=DEV)
        offsets = torch.cat([counts.new_zeros(1), counts.cumsum(0)])
        dz = _gate_bwd(idx, w, p, _d_topk(case, seed).double(), case["renorm"])
        return {"idx": idx.int(), "w": w, "counts": counts.int(), "offsets": offsets.int(), "perm": perm.int(),
                "inv_perm": inv_perm.int(), "d_logits": dz}
    if kind == "rows":
        s = _rows_inputs(case, seed)
        T, d, k = case["T"], case["d"], case["k"]
        row = s["inv_perm"].long()
        xp = torch.empty((T * k, d), dtype=torch.float64, device=DEV)
        dyp = torch.empty_like(xp)
        xp[row] = s["x"].double().repeat_interleave(k, dim=0)
        dyp[row] = s["dy"].double().repeat_interleave(k, dim=0) * s["w"].double().view(-1, 1)
        y, dx = torch.zeros((T, d), dtype=torch.float64, device=DEV), torch.zeros((T, d), dtype=torch.float64, device=DEV)
        dw = torch.empty((T, k), dtype=torch.float64, device=DEV)
        for j in range(k):
            r = s["yp"][row.view(T, k)[:, j]].double()
            y += s["w"][:, j:j + 1].double() * r
            dx += r
            dw[:, j] = (s["dy"].double() * r).sum(dim=1)
        return {"xp": xp, "y": y, "dw": dw, "dyp": dyp, "dx": dx}
    if kind == "cast":
        x, dy = _cast_inputs(case, seed)
        xc, xs = _q_row(x)
        gc, gs = _q_group(dy)
        xd = xc.double() * xs.double()
        gd = gc.double() * gs.double().repeat_interleave(128, dim=0)[: case["rows"]]
        return {"xc": xc.view(torch.uint8), "xs": xs.view(-1), "xd": xd, "gc": gc.view(torch.uint8), "gs": gs, "gd": gd}
    return _exact_layer(case, seed)
