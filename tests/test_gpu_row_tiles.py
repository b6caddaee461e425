"""The row-segmented grouped GEMMs with few rows per expert (64- and 128-row tiles), bf16, fused order and e4m3, against float64."""
import math

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from tests.gpu_util import DEV, to_np

pytestmark = pytest.mark.gpu

# rows per expert: averages up to 32 select the 64-row tile, the others (so few tiles) the 128-row one; segments end before, on
# and after tile and 32-row block edges, experts are empty, one expert holds far more than the average
ROWS = [[1], [0, 1, 63, 64, 65, 0, 30, 33], [2] * 70, [0, 0, 0, 128], [0, 127, 128, 129, 1, 95], [300, 0, 0, 31], [33, 97],
        [700, 0, 24, 1000]]
# d, f: several k-steps with remainders, 16-column tails of the 128- and 64-wide tiles, one k-step and less, contractions long
# enough to be cut into parts (bf16 from 2560 elements on with the 128-row tile, 1024 with the 64-row one)
DIMS = [(272, 336), (512, 128), (16, 48), (144, 2752)]
# averages from 96 rows on: 128-row tiles, two workgroups per CU, in FC1 (both), dgrad2 (the second) and the weight gradients
# (the first); segments end before, on and after tile edges, the tiles fill less and more than one per CU
PAIR_ROWS = [[129, 0, 300, 128, 127], [255, 257, 1, 128, 100, 0, 64], [1000]]
PAIR_DIMS = [(272, 336), (144, 4240)]
STEP = 2.0 ** -9            # one bf16 rounding
# rows past the last segment (an expert-parallel share is given the bound T * k): the tile is chosen for all of them, the
# buffers hold NaN there before the call, outputs keep what they held
SPARE = [([0, 1, 63, 64, 65, 0, 30, 33], 300), ([33, 97], 1), ([2] * 70, 4000), ([129, 0, 5], 2000)]


def rel(got, ref):
    n = float(ref.norm())
    return float((got.double() - ref).norm()) / (n if n > 0 else 1.0)


def setup(rows, d, f, spare=0):
    E, n = len(rows), sum(rows)
    M = n + spare
    g = torch.Generator(device=DEV).manual_seed(M * 7 + d)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    off = [sum(rows[:e]) for e in range(E + 1)]
    offsets = torch.tensor(off, dtype=torch.int32, device=DEV)
    w1, w2 = rnd(E, 2 * f, d) / math.sqrt(d), rnd(E, d, f) / math.sqrt(f)
    x, dy = rnd(M, d).bfloat16(), rnd(M, d).bfloat16()
    x[n:], dy[n:] = math.nan, math.nan
    return E, M, off, offsets, w1.bfloat16(), w2.bfloat16(), x, dy


def swiglu_bwd(H, dA, f):
    G, U = H[:, :f], H[:, f:]
    s = torch.sigmoid(G)
    return G * s * U, torch.cat([dA * U * s * (1 + G * (1 - s)), dA * G * s], 1)


@pytest.mark.parametrize("d,f", DIMS)
@pytest.mark.parametrize("rows", ROWS)
def test_bf16_and_fused(rows, d, f):
    check_bf16_and_fused(rows, d, f, 0)


@pytest.mark.parametrize("d,f", PAIR_DIMS)
@pytest.mark.parametrize("rows", PAIR_ROWS)
def test_bf16_and_fused_in_pairs(rows, d, f):
    check_bf16_and_fused(rows, d, f, 0)


@pytest.mark.parametrize("rows,spare", SPARE)
def test_bf16_and_fused_below_the_bound(rows, spare):
    check_bf16_and_fused(rows, 272, 336, spare)


def test_bf16_and_fused_in_many_rounds():
    """Six and more rounds of 256 x 256 tiles (FC1, d_w1): segments of no, one and two steps of contraction, and with a remainder."""
    check_bf16_and_fused([0, 3, 700, 64, 2500, 65, 3668, 1000], 1040, 6160, 0)


def test_equal_tiles_get_equal_bits():
    """On 256 x 256 tiles FC1 and the weight gradients add their products in the order of the contraction, whichever workgroup has the tile:
    experts that hold the same rows and weights get the same bits.  Seven rounds of tiles and more, and no expert's tiles are a multiple of
    the 32 workgroups of an XCD, so that other workgroups get the next expert's."""
    from paper_2505_11432_amd import binding as B
    E, n, d, f = 8, 512, 4096, 10368
    M = E * n
    g = torch.Generator(device=DEV).manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)
    same = lambda t: t.expand(E, *t.shape).contiguous()
    x, dy, w1, w2 = same(rnd(n, d)).view(M, d), same(rnd(n, d)).view(M, d), same(rnd(2 * f, d) / 64), same(rnd(d, f) / 101)
    offsets = torch.arange(E + 1, dtype=torch.int32, device=DEV) * n
    bf = dict(dtype=torch.bfloat16, device=DEV)
    h, yp, dxp = torch.empty((M, 2 * f), **bf), torch.empty((M, d), **bf), torch.empty((M, d), **bf)
    dw1, dw2 = torch.empty((E, 2 * f, d), device=DEV), torch.empty((E, d, f), device=DEV)
    ws = torch.empty(B.moe_workspace_bytes(M, d, E, 1, f, B.BF16), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(x, None, offsets, w1, None, w2, None, h, yp, None, ws)
    B.moe_expert_ffn_bwd(x, h, dy, None, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    for name, t in (("h", h.view(E, n, 2 * f)), ("d_w1", dw1), ("d_w2", dw2)):
        for e in range(1, E):
            assert torch.equal(t[e], t[0]), (name, e)


def check_bf16_and_fused(rows, d, f, spare):
    from paper_2505_11432_amd import binding as B
    E, M, off, offsets, w1, w2, x, dy = setup(rows, d, f, spare)
    n = sum(rows)
    bf = dict(dtype=torch.bfloat16, device=DEV)
    h, yp, dxp = torch.full((M, 2 * f), 7.0, **bf), torch.full((M, d), 7.0, **bf), torch.full((M, d), 7.0, **bf)
    dw1, dw2 = torch.empty((E, 2 * f, d), device=DEV), torch.empty((E, d, f), device=DEV)
    ws = torch.empty(B.moe_workspace_bytes(M, d, E, 1, f, B.BF16), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(x, None, offsets, w1, None, w2, None, h, yp, None, ws)
    B.moe_expert_ffn_bwd(x, h, dy, None, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    # the fused order on the same rows: top-1, rows in a shuffled token order, weights in (0, 1)
    g = torch.Generator(device=DEV).manual_seed(5)
    tok = torch.randperm(M, generator=g, device=DEV)
    wt = torch.rand((M, 1), generator=g, device=DEV) + 0.1
    xt, dyt, inv = torch.empty_like(x), torch.empty_like(dy), torch.empty((M,), dtype=torch.int32, device=DEV)
    xt[tok], dyt[tok] = x, dy
    inv[tok] = torch.arange(M, dtype=torch.int32, device=DEV)
    inv[tok[n:]] = -1                                   # tokens without a row
    row_w = wt.view(-1)[tok].contiguous()
    hf, yf, dxf = torch.full_like(h, 7.0), torch.full_like(yp, 7.0), torch.full_like(dxp, 7.0)
    fw1, fw2, fdw = torch.empty_like(dw1), torch.empty_like(dw2), torch.empty((M, 1), device=DEV)
    fws = torch.empty(B.moe_expert_ffn_fused_workspace_bytes(M, 1, d, f), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fused_fwd(xt, tok.int(), row_w, offsets, w1, w2, 1, hf, yf, fws)
    B.moe_expert_ffn_fused_bwd(xt, dyt, hf, inv, wt, row_w, offsets, w1, w2, 1, dxf, fw1, fw2, 0, fdw, fws)
    H, Y, DX = (torch.zeros(s, dtype=torch.float64, device=DEV) for s in ((M, 2 * f), (M, d), (M, d)))
    DW1, DW2, DWT = torch.zeros_like(dw1).double(), torch.zeros_like(dw2).double(), torch.zeros(M, dtype=torch.float64, device=DEV)
    FW1, FW2 = torch.zeros_like(DW1), torch.zeros_like(DW2)
    for e in range(E):
        s = slice(off[e], off[e + 1])
        X, DY, a, b, w = x[s].double(), dy[s].double(), w1[e].double(), w2[e].double(), row_w[s].double()[:, None]
        H[s] = X @ a.t()
        dA = DY @ b
        A, dH = swiglu_bwd(H[s], dA, f)
        Y[s], DX[s] = A @ b.t(), dH @ a
        DWT[s] = (dA * A).sum(1)
        DW1[e], DW2[e] = dH.t() @ X, DY.t() @ A
        FW1[e], FW2[e] = dH.t() @ (w * X), DY.t() @ (w * A)
    # a result carries at most four stored bf16 roundings on its way (H, A or dA, dH, itself)
    assert torch.equal(h, hf)
    for name, got, ref in (("h", h, H), ("yp", yp, Y), ("d_xp", dxp, DX), ("ypw", yf, Y * row_w.double()[:, None]), ("fused d_xp", dxf, DX)):
        assert rel(got[:n], ref[:n]) < 4 * STEP, (name, rel(got[:n], ref[:n]))
        assert bool((got[n:] == 7.0).all()), name
    # (the fused order's d_w1: its weighted rows carry one more rounding)
    for name, got, ref in (("d_w1", dw1, DW1), ("d_w2", dw2, DW2), ("fused d_w1", fw1, FW1), ("fused d_w2", fw2, FW2)):
        assert rel(got, ref) < 4 * STEP, (name, rel(got, ref))
    # a dot product of f terms of random sign, each with the roundings of dA and of H
    assert rel(fdw.view(-1)[tok[:n]], DWT[:n]) < 4 * STEP
    assert not fdw.view(-1)[tok[n:]].any()


@pytest.mark.parametrize("d,f", DIMS)
@pytest.mark.parametrize("rows", ROWS)
def test_e4m3(rows, d, f):
    check_e4m3(rows, d, f, 0)


@pytest.mark.parametrize("d,f", PAIR_DIMS)
@pytest.mark.parametrize("rows", PAIR_ROWS)
def test_e4m3_in_pairs(rows, d, f):
    check_e4m3(rows, d, f, 0)


@pytest.mark.parametrize("rows,spare", SPARE)
def test_e4m3_below_the_bound(rows, spare):
    check_e4m3(rows, 272, 336, spare)


@pytest.mark.parametrize("d,f", [(1040, 6160), (2048, 8192)])
def test_e4m3_in_groups(d, f):
    """Workgroups that start in groups and walk the contraction from different steps on: eight of them in FC1, four (first) and eight in
    d_w1; segments of no, one and a few steps, fewer than the groups lie apart, and with a remainder."""
    check_e4m3([0, 3, 700, 64, 2500, 65, 3668, 1000], d, f, 0)


def check_e4m3(rows, d, f, spare):
    from paper_2505_11432_amd import binding as B
    E, M, off, offsets, w1, w2, x, dy = setup(rows, d, f, spare)
    used = sum(rows)
    u8, bf = dict(dtype=torch.uint8, device=DEV), dict(dtype=torch.bfloat16, device=DEV)

    def q(t):
        v = t.reshape(-1, t.shape[-1]).contiguous()
        c, s = torch.empty(v.shape, **u8), torch.empty((v.shape[0],), device=DEV)
        B.moe_quant_fp8(v, B.Q_ROW, c, s)
        return c.view(t.shape), s.view(t.shape[:-1])

    deq = lambda c, s: c.view(torch.float8_e4m3fn).double() * s.double()[..., None]
    (xc, xs), (c1, s1), (c2, s2) = q(x), q(w1), q(w2)
    (t1, ts1), (t2, ts2) = q(w1.transpose(1, 2).contiguous()), q(w2.transpose(1, 2).contiguous())
    h, yp, dxp = torch.full((M, 2 * f), 7.0, **bf), torch.full((M, d), 7.0, **bf), torch.full((M, d), 7.0, **bf)
    ac, asc = torch.empty((M, f), **u8), torch.empty((M,), device=DEV)
    ws = torch.empty(B.moe_workspace_bytes(M, d, E, 1, f, B.F8E4M3), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(xc, xs, offsets, c1, s1, c2, s2, h, yp, None, ws, ac, asc)
    ldt = B.moe_tgroup_tokens(M, E)
    f32 = dict(device=DEV)
    it = dict(dy_codes=torch.empty((M, d), **u8), dy_scale=torch.empty((M,), **f32), dh=torch.empty((M, 2 * f), **bf),
              dh_codes=torch.empty((M, 2 * f), **u8), dh_scale=torch.empty((M,), **f32),
              pad_offsets=torch.empty((E + 1,), dtype=torch.int32, device=DEV), splitk_ws=torch.empty((B.SPLITK_WS_BYTES,), **u8))
    for n, c in (("dy", d), ("dh", 2 * f), ("a", f), ("x", d)):
        it[n + "_t"], it[n + "_e8m0"] = torch.empty((c, ldt), **u8), torch.empty((ldt // 128, c), **u8)
    dw1, dw2 = torch.empty((E, 2 * f, d), **f32), torch.empty((E, d, f), **f32)
    B.moe_expert_ffn_bwd_fp8(dy, h, (xc, xs), (ac, asc), offsets, t1, ts1, t2, ts2, dxp, dw1, dw2, 0, it)
    # every stage from the codes the kernels themselves read: one stored rounding per result (dH: dA as well)
    X, A, DY, DH = deq(xc, xs), deq(ac, asc), deq(it["dy_codes"], it["dy_scale"]), deq(it["dh_codes"], it["dh_scale"])
    W1, W2, T1, T2 = deq(c1, s1), deq(c2, s2), deq(t1, ts1), deq(t2, ts2)
    for e in range(E):
        s = slice(off[e], off[e + 1])
        if off[e] == off[e + 1]:
            continue
        ref_dh = swiglu_bwd(h[s].double(), DY[s] @ T2[e].t(), f)[1]
        for name, got, ref in (("h", h[s], X[s] @ W1[e].t()), ("yp", yp[s], A[s] @ W2[e].t()), ("dh", it["dh"][s], ref_dh),
                               ("d_xp", dxp[s], DH[s] @ T1[e].t())):
            assert rel(got, ref) < 2 * STEP, (name, e, rel(got, ref))
    for name, got in (("h", h), ("yp", yp), ("d_xp", dxp)):
        assert bool((got[used:] == 7.0).all()), name
    # the operands of the weight gradients: transposed codes of 128-token groups, the forward's from its row codes (the
    # value a code stands for, rounded once to fp32), bit for bit
    from tests.test_gpu_parity import _check_tgroup
    I = {k: to_np(it[k]) for k in ("a_t", "a_e8m0", "x_t", "x_e8m0", "pad_offsets")}
    for name, c, sc in (("a", ac, asc), ("x", xc, xs)):
        v = O.e4m3_decode(to_np(c[:used])).astype(np.float32) * to_np(sc[:used]).astype(np.float32)[:, None]
        _check_tgroup(I[name + "_t"], I[name + "_e8m0"], I["pad_offsets"], v, np.array(off))
    # and the weight gradients from them.  The e4m3 matrix instruction adds its 64 products aligned to the largest one, not
    # each in full fp32 (3.8e-5 of the norm seen with 63 rows): at 2^-16 of the largest per product that is 2^-10 of it, and
    # one bf16 rounding, the bar of the other results, is above it
    po = I["pad_offsets"]
    for name, got, p, q in (("d_w1", dw1, "dh", "x"), ("d_w2", dw2, "dy", "a")):
        for e in range(E):
            s = slice(int(po[e]), int(po[e]) + rows[e])
            P, Q = ((it[t + "_t"][:, s].view(torch.float8_e4m3fn).double() *
                     torch.exp2(it[t + "_e8m0"].double() - 127).repeat_interleave(128, 0)[s].t()) for t in (p, q))
            assert rel(got[e], P @ Q.t()) < STEP, (name, e, rel(got[e], P @ Q.t()))
