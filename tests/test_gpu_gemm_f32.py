"""fp32 grouped GEMMs on the matrix cores: tile edges, remainders, empty experts and the three tile shapes, against float64."""
import math

import pytest
import torch

from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

# rows per expert, d, f: segments around the 32- and 64-row tiles, widths with 16-column tails; weight gradients of few rows per expert on
# 64 x 32 (from 256 tiles of 64 x 64 on) and 64 x 64 tiles (d_w2 and d_w1 of the last, from 1024 on); the fourth takes the split products
CASES = [
    ([1, 31, 0, 32], 16, 48),
    ([33, 63, 64, 65], 144, 80),
    ([0, 0, 129, 0], 48, 272),
    ([500, 511, 0, 1049], 272, 2000),
    ([3] * 70, 64, 32),                    # more segments than lanes in a wave
    ([20, 32, 0, 33, 7, 31, 17, 20], 256, 512),
    ([20, 25, 31, 0, 40, 25, 30, 28], 512, 1408),
]


def rel(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("rows,d,f", CASES)
def test_ffn_f32_tile_edges(rows, d, f):
    from paper_2505_11432_amd import binding as B
    E, M = len(rows), sum(rows)
    g = torch.Generator(device=DEV).manual_seed(M + d)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    xp, dyp, w1, w2 = rnd(M, d), rnd(M, d), rnd(E, 2 * f, d) / math.sqrt(d), rnd(E, d, f) / math.sqrt(f)
    off = [sum(rows[:e]) for e in range(E + 1)]
    offsets = torch.tensor(off, dtype=torch.int32, device=DEV)
    h, yp, dxp = (torch.full((M, n), 7.0, device=DEV) for n in (2 * f, d, d))
    dw1, dw2 = torch.full_like(w1, 7.0), torch.full_like(w2, 7.0)
    ws = torch.empty(max(B.moe_workspace_bytes(M, d, E, 1, f, B.F32), 256), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(xp, None, offsets, w1, None, w2, None, h, yp, None, ws)
    B.moe_expert_ffn_bwd(xp, h, dyp, None, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    H, Y, DX = (torch.zeros_like(t, dtype=torch.float64) for t in (h, yp, dxp))
    DW1, DW2 = torch.zeros_like(dw1, dtype=torch.float64), torch.zeros_like(dw2, dtype=torch.float64)
    for e in range(E):
        s = slice(off[e], off[e + 1])
        X, DY, a, b = xp[s].double(), dyp[s].double(), w1[e].double(), w2[e].double()
        H[s] = X @ a.t()
        G, U = H[s, :f], H[s, f:]
        sg = torch.sigmoid(G)
        A = G * sg * U
        Y[s] = A @ b.t()
        dA = DY @ b
        dH = torch.cat([dA * U * sg * (1 + G * (1 - sg)), dA * G * sg], 1)
        DW2[e], DX[s], DW1[e] = DY.t() @ A, dH @ a, dH.t() @ X
    # three chained contractions of at most K terms, each rounding its running sum K times: sqrt(K) * 2^-24 each for
    # rounding errors of random sign, times 3 as the margin
    tol = 3 * 3 * math.sqrt(max(d, 2 * f, max(rows))) * 2.0 ** -24
    for name, got, ref in (("h", h, H), ("yp", yp, Y), ("d_xp", dxp, DX), ("d_w1", dw1, DW1), ("d_w2", dw2, DW2)):
        assert rel(got, ref) < tol, (name, rel(got, ref), tol)
    for e in range(E):
        if rows[e] == 0:
            assert not dw1[e].any() and not dw2[e].any()
    before1, before2 = dw1.clone(), dw2.clone()
    B.moe_expert_ffn_bwd(xp, h, dyp, None, offsets, w1, w2, dxp, dw1, dw2, 1, ws)
    assert rel(dw1, before1.double() + DW1) < tol
    assert rel(dw2, before2.double() + DW2) < tol


# rows, d, f: split products on 64 x 64 tiles (of the second FC1, FC2 and d_w1 on 128 x 128; which product takes which is pinned in
# test_row_plan.py), edges of tiles, k tails of 16, odd and even numbers of steps, a segment of one row, an empty one, segments of a few rows
SPLIT = [
    ([1, 0, 700, 130, 63], 272, 1040),
    ([500, 511, 0, 1049], 1024, 1408),
    ([40] * 30, 48, 528),
    ([1027], 1552, 784),
]
# 128 x 128 tiles in FC1, dgrad2 and both weight gradients
LARGE = ([240, 255, 245, 260, 262, 238, 240, 260], 1024, 2816)
# 128 x 128 tiles of eight waves in FC1 and d_w2, in dgrad2 and d_w1 (dgrad1 of the last in five parts of 128 x 128): edges, k tails of 16, a segment of
# one row
EIGHT = [([871, 1, 628], 1008, 1040), ([1500], 784, 2064)]


def ffn_f32(rows, d, f, xp, dyp, w1, w2, a_override=None):
    from paper_2505_11432_amd import binding as B
    E, M = len(rows), sum(rows)
    offsets = torch.tensor([sum(rows[:e]) for e in range(E + 1)], dtype=torch.int32, device=DEV)
    h, yp, dxp = (torch.full((M, n), 7.0, device=DEV) for n in (2 * f, d, d))
    dw1, dw2 = torch.full_like(w1, 7.0), torch.full_like(w2, 7.0)
    ws = torch.empty(max(B.moe_workspace_bytes(M, d, E, 1, f, B.F32), 256), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(xp, None, offsets, w1, None, w2, None, h, yp, None, ws)
    B.moe_expert_ffn_bwd(xp, h, dyp, a_override, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    return h, yp, dxp, dw1, dw2


def inputs_f32(rows, d, f):
    E, M = len(rows), sum(rows)
    g = torch.Generator(device=DEV).manual_seed(M + d)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    return rnd(M, d), rnd(M, d), rnd(E, 2 * f, d) / math.sqrt(d), rnd(E, d, f) / math.sqrt(f)


@pytest.mark.parametrize("rows,d,f", SPLIT + [LARGE] + EIGHT)
def test_split_products_are_as_close_as_fp32(rows, d, f):
    """Every product against float64, on the operands that the library itself made: within what an fp32 sum of K terms that is rounded
    every second term loses (sqrt(K / 2) roundings of random sign, 2^-24 at most and 0.58 of that each in the mean square).  Sums of one
    and two terms have a test of their own below: here the operands' own roundings cover them."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    h, yp, dxp, dw1, dw2 = ffn_f32(rows, d, f, xp, dyp, w1, w2)
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        a, b, X, DY = w1[e].double(), w2[e].double(), xp[s].double(), dyp[s].double()
        if n == 0:
            assert not dw1[e].any() and not dw2[e].any()
            continue
        G, U = h[s, :f].double(), h[s, f:].double()
        sg = torch.sigmoid(G)
        A, dA = G * sg * U, DY @ b
        dH = torch.cat([dA * U * sg * (1 + G * (1 - sg)), dA * G * sg], 1)
        # fp32 operands in between (A, dA, dH: a few roundings per element) add up to 4 * 2^-24 in all
        for name, got, ref, K in (("h", h[s], X @ a.t(), d), ("yp", yp[s], A @ b.t(), f), ("d_xp", dxp[s], dH @ a, 2 * f),
                                  ("d_w1", dw1[e], dH.t() @ X, n), ("d_w2", dw2[e], DY.t() @ A, n)):
            tol = (0.58 * math.sqrt(K / 2) + 4) * 2.0 ** -24
            assert rel(got, ref) < tol, (name, e, rel(got, ref), tol)


# FC2 and dgrad1 cut along K: 64 x 64 and 128 x 128 tiles, numbers of steps that the parts do not divide, a k tail of 16, rows past the
# segments.  With the workspace of the forward alone FC2 is not cut.  The last is not cut: 64 x 64 tiles, d_w1 on eight waves.
CUT = [([64, 0, 127, 1, 64, 40, 90, 126], 1024, 2832, 0), ([255, 1, 0, 700, 129, 300, 415, 200], 1024, 2832, 77), ([500, 511, 0, 1049], 1024, 1408, 3),
       ([300, 333, 0, 567], 496, 1008, 5)]


@pytest.mark.parametrize("rows,d,f,spare", CUT)
def test_products_cut_along_k(rows, d, f, spare):
    from paper_2505_11432_amd import binding as B
    E, n = len(rows), sum(rows)
    M = n + spare
    xp, dyp, w1, w2 = inputs_f32(rows + [spare], d, f)
    w1, w2 = w1[:E].contiguous(), w2[:E].contiguous()
    offsets = torch.tensor([sum(rows[:e]) for e in range(E + 1)], dtype=torch.int32, device=DEV)
    full, least = B.moe_workspace_bytes(M, d, E, 1, f, B.F32), -(-M * f * 4 // 256) * 256
    out = []
    for nbytes in (full, least):
        h, yp = torch.full((M, 2 * f), 7.0, device=DEV), torch.full((M, d), 7.0, device=DEV)
        ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)          # (NaN where a part would be read unwritten)
        B.moe_expert_ffn_fwd(xp, None, offsets, w1, None, w2, None, h, yp, None, ws[:nbytes])
        assert bool((ws[nbytes:] == 0xff).all()) and bool((yp[n:] == 7.0).all())
        out.append(yp)
    dxp, dw1, dw2 = torch.full((M, d), 7.0, device=DEV), torch.empty_like(w1), torch.empty_like(w2)
    ws = torch.full((full,), 0xff, dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_bwd(xp, h, dyp, None, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    assert bool((dxp[n:] == 7.0).all())
    at = 0
    for e, k in enumerate(rows):
        s, at = slice(at, at + k), at + k
        if k == 0:
            assert not dw1[e].any() and not dw2[e].any()
            continue
        a, b, DY = w1[e].double(), w2[e].double(), dyp[s].double()
        G, U = h[s, :f].double(), h[s, f:].double()
        sg = torch.sigmoid(G)
        dA = DY @ b
        dH = torch.cat([dA * U * sg * (1 + G * (1 - sg)), dA * G * sg], 1)
        # the bound of the uncut products: sqrt(K / 2) roundings, and the operands' own
        A = G * sg * U
        for got, ref, K in ((out[0][s], A @ b.t(), f), (out[1][s], A @ b.t(), f), (dxp[s], dH @ a, 2 * f),
                            (dw1[e], dH.t() @ xp[s].double(), k), (dw2[e], DY.t() @ A, k)):
            assert rel(got, ref) < (4 + 0.58 * math.sqrt(K / 2)) * 2.0 ** -24, (e, rel(got, ref))


@pytest.mark.parametrize("rows,d,f", CASES[:2] + [([70, 3, 129, 0, 64, 31, 95, 120], 128, 256), ([20, 32, 0, 33], 272, 1040), CASES[3]])
@pytest.mark.parametrize("at", [0, 1])
def test_output_written_over_the_saved_activations(rows, d, f, at):
    """A forward without a backward may give yp the room of H (from its start, from its second half on): the bits of the call with
    separate buffers."""
    from paper_2505_11432_amd import binding as B
    E, M = len(rows), sum(rows)
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    want = ffn_f32(rows, d, f, xp, dyp, w1, w2)[1]
    offsets = torch.tensor([sum(rows[:e]) for e in range(E + 1)], dtype=torch.int32, device=DEV)
    room = torch.full((M * (f + max(2 * f, d)),), 7.0, device=DEV)
    yp = room[at * M * f:][:M * d].view(M, d)
    ws = torch.empty(max(B.moe_workspace_bytes(M, d, E, 1, f, B.F32), 256), dtype=torch.uint8, device=DEV)
    B.moe_expert_ffn_fwd(xp, None, offsets, w1, None, w2, None, room[:2 * M * f].view(M, 2 * f), yp, None, ws)
    assert torch.equal(yp, want)


# small layers, whose last three products of a backward share a launch, and one whose products do not
@pytest.mark.parametrize("rows,d,f", [([1, 31, 0, 32], 16, 48), ([70, 3, 129, 0, 64, 31, 95, 120], 128, 256), ([20, 32, 0, 33], 272, 272), CASES[3]])
@pytest.mark.parametrize("over", ["d_yp", "a_override", "w1", "d_yp, part"])
def test_gradients_written_over_what_earlier_products_read(rows, d, f, over):
    """d_xp over d_yp or a_override (d_w2 reads both), d_w1 over w1 (d_xp reads it): the bits of the call with separate buffers."""
    from paper_2505_11432_amd import binding as B
    E, M = len(rows), sum(rows)
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    a = torch.randn(M * max(d, f), generator=torch.Generator(device=DEV).manual_seed(7), device=DEV)[:M * f].view(M, f)
    a = a if over == "a_override" else None
    ref = ffn_f32(rows, d, f, xp, dyp, w1, w2, a_override=a)
    offsets = torch.tensor([sum(rows[:e]) for e in range(E + 1)], dtype=torch.int32, device=DEV)
    ws = torch.empty(max(B.moe_workspace_bytes(M, d, E, 1, f, B.F32), 256), dtype=torch.uint8, device=DEV)
    dxp, dw1, dw2 = torch.full_like(xp, 7.0), torch.full_like(w1, 7.0), torch.full_like(w2, 7.0)
    if over == "d_yp":
        dxp = dyp
    elif over == "d_yp, part":                       # the second half of d_yp
        both = torch.full((2 * M, d), 7.0, device=DEV)
        both[:M] = dyp
        dyp, dxp = both[:M], both[M // 2:M // 2 + M]
    elif over == "a_override":
        dxp = torch.as_strided(a, (M, d), (d, 1))
    else:
        dw1 = w1
    B.moe_expert_ffn_bwd(xp, ref[0], dyp, a, offsets, w1, w2, dxp, dw1, dw2, 0, ws)
    for name, got, want in (("d_xp", dxp, ref[2]), ("d_w1", dw1, ref[3]), ("d_w2", dw2, ref[4])):
        assert torch.equal(got, want), name


@pytest.mark.parametrize("rows,d,f", [SPLIT[1], LARGE])
def test_split_weight_gradients_accumulate(rows, d, f):
    """accumulate = 1 adds the product, the same bits as without it, to what is there."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    from paper_2505_11432_amd import binding as B
    h, _, dxp, dw1, dw2 = ffn_f32(rows, d, f, xp, dyp, w1, w2)
    offsets = torch.tensor([sum(rows[:e]) for e in range(len(rows) + 1)], dtype=torch.int32, device=DEV)
    ws = torch.empty(B.moe_workspace_bytes(sum(rows), d, len(rows), 1, f, B.F32), dtype=torch.uint8, device=DEV)
    a1, a2 = torch.randn_like(dw1), torch.randn_like(dw2)
    r1, r2 = a1 + dw1, a2 + dw2
    B.moe_expert_ffn_bwd(xp, h, dyp, None, offsets, w1, w2, dxp, a1, a2, 1, ws)
    assert torch.equal(a1, r1) and torch.equal(a2, r2)


def test_weight_gradients_of_one_and_two_rows_round_as_fp32():
    """Beside segments that make the launch take the split: one row gives the rounded product, two rows a product rounded and the
    other added to it and rounded, half a unit in the last place each."""
    rows, d, f = [1, 2, 700, 1, 130, 2, 0], 272, 1040
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    a = torch.randn(sum(rows), f, generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    dw2 = ffn_f32(rows, d, f, xp, dyp, w1, w2, a_override=a)[4]
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        if n == 1:
            assert torch.equal(dw2[e], (dyp[s].double().t() * a[s].double()).float()), e
        elif n == 2:
            p, q = (dyp[s][i].double()[:, None] * a[s][i].double()[None] for i in (0, 1))
            bound = (torch.maximum(p.abs(), q.abs()) + (p + q).abs()) * 2.0 ** -24 * (1 + 2.0 ** -20)
            assert ((dw2[e].double() - p - q).abs() <= bound).all(), e


@pytest.mark.parametrize("rows,d,f", SPLIT[:2])
@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -110, 2.0 ** -126, 2.0 ** -140, 2.0 ** 120])
def test_split_products_of_tiny_and_huge_elements(rows, d, f, scale):
    """The whole range of fp32, subnormal numbers included (half a unit of 2^-149 per element and result is what they leave)."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    xp[5:] *= scale                                                     # ordinary rows beside them in the first tile
    h = ffn_f32(rows, d, f, xp, dyp, w1, w2)[0]
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        ref = xp[s].double() @ w1[e].double().t()
        tol = 3 * math.sqrt(d) * 2.0 ** -24 * ref.norm() + math.sqrt(d * ref.numel()) * 2.0 ** -149
        assert n == 0 or float((h[s].double() - ref).norm()) < float(tol), (e, float((h[s].double() - ref).norm()), float(tol))


@pytest.mark.parametrize("rows,d,f", SPLIT[:2] + [LARGE] + EIGHT)
def test_tiny_rows_leave_the_others_alone(rows, d, f):
    """What a row holds does not change how the rows of its tile are computed: the same bits beside it."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    ref = ffn_f32(rows, d, f, xp, dyp, w1, w2)
    touched = torch.arange(0, sum(rows), 37, device=DEV)
    xp[touched] *= 2.0 ** -115
    dyp[touched] *= 2.0 ** -115
    got = ffn_f32(rows, d, f, xp, dyp, w1, w2)
    rest = torch.ones(sum(rows), dtype=torch.bool, device=DEV)
    rest[touched] = False
    for name, i in (("h", 0), ("yp", 1), ("d_xp", 2)):
        assert torch.equal(got[i][rest], ref[i][rest]), name


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -70, 2.0 ** -90, 2.0 ** -110, 2.0 ** -126, 2.0 ** -140, 2.0 ** 100])
@pytest.mark.parametrize("rows,d,f", SPLIT[:2] + [LARGE])
def test_split_products_of_mixed_magnitudes(rows, d, f, scale):
    """Rows (in the weight gradient columns) of ordinary and of tiny or huge elements in one tile, each judged by its own size; 2^-149 and
    half of it are what subnormal elements and sums leave.  2^100: every tile goes back to the fp32 instruction."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    a = torch.randn(sum(rows), f, generator=torch.Generator(device=DEV).manual_seed(9), device=DEV)
    small = torch.arange(sum(rows), device=DEV) % 16 > 5
    xs, ys = xp.clone(), dyp.clone()
    xs[small] *= scale
    ys[small] *= scale
    a[:, torch.arange(f, device=DEV) % 16 > 5] *= scale
    h, _, _, _, dw2 = ffn_f32(rows, d, f, xs, dyp, w1, w2, a_override=a)
    _, _, dxp, _, _ = ffn_f32(rows, d, f, xp, ys, w1, w2)
    h0 = ffn_f32(rows, d, f, xp, ys, w1, w2)[0]
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        if n == 0:
            continue
        w1e, w2e, G, U = w1[e].double(), w2[e].double(), h0[s, :f].double(), h0[s, f:].double()
        sg, dA = torch.sigmoid(G), ys[s].double() @ w2e
        dX = torch.cat([dA * U * sg * (1 + G * (1 - sg)), dA * G * sg], 1) @ w1e
        for name, got, ref, K in (("h", h[s], xs[s].double() @ w1e.t(), d), ("d_xp", dxp[s], dX, 2 * f), ("d_w2", dw2[e], dyp[s].double().t() @ a[s].double(), n)):
            size, out = (ref.norm(dim=1), (got.double() - ref).norm(dim=1)) if name != "d_w2" else (ref.norm(dim=0), (got.double() - ref).norm(dim=0))
            # d_xp: three products in a row, whose operands are rounded to 2^-149 as well
            tol = 3 * 3 * math.sqrt(K) * 2.0 ** -24 * size + 3 * math.sqrt(K * (ref.numel() // size.numel())) * 2.0 ** -149
            assert (out <= tol).all(), (name, e, float((out / tol).max()))


@pytest.mark.parametrize("rows,d,f", SPLIT[:2] + [LARGE])
@pytest.mark.parametrize("ex,ew", [(-70, -70), (-60, -70), (-20, -120), (10, -140), (-149, 100)])
def test_split_products_below_the_normal_range(rows, d, f, ex, ew):
    """Ordinary elements whose products are subnormal numbers, subnormal elements whose products are not."""
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    xp, w1 = xp * 2.0 ** (ex / 2) * 2.0 ** (ex / 2), w1 * 2.0 ** (ew / 2) * 2.0 ** (ew / 2)
    h = ffn_f32(rows, d, f, xp, dyp, w1, w2)[0]
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        ref = xp[s].double() @ w1[e].double().t()
        # every element to half a unit in the last place of its own sum's terms, and to a unit of 2^-149 for each rounding
        tol = 3 * math.sqrt(d) * 2.0 ** -24 * ref.norm() + math.sqrt(d * ref.numel()) * 2.0 ** -149
        assert n == 0 or float((h[s].double() - ref).norm()) <= float(tol), (e, float((h[s].double() - ref).norm()), float(tol))
        assert n == 0 or ew < -130 or h[s].any()


@pytest.mark.parametrize("rows,d,f", [SPLIT[0], EIGHT[0]])
def test_split_products_of_infinities_and_nan(rows, d, f):
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    inf = float("inf")
    xp[3, 7], xp[9, 200], xp[300, 0], xp[301, 1] = inf, -inf, float("nan"), 3.4e38         # the last: above bf16's largest
    w1[2, 40, 11] = inf
    xp[20] = 0.0                                                                            # 0 * inf
    h = ffn_f32(rows, d, f, xp, dyp, w1, w2)[0]
    at = 0
    for e, n in enumerate(rows):
        s, at = slice(at, at + n), at + n
        ref = xp[s].double() @ w1[e].double().t()
        over = ref.abs() > torch.finfo(torch.float32).max
        ref[over] = ref[over].sign() * inf
        got = h[s].double()
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got[ref.isinf()], ref[ref.isinf()])
        fin = ref.isfinite()
        assert n == 0 or rel(got[fin], ref[fin]) < 3 * math.sqrt(d) * 2.0 ** -24


@pytest.mark.parametrize("rows,d,f", [SPLIT[0], LARGE] + EIGHT)
def test_split_products_of_infinities_and_nan_in_every_layout(rows, d, f):
    """The other operand layouts (weights across their rows, weight gradients) on every tile: what a row or column that holds no such
    element gets is finite and as close as ever, also inside a tile that is made again."""
    inf, nan = float("inf"), float("nan")
    xp, dyp, w1, w2 = inputs_f32(rows, d, f)
    a = torch.randn(sum(rows), f, generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
    clean = ffn_f32(rows, d, f, xp, dyp, w1, w2, a_override=a)
    bad, cols = torch.tensor([4, 70, 261, 703], device=DEV), torch.tensor([5, 130, 200, f - 1], device=DEV)
    ys, ab = dyp.clone(), a.clone()
    ys[bad, torch.tensor([0, 17, d - 1, 100], device=DEV)] = torch.tensor([inf, nan, -inf, nan], device=DEV)
    ab[bad, cols] = torch.tensor([nan, inf, -inf, nan], device=DEV)
    dxp = ffn_f32(rows, d, f, xp, ys, w1, w2)[2]
    dw2 = ffn_f32(rows, d, f, xp, dyp, w1, w2, a_override=ab)[4]
    good = torch.ones(sum(rows), dtype=torch.bool, device=DEV)
    good[bad] = False
    # two results of the same product, each off by at most what one product (d_xp: three in a row) may be
    K = max(rows + [2 * f])
    assert not dxp[bad].isfinite().any()
    assert dxp[good].isfinite().all() and rel(dxp[good], clean[2][good].double()) < 2 * 3 * 3 * math.sqrt(K) * 2.0 ** -24
    ok = torch.ones(f, dtype=torch.bool, device=DEV)
    ok[cols] = False
    assert dw2[:, :, ok].isfinite().all() and rel(dw2[:, :, ok], clean[4][:, :, ok].double()) < 2 * 3 * math.sqrt(max(rows)) * 2.0 ** -24
    for r, c in zip(bad.tolist(), cols.tolist()):
        e = next(i for i in range(len(rows)) if r < sum(rows[: i + 1]))
        assert not dw2[e, :, c].isfinite().any(), (r, c)


@pytest.mark.parametrize("T,d,E", [(1, 16, 1), (33, 260, 5), (1000, 1024, 64), (65, 4, 3), (50, 30, 4)])
def test_router_f32_edges(T, d, E):
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T)
    x, w = torch.randn((T, d), generator=g, device=DEV), torch.randn((E, d), generator=g, device=DEV)
    bias = torch.randn((E,), generator=g, device=DEV)
    z = torch.full((T, E), 7.0, device=DEV)
    B.moe_router_fwd(x, w, bias, z)
    ref = x.double() @ w.double().t() + bias.double()
    assert rel(z, ref) < 3 * math.sqrt(d) * 2.0 ** -24 + 2.0 ** -23


def test_router_f32_of_many_tokens():
    """More tokens than one launch of 64 x 32 tiles can take (2^29 with 33 to 64 experts: a launch holds less than 2^32 threads)."""
    from paper_2505_11432_amd import binding as B
    T, d, E, n = 2 ** 29 + 65, 4, 33, 2 ** 16
    if torch.cuda.mem_get_info()[0] < 90e9:
        pytest.skip("needs 80 GB")
    g = torch.Generator(device=DEV).manual_seed(0)
    part, w = (torch.randint(-4, 5, s, generator=g, device=DEV).float() for s in ((n, d), (E, d)))      # exact sums
    want = (part.double() @ w.double().t()).float()
    x, z = torch.empty((T, d), device=DEV), torch.empty((T, E), device=DEV)
    whole = T // n * n
    x[:whole].view(-1, n, d).copy_(part.expand(whole // n, -1, -1))
    x[whole:] = part[:T - whole]
    B.moe_router_fwd(x, w, None, z)
    for a in range(0, whole, 64 * n):
        assert bool((z[a:a + 64 * n][:min(64 * n, whole - a)].view(-1, n, E) == want).all()), a
    assert torch.equal(z[whole:], want[:T - whole])
