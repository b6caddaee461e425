"""fp32 grouped GEMMs on the matrix cores: tile edges, remainders, empty experts and the three tile shapes, against float64."""
import math

import pytest
import torch

from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

# rows per expert, d, f: segments around the 32- and 64-row tiles, widths with 16-column tails, and sizes that reach the
# 64 x 32 and 64 x 64 tiles (from 256 and 1024 tiles on)
CASES = [
    ([1, 31, 0, 32], 16, 48),
    ([33, 63, 64, 65], 144, 80),
    ([0, 0, 129, 0], 48, 272),
    ([500, 511, 0, 1049], 272, 2000),
    ([3] * 70, 64, 32),                    # more segments than lanes in a wave
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
