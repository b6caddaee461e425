"""Gate and row map at the edges of their kernels: both sides of the histogram size that drops the scan launch, chunks of more
than 512 assignments, every group width, and the gate's backward; the small router matmul around its tiles."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from synth.moe_inputs import random_logits
from tests.gpu_util import DEV, max_norm_err, to_dev, to_np
from tests.test_gpu_parity import run_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,quantum", [
    (4096, 256, 2, 0.5), (4097, 256, 2, 0.5),      # 64 and 65 chunks of 256 counts: without and with the scan kernel
    (33000, 32, 3, 1.0),                           # 516 chunks of 32
    (130, 256, 16, 0.25), (70001, 40, 16, 2.0),    # 1024 and 2048 assignments per chunk: two and four rounds of ranking
    (1, 1, 1, None), (65, 2, 2, None), (63, 3, 3, 0.5), (64, 7, 4, 0.5), (191, 13, 13, 0.5), (127, 65, 9, 0.5), (66, 129, 5, 0.5),
])
def test_route_edges(T, E, k, quantum):
    from paper_2505_11432_amd import binding as B
    z = random_logits(T, E, seed=T + E, quantum=quantum)
    if T > 8:
        z[3] = np.finfo(np.float32).min             # a row of the lowest value: ids decide
        z[3, E // 2] = 0.0
        z[4, ::2], z[4, 1::2] = -0.0, 0.0          # signed zeros are equal
    ref = O.route(z, k, 1)
    got = run_route(B, z, k, 1)
    for name in ("idx", "counts", "offsets", "perm", "inv_perm"):
        assert np.array_equal(to_np(got[name]), ref[name]), name
    assert np.allclose(to_np(got["w"]), ref["w"], rtol=2e-6, atol=1e-7)


@pytest.mark.parametrize("T,E,k", [(70, 8, 2), (65, 40, 5), (64, 256, 16)])
def test_route_nan_last(T, E, k):
    """A NaN logit (either sign) is selected only when fewer than k others are left; the ids stay valid even then."""
    from paper_2505_11432_amd import binding as B
    z = random_logits(T, E, seed=T + E, quantum=0.5)
    z[1, ::2], z[2, 1::2], z[3, : E - k] = np.nan, -np.nan, np.nan
    z[4, :], z[5, 1:] = np.nan, np.nan
    got = {n: to_np(v) for n, v in run_route(B, z, k, 1).items()}
    # k numbers are left in rows 1 to 3: there a NaN counts as less than everything
    ref = O.route(np.where(np.isnan(z), np.finfo(np.float32).min, z), k, 1)
    rows = np.arange(T) != 5                       # (row 4: all equal either way, the lowest ids)
    assert np.array_equal(got["idx"][rows], ref["idx"][rows]) and np.array_equal(got["idx"][5], np.arange(k))
    numbers = np.setdiff1d(np.arange(T), [4, 5])
    assert np.allclose(got["w"][numbers], ref["w"][numbers], rtol=2e-6, atol=1e-7)
    assert np.array_equal(got["counts"], np.bincount(got["idx"].ravel(), minlength=E))
    assert np.array_equal(np.sort(got["perm"]), np.arange(T * k))


@pytest.mark.parametrize("renorm", [1, 0])
@pytest.mark.parametrize("T,E,k", [(1, 1, 1), (33, 2, 1), (257, 8, 2), (15, 16, 16), (17, 33, 5), (100, 100, 7), (31, 256, 16)])
def test_route_bwd_edges(T, E, k, renorm):
    from paper_2505_11432_amd import binding as B
    z = random_logits(T, E, seed=T)
    ref = O.route(z, k, renorm)
    dw = np.random.default_rng(E).standard_normal((T, k)).astype(np.float32)
    want = O.route_bwd(z, ref["idx"], ref["w"], dw, renorm)
    guard = torch.full((T * E + 64,), 9.0, device=DEV)
    dz = guard[:T * E].view(T, E)
    B.moe_route_bwd(to_dev(z), to_dev(ref["idx"]), to_dev(ref["w"].astype(np.float32)), to_dev(dw), E, renorm, dz)
    # sums of at most 256 fp32 terms of either sign against the largest entry
    assert max_norm_err(to_np(dz), want) < 1e-5
    assert bool((guard[T * E:] == 9.0).all())


def test_route_bwd_zeros_are_positive():
    from paper_2505_11432_amd import binding as B
    z = random_logits(40, 24, seed=2)
    ref = O.route(z, 3, 1)
    dz = torch.full((40, 24), 9.0, device=DEV)
    for dw in (np.ones((40, 3), np.float32), -np.ones((40, 3), np.float32)):
        B.moe_route_bwd(to_dev(z), to_dev(ref["idx"]), to_dev(ref["w"].astype(np.float32)), to_dev(dw), 24, 1, dz)
        other = np.ones((40, 24), bool)
        np.put_along_axis(other, ref["idx"].astype(np.int64), False, axis=1)
        assert not to_np(dz)[other].any() and not np.signbit(to_np(dz)[other]).any()


@pytest.mark.parametrize("renorm", [1, 0])
def test_route_bwd_of_many_tokens(renorm):
    """More tokens than one launch of 16 threads each can take (2^28: a launch holds less than 2^32 threads): 22 GB."""
    from paper_2505_11432_amd import binding as B
    T, E, k, n = 2 ** 28 + 3, 9, 1, 4099
    g = torch.Generator(device=DEV).manual_seed(renorm)
    whole = T // n * n

    def spread(part):
        out = torch.empty((T,) + part.shape[1:], dtype=part.dtype, device=DEV)
        out[:whole].view((-1, n) + part.shape[1:]).copy_(part.expand((whole // n,) + part.shape))
        out[whole:] = part[:T - whole]
        return out

    z, w, dw = (torch.rand(s, generator=g, device=DEV) for s in ((n, E), (n, k), (n, k)))
    idx = torch.randint(0, E, (n, k), generator=g, device=DEV, dtype=torch.int32)
    want = torch.empty((n, E), device=DEV)
    B.moe_route_bwd(z, idx, w, dw, E, renorm, want)
    got = torch.full((T, E), 9.0, device=DEV)
    B.moe_route_bwd(None if renorm else spread(z), spread(idx), spread(w), spread(dw), E, renorm, got)
    step = n * 4096
    for a in range(0, whole, step):
        assert bool((got[a:min(a + step, whole)].view(-1, n, E) == want).all()), a
    assert torch.equal(got[whole:], want[:T - whole])


@pytest.mark.parametrize("T,d,E", [(1, 8, 1), (16, 64, 16), (17, 72, 17), (100, 2048, 64), (15, 4104, 8), (2049, 520, 64), (8176, 16, 16),
                                   (8193, 16, 16), (40, 1000, 256)])      # 512 tiles and more: the other kernel
def test_router_fwd_edges(T, d, E):
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T + E)
    x, w = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((T, d), (E, d)))
    bias = torch.randn((E,), generator=g, device=DEV)
    z = torch.full((T * E + 64,), 7.0, device=DEV)
    for b in (bias, None):
        B.moe_router_fwd(x, w, b, z[:T * E].view(T, E))
        ref = x.double() @ w.double().t() + (b.double() if b is not None else 0.0)
        # products are exact in fp32; d additions, each rounding by at most 2^-24 of a partial sum
        assert float((z[:T * E].view(T, E).double() - ref).norm() / ref.norm()) < 3 * np.sqrt(d) * 2.0 ** -24 + 2.0 ** -23
    assert bool((z[T * E:] == 7.0).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,d,E,shift", [(1, 1, 1, 0), (64, 16, 64, 1), (65, 17, 65, 0), (130, 1030, 5, 0), (200, 64, 130, 3)])
def test_router_fwd_any_rows(T, d, E, shift, dtype):
    """Rows that cannot be read in 16-byte pieces: odd widths, buffers that start `shift` elements past an aligned address."""
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T + d)
    x = torch.randn((shift + T * d,), generator=g, device=DEV).to(dtype)[shift:].view(T, d)
    w = torch.randn((E, d), generator=g, device=DEV).to(dtype)
    bias = torch.randn((E,), generator=g, device=DEV)
    z = torch.full((T * E + 64,), 7.0, device=DEV)
    for b in (bias, None):
        B.moe_router_fwd(x, w, b, z[:T * E].view(T, E))
        ref = x.double() @ w.double().t() + (b.double() if b is not None else 0.0)
        # d fp32 additions, each rounding by at most 2^-24 of a partial sum
        assert float((z[:T * E].view(T, E).double() - ref).norm() / ref.norm()) < 3 * np.sqrt(d) * 2.0 ** -24 + 2.0 ** -23
    assert bool((z[T * E:] == 7.0).all())


# assignments on both sides of what the one-launch selection holds (8192 and 32768), one device, a device per expert, many
# equal affinities (odd T quantises the logits), nothing kept, everything kept
@pytest.mark.parametrize("T,E,k,G,cap,skew", [(4096, 8, 2, 4, 1500, 1.0), (8193, 8, 1, 2, 2000, 1.0), (16384, 4, 2, 2, 9000, 0.5),
                                             (16385, 16, 2, 8, 3000, 1.0), (1023, 256, 4, 256, 10, 0.0), (777, 12, 3, 1, 1200, 0.0),
                                             (999, 6, 2, 3, 0, 0.0), (999, 6, 2, 3, 1998, 0.0), (1, 3, 1, 3, 1, 0.0)])
def test_route_capacity_edges(T, E, k, G, cap, skew):
    from paper_2505_11432_amd import binding as B
    from tests.test_gpu_parity import test_route_capacity as check
    check(B, T, E, k, G, cap, skew)


@pytest.mark.parametrize("T,E,k,G", [(1, 1, 1, 1), (63, 2, 1, 2), (64, 3, 2, 3), (129, 12, 3, 4), (4097, 24, 3, 8), (70000, 16, 2, 4), (200, 130, 5, 10), (300, 256, 4, 8)])
def test_balance_loss_edges(T, E, k, G):
    from paper_2505_11432_amd import binding as B
    from tests.test_gpu_parity import test_balance_loss_and_gradient as check
    check(B, T, E, k, G)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,d,E", [(1, 16, 1), (63, 272, 8), (65, 528, 9), (129, 1040, 17), (200, 144, 33), (130, 80, 100), (8200, 2064, 3)])
def test_router_bwd_edges(T, d, E, dtype):
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T)
    x, w, dz = (torch.randn(s, generator=g, device=DEV) for s in ((T, d), (E, d), (T, E)))
    x, w = x.to(dtype), w.to(dtype)
    buf = torch.randn((T * d + 64,), generator=g, device=DEV).to(dtype)
    dx, tail, dx0 = buf[:T * d].view(T, d), buf[T * d:].clone(), buf[:T * d].double().view(T, d)
    dwr = torch.full((E, d), 7.0, device=DEV)
    ws = torch.empty(max(B.moe_workspace_bytes(T, d, E, 1, 16, B.dtype_code(dtype)), 256), dtype=torch.uint8, device=DEV)
    B.moe_router_bwd(x, w, dz, dwr, dx, ws)
    want_w, want_x = dz.double().t() @ x.double(), dx0 + dz.double() @ w.double()
    # d_w_r: T fp32 additions of random sign; dx: E of them and one rounding to its type per pass of 64 experts
    assert float((dwr.double() - want_w).norm() / want_w.norm()) < 3 * np.sqrt(T) * 2.0 ** -24 + 2.0 ** -23
    step = 2.0 ** -9 if dtype == torch.bfloat16 else 2.0 ** -24 * 3 * np.sqrt(E) + 2.0 ** -23
    assert float((dx.double() - want_x).norm() / want_x.norm()) < 2 * step
    assert torch.equal(buf[T * d:], tail)


# up to 8 tokens and more (which the waves of a block share), gate gradients as scalar loads (bf16, more than 16 experts)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,d,E", [(8, 272, 20), (9, 272, 20), (40, 1040, 12), (8200, 528, 24), (4099, 1040, 41), (4099, 4112, 41)])
def test_router_bwd_splits(T, d, E, dtype):
    test_router_bwd_edges(T, d, E, dtype)


@pytest.mark.parametrize("T,d,E", [(100, 512, 9), (4096, 576, 16), (33, 2048, 5), (20, 2056, 40)])
def test_router_fwd_short_rows(T, d, E):
    """Rows that end inside a wave's four blocks of 64 columns, at their edges and past them."""
    test_router_fwd_edges(T, d, E)


@pytest.mark.parametrize("T,d,E", [(16383, 16, 33), (16384, 16, 33), (16400, 28, 5), (16384, 32, 70)])
def test_router_fwd_f32_narrow(T, d, E):
    test_router_fwd_any_rows(T, d, E, 0, torch.float32)


# few experts in the most chunks, many ties and several winners among the logits of one lane
@pytest.mark.parametrize("T,E,k,quantum", [(65536, 1, 1, None), (65537, 3, 2, 1.0), (33000, 250, 16, 0.5), (300, 256, 16, 2.0), (300, 100, 16, None)])
def test_route_lane_keys(T, E, k, quantum):
    test_route_edges(T, E, k, quantum)


@pytest.mark.parametrize("T,E,k", [(33000, 20, 3), (32768, 256, 4)])
def test_route_nan_last_of_many_tokens(T, E, k):
    test_route_nan_last(T, E, k)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,d,E", [(9, 16, 1), (65, 528, 8), (257, 272, 9), (1000, 1040, 16), (300, 4096, 17), (1531, 1040, 24), (70, 48, 31),
                                   (16000, 256, 8), (4097, 272, 12)])
def test_router_gradients_in_one_launch(T, d, E, dtype):
    """d_w_r and dx asked for together (one launch up to 1024 blocks, 16 experts in fp32 and 31 in bf16) and one by one: the same sums in
    the same order, bit for bit; against float64 (sums of T and of E terms); and dx written over x."""
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T + d)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)
    x, w, dz, dx0 = rnd(T, d).to(dtype), rnd(E, d).to(dtype), rnd(T, E), rnd(T, d).to(dtype)
    ws = torch.empty(max(B.moe_workspace_bytes(T, d, E, 1, 16, B.dtype_code(dtype)), 256), dtype=torch.uint8, device=DEV)
    both_w, one_w = torch.empty((E, d), device=DEV), torch.empty((E, d), device=DEV)
    both_x, one_x, over_x = dx0.clone(), dx0.clone(), x.clone()
    B.moe_router_bwd(x, w, dz, both_w, both_x, ws)
    B.moe_router_bwd(x, w, dz, one_w, None, ws)
    B.moe_router_bwd(x, w, dz, None, one_x, ws)
    assert torch.equal(both_w, one_w) and torch.equal(both_x, one_x)
    ref_w, ref_x = dz.double().t() @ x.double(), dz.double() @ w.double()
    assert float((both_w.double() - ref_w).norm() / ref_w.norm()) < 2.0 ** -24 * (T ** 0.5 + 4)
    want = dx0.double() + ref_x
    assert float((both_x.double() - want).norm() / want.norm()) < (2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -24 * (E ** 0.5 + 4))
    over_w = torch.empty((E, d), device=DEV)
    B.moe_router_bwd(over_x, w, dz, over_w, over_x, ws)
    assert torch.equal(over_w, one_w)
