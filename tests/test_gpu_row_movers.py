"""Dispatch where its waves split: one to many per token, rows that end inside a chunk group, more tokens than one round of the
grid, tokens without a local expert."""
import pytest
import torch

from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32, torch.uint8])
@pytest.mark.parametrize("T,d,k", [(1, 16, 1), (3, 16400, 3), (257, 4112, 8), (1023, 2064, 2), (1025, 2064, 2), (4096, 1040, 1), (8193, 1040, 2),
                                   (16385, 528, 1), (40000, 16, 16), (70001, 272, 1)])
def test_dispatch_splits(T, d, k, dtype):
    from paper_2505_11432_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(T + d)
    M = T * k
    codes = dtype == torch.uint8
    x = torch.randint(0, 256, (T, d), generator=g, device=DEV, dtype=dtype) if codes else torch.randn((T, d), generator=g, device=DEV).to(dtype)
    w = torch.rand((M,), generator=g, device=DEV)
    scale = torch.rand((T,), generator=g, device=DEV) if codes else None
    order = torch.randperm(M, generator=g, device=DEV).to(torch.int32)
    some = torch.where(torch.rand((M,), generator=g, device=DEV) < 0.2, order, torch.full_like(order, -1))
    token = torch.arange(M, device=DEV) // k
    for inv in (order, some):
        local = inv >= 0
        row, src = inv[local].long(), token[local]
        for mul in (None,) if codes else (None, w):
            xp = torch.full((M, d), 3, dtype=dtype, device=DEV)
            xs = torch.full((M,), 3.0, device=DEV) if codes else None
            B.moe_dispatch(x, scale, inv, mul, k, xp, xs)
            want = torch.full((M, d), 3, dtype=dtype, device=DEV)
            want[row] = x[src] if mul is None else (x[src].float() * w[local][:, None]).to(dtype)
            assert torch.equal(xp, want)
            if codes:
                ws = torch.full((M,), 3.0, device=DEV)
                ws[row] = scale[src]
                assert torch.equal(xs, ws)
