"""E4M3 cast at the edges of its kernels: codes, scales and decoded values equal to the oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from synth.moe_inputs import bf16_round
from tests.gpu_util import DEV, to_dev, to_np, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
# vectors per row at and past 2, 4 and 8 per lane of a wave (bf16: 1024, 2048, 4096 columns; fp32: half), a 16-column
# tail, one row, a short last group of 128, a last block of pieces that is not full
@pytest.mark.parametrize("rows,cols", [(1, 16), (5, 512), (127, 528), (128, 1024), (129, 1040), (3, 2048), (6, 2064),
                                       (257, 4096), (2, 4112), (9, 16400)])
def test_cast_edges(dtype, rows, cols):
    from paper_2505_11432_amd import binding as B
    rng = np.random.default_rng(rows * cols)
    v = (rng.standard_normal((rows, cols)) * np.exp(rng.standard_normal((rows, 1)) * 3)).astype(np.float32)
    v[0, :8] = 0.0
    if rows > 2:
        v[1] = 0.0                                # a row of zeros: scale 1
        v[:, 9] = 0.0
    if dtype == "bf16":
        v = bf16_round(v)
    t = to_dev(v, torch_dtype(dtype))
    for mode, quant, dequant, shape in ((B.Q_ROW, O.quant_rows, O.dequant_rows, (rows,)),
                                        (B.Q_COLGROUP128, O.quant_colgroup128, O.dequant_colgroup128, ((rows + 127) // 128, cols))):
        codes = torch.full((rows + 1, cols), 9, dtype=torch.uint8, device=DEV)
        scales = torch.full(shape, 9.0, device=DEV)
        B.moe_quant_fp8(t, mode, codes[:rows], scales)
        want_c, want_s = quant(v)
        assert np.array_equal(to_np(codes[:rows]), want_c) and np.array_equal(to_np(scales).astype(np.float32), want_s.reshape(shape))
        assert bool((codes[rows] == 9).all())
        want = dequant(want_c, want_s)
        shifted = torch.empty((scales.numel() + 1,), device=DEV)[1:].view(shape)      # scales that are not 16-byte aligned
        shifted.copy_(scales)
        for sc in (scales, shifted):
            for td in (torch.float32, torch.bfloat16):
                out = torch.full((rows + 1, cols), 7.0, dtype=td, device=DEV)
                B.moe_dequant_fp8(codes[:rows], sc, mode, out[:rows])
                ref = want.astype(np.float32)
                assert np.array_equal(to_np(out[:rows]).astype(np.float32), ref if td == torch.float32 else bf16_round(ref))
                assert bool((out[rows] == 7.0).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_tgroup_cast_short_segments(dtype):
    from paper_2505_11432_amd import binding as B
    counts = [1, 0, 128, 129, 7, 300, 0]
    rows, cols, E = sum(counts), 144, len(counts)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    v = np.random.default_rng(3).standard_normal((rows, cols)).astype(np.float32) * 30
    v = bf16_round(v) if dtype == "bf16" else v
    ldt = B.moe_tgroup_tokens(rows, E)
    pad = torch.empty((E + 1,), dtype=torch.int32, device=DEV)
    ct, e8 = torch.full((cols, ldt), 9, dtype=torch.uint8, device=DEV), torch.full((ldt // 128, cols), 9, dtype=torch.uint8, device=DEV)
    B.moe_quant_fp8_tgroup(to_dev(v, torch_dtype(dtype)), to_dev(off), pad, ct, e8)
    p = to_np(pad)
    got_c, got_e = to_np(ct), to_np(e8)
    for e in range(E):
        for j, s in enumerate(range(0, counts[e], 128)):
            block = v[off[e] + s: off[e] + min(s + 128, counts[e])]
            k = O.pow2_exponent(np.abs(block).max(axis=0).astype(np.float32))
            want = O.e4m3_encode((block * np.exp2(-k.astype(np.float64))).astype(np.float32)).T
            c0 = p[e] + s
            assert np.array_equal(got_c[:, c0:c0 + want.shape[1]], want)
            assert not got_c[:, c0 + want.shape[1]:c0 + 128].any()
            assert np.array_equal(got_e[c0 // 128], (k + 127).astype(np.uint8))


def test_row_cast_of_many_rows():
    """More rows than one launch of a wave per row can take (2^26: a launch holds less than 2^32 threads), 16 bf16 columns."""
    from paper_2505_11432_amd import binding as B
    rows, cols = 2 ** 26 + 5, 16
    part = torch.randn((4099, cols), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV).bfloat16()
    src = torch.empty((rows, cols), dtype=torch.bfloat16, device=DEV)
    whole = rows // 4099 * 4099
    src[:whole].view(-1, 4099, cols).copy_(part.expand(whole // 4099, -1, -1))
    src[whole:] = part[:rows - whole]
    codes, scales = torch.empty((rows, cols), dtype=torch.uint8, device=DEV), torch.empty((rows,), device=DEV)
    want_c, want_s = torch.empty((4099, cols), dtype=torch.uint8, device=DEV), torch.empty((4099,), device=DEV)
    B.moe_quant_fp8(part, B.Q_ROW, want_c, want_s)
    B.moe_quant_fp8(src, B.Q_ROW, codes, scales)
    assert bool((codes[:whole].view(-1, 4099, cols) == want_c).all()) and bool((scales[:whole].view(-1, 4099) == want_s).all())
    assert torch.equal(codes[whole:], want_c[:rows - whole]) and torch.equal(scales[whole:], want_s[:rows - whole])


# column slabs of 32, 64 and 128 columns and one past them, with full, short and one-row last groups
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,cols", [(129, 32), (130, 48), (127, 64), (3, 80), (256, 144)])
def test_cast_column_slabs(dtype, rows, cols):
    test_cast_edges(dtype, rows, cols)


def test_colgroup_cast_of_a_large_fp32_tensor():
    """2^26 elements: read past the caches.  Every group of 128 rows gives what it gives alone."""
    from paper_2505_11432_amd import binding as B
    rows, cols = 2 ** 16 + 3, 1024
    src = torch.randn((rows, cols), generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
    codes, scales = torch.empty((rows, cols), dtype=torch.uint8, device=DEV), torch.empty(((rows + 127) // 128, cols), device=DEV)
    B.moe_quant_fp8(src, B.Q_COLGROUP128, codes, scales)
    part_c, part_s = torch.empty((8192, cols), dtype=torch.uint8, device=DEV), torch.empty((64, cols), device=DEV)
    for a in range(0, rows, 8192):
        n = min(8192, rows - a)
        g = (n + 127) // 128
        B.moe_quant_fp8(src[a:a + n], B.Q_COLGROUP128, part_c[:n], part_s[:g])
        assert torch.equal(codes[a:a + n], part_c[:n]) and torch.equal(scales[a // 128:a // 128 + g], part_s[:g]), a


# pieces of 16 bytes on both sides of where a thread takes one of them or four: 2^18 with row scales; with channel scales 2^23
# to bf16 and 2^21 to fp32
@pytest.mark.parametrize("mode,td,rows,cols", [(0, torch.bfloat16, 2048, 1024), (0, torch.bfloat16, 2049, 1024), (0, torch.float32, 1025, 1024),
                                               (1, torch.bfloat16, 8192, 8192), (1, torch.bfloat16, 8193, 8192), (1, torch.float32, 4096, 2048),
                                               (1, torch.float32, 4097, 2048)])
def test_dequant_sizes(mode, td, rows, cols):
    from paper_2505_11432_amd import binding as B
    assert (B.Q_ROW, B.Q_COLGROUP128) == (0, 1)
    g = torch.Generator(device=DEV).manual_seed(rows)
    codes = torch.randint(0, 256, (rows, cols), generator=g, device=DEV, dtype=torch.uint8)
    codes[(codes & 127) == 127] = 0                         # no NaN codes
    scales = torch.rand((rows,) if mode == 0 else ((rows + 127) // 128, cols), generator=g, device=DEV) + 0.5
    out = torch.full((rows + 1, cols), 7.0, dtype=td, device=DEV)
    B.moe_dequant_fp8(codes, scales, mode, out[:rows])
    per = scales[:, None] if mode == 0 else scales.repeat_interleave(128, dim=0)[:rows]
    assert torch.equal(out[:rows], (codes.view(torch.float8_e4m3fn).float() * per).to(td))      # one fp32 product, one rounding
    assert bool((out[rows] == 7.0).all())
