"""Argument checks of the Python entry points (no GPU needed: every call here is refused before it reaches a stream)."""
import pytest
import torch


class Duck:
    """Looks like a tensor to Python only."""

    def __init__(self, is_cuda, contiguous):
        self.is_cuda, self._c = is_cuda, contiguous

    def is_contiguous(self):
        return self._c

    def data_ptr(self):
        raise RuntimeError("asked for the pointer")


def test_refused_arguments():
    from paper_2505_11432_amd import binding as B
    n = B._native
    cpu = torch.zeros((4, 8))
    with pytest.raises(AssertionError, match="contiguous and on the GPU"):
        n.moe_transpose(cpu, B.F32, 1, 4, 8, None)
    for cuda, contiguous in ((False, True), (True, False)):
        with pytest.raises(AssertionError, match="contiguous and on the GPU"):
            n.moe_transpose(Duck(cuda, contiguous), B.F32, 1, 4, 8, None)
    with pytest.raises(RuntimeError, match="asked for the pointer"):
        n.moe_transpose(Duck(True, True), B.F32, 1, 4, 8, None)
    with pytest.raises(AttributeError):
        n.moe_transpose(3, B.F32, 1, 4, 8, None)
    with pytest.raises(TypeError):
        n.moe_transpose(None, "f32", 1, 4, 8, None)
    with pytest.raises(TypeError, match="takes 6 arguments"):
        n.moe_transpose(None, B.F32, 1, 4, 8)
    with pytest.raises(TypeError):
        n.moe_balance_loss_bwd(None, None, 1, 1, 1, "x", None)
