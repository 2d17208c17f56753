"""Workspace of a training step of the cost network: what the kernels use, which stops
growing with the samples once every workgroup has a tile."""
import pytest

from paper_1509_04394_amd import fz


@pytest.mark.parametrize("F", [1, 7, 20, 31, 32])
def test_workspace_holds_the_partial_gradients_and_no_more(F):
    row = 4 * (fz.fz_mlp_param_count(F) + 1)  # a workgroup's gradient and loss
    last = 0
    for n in (1, 31, 32, 33, 64, 65, 97, 8192, 16384, 16385, 65536, 1 << 20, (1 << 31) - 1):
        need = fz.fz_mlp_workspace_bytes(F, n)
        assert need == row * min(-(-n // 32), 512) and need >= last
        last = need
    assert fz.fz_mlp_workspace_bytes(F, 0) == fz.fz_mlp_workspace_bytes(33, 10) == 0
