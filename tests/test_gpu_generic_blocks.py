"""The interpreted generic kernels at block, tile and alignment edges: four-cell loads
and stores on aligned buffers, single cells on others, border tiles, an IIR after a window
stage, frames smaller than a tile.  The reference is the FP64 oracle with its FP32 bound;
every alignment and partition must give the same bits."""
import numpy as np
import pytest

import oracle
from paper_1509_04394_amd import fz
from tests import parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

W3 = (np.arange(9, dtype=np.float32).reshape(3, 3) - 3) / 32
W75 = (np.arange(35, dtype=np.float32).reshape(5, 7) % 6 - 2) / 64
BACK = (np.arange(2 * 15, dtype=np.float32).reshape(2, 5, 3) % 5 + 1) / 96
CHAINS = {
    "windows": [("point", "affine", 0.5, 1.0), ("stencil", 1, 1, W3), ("point", "abs", 0, 0), ("box", 3, 2),
                ("stencil", 3, 2, W75), ("point", "sqrtabs", 0, 0)],
    "one": [("stencil", 0, 0, np.full((1, 1), 0.75, np.float32))],
    "points": [("point", "square", 0, 0), ("point", "affine", -0.25, 3.0), ("point", "clamp", -900.0, 2.0)],
    "temporal": [("iir", 0.375), ("box", 1, 1), ("point", "affine", 0.125, 0.0), ("iir", 0.75), ("stencil", 1, 2, BACK),
                 ("point", "abs", 0, 0)],
    "resumed": [("iir", 0.375), ("stencil", 3, 2, W75), ("point", "abs", 0, 0)],
}


def shifted(a, off):
    """A copy of device tensor a that starts `off` elements into its allocation."""
    t = torch.empty(a.numel() + off, dtype=a.dtype, device=a.device)[off:]
    return t.copy_(a.reshape(-1)).view(a.shape)


@pytest.mark.parametrize("W,H", [(128, 64), (129, 65), (66, 33), (64, 31), (67, 34), (3, 2), (1, 1), (5, 40), (200, 3)])
@pytest.mark.parametrize("chain", sorted(CHAINS))
@pytest.mark.parametrize("dtype", ["u8", "f32"])
def test_blocks_and_alignment(chain, W, H, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    spec, T = CHAINS[chain], 9
    vol = np.random.default_rng(W * H).integers(0, 256, (T, H, W), dtype=np.uint8)
    x = torch.from_numpy(vol).cuda()
    if dtype == "f32":
        x = x.float()[None].contiguous()
    kw = dict(frames_per_block=4) if chain == "resumed" else {}
    fused = fz.Plan(spec, W, H, T, partition=[], in_dtype=dtype, **kw)
    out, _, _ = fused.run(x)
    ref, bound = parity.generic_reference(oracle, spec, vol)
    parity.assert_within_bound(out.cpu().numpy()[0], ref, bound, f"{chain} {W}x{H} {dtype}")
    _, _, _, ws = fused.alloc()
    for i, o in ((1, 0), (0, 1), (2, 3)):  # elements off the allocation's alignment
        y = shifted(torch.full_like(out, -1.0), o)
        fused.run(shifted(x, i), y, workspace=ws)
        assert torch.equal(y, out), (i, o)
    y, _, _ = fz.Plan(spec, W, H, T, partition="unfused", in_dtype=dtype).run(x)
    assert torch.equal(y, out)
