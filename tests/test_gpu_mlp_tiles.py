"""The cost network's matrix-core kernel at the edges of its sample tiles, feature
groups and workgroup count, against the FP64 oracle (oracle/mlp.py)."""
import numpy as np
import pytest

from oracle import mlp
from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# samples around the 32-row tiles and past the 512 workgroups (several tiles
# each); features around the groups of four and the two 16-column tiles
@pytest.mark.parametrize("n,F", [(1, 1), (31, 3), (32, 4), (33, 5), (64, 16), (65, 17), (500, 20), (16385, 31),
                                 (40001, 32)])
def test_step_at_tile_edges(n, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(1000 * F + n)
    p = mlp.init(F, seed=n).astype(np.float32)
    x = rng.normal(size=(n, F)).astype(np.float32)
    t = (np.sin(x[:, 0]) + 0.1 * x.sum(1)).astype(np.float32)
    dp, dx, dt = (torch.tensor(a, device="cuda") for a in (p, x, t))
    need = fz.fz_mlp_workspace_bytes(F, n)
    ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    g = torch.empty(p.size, device="cuda")
    L = torch.empty(1, device="cuda")
    y = torch.full((n + 64,), 7.0, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    fz.fz_mlp_loss_grad(dp.data_ptr(), F, dx.data_ptr(), dt.data_ptr(), n, g.data_ptr(), L.data_ptr(), ws.data_ptr(),
                        need, s)
    fz.fz_mlp_forward(dp.data_ptr(), F, dx.data_ptr(), n, y.data_ptr(), s)
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xA5).all()) and bool((y[n:] == 7.0).all())  # nothing past the buffers
    p64, x64, t64 = p.astype(np.float64), x.astype(np.float64), t.astype(np.float64)
    ref = mlp.forward(p64, x64, F)
    assert np.max(np.abs(y[:n].cpu().numpy() - ref)) <= 1e-5 * (1 + np.max(np.abs(ref)))
    Lr, gr = mlp.loss_grad(p64, x64, t64, F)
    assert abs(L.item() - Lr) <= 1e-5 * max(1.0, Lr)
    gg = g.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(gg - gr) <= 1e-4 * np.linalg.norm(gr)
