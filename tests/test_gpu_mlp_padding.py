"""The cost network's gradient where the last tile of samples is not full: the rows past
the last sample must add nothing, whatever a sample of zeros would have given."""
import numpy as np
import pytest

from oracle import mlp
from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 5, 31, 33, 40, 97])
def test_rows_past_the_last_sample_add_nothing(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    F, h = 20, 64
    rng = np.random.default_rng(n)
    p = mlp.init(F, seed=n).astype(np.float32)
    x = rng.normal(size=(n, F)).astype(np.float32)
    t = x.sum(1)
    # eight hidden units whose bias the first feature cancels exactly in every
    # sample; in a sample of zeros they reach 3e38 and the next layer overflows
    x[:, 0] = 2.0
    w1, b1 = p[:h * F].reshape(h, F), p[h * F:h * F + h]
    b1[:8] = 3e38
    w1[:8] = 0.0
    w1[:8, 0] = -b1[:8] / 2
    w1[8:, 0] = 0.1
    p[h * F + h:h * F + h + h * h].reshape(h, h)[:4, :8] = 1.0
    dp, dx, dt = (torch.tensor(a, device="cuda") for a in (p, x, t.astype(np.float32)))
    ws = torch.empty(fz.fz_mlp_workspace_bytes(F, n), dtype=torch.uint8, device="cuda")
    g, L = torch.empty(p.size, device="cuda"), torch.empty(1, device="cuda")
    fz.fz_mlp_loss_grad(dp.data_ptr(), F, dx.data_ptr(), dt.data_ptr(), n, g.data_ptr(), L.data_ptr(), ws.data_ptr(),
                        ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    Lr, gr = mlp.loss_grad(p.astype(np.float64), x.astype(np.float64), dt.cpu().numpy().astype(np.float64), F)
    gg = g.cpu().numpy().astype(np.float64)
    assert np.isfinite(gr).all() and np.isfinite(gg).all()
    assert abs(L.item() - Lr) <= 1e-5 * max(1.0, Lr)
    assert np.linalg.norm(gg - gr) <= 1e-4 * np.linalg.norm(gr)
