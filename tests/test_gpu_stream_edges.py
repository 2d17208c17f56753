"""The streaming kernels' vectors: buffers at every byte (or float) of their alignment,
clips of a few pixels, a first frame that ends inside a thread's pixels.  The reference
is integer or FP32 arithmetic in torch, equal to the bit."""
import pytest

from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(1, 1, 40), (3, 1, 7), (5, 3, 5), (15, 1, 3), (16, 1, 2), (17, 1, 4), (31, 2, 3), (61, 33, 3), (64, 16, 2), (1023, 1, 2)]


def shifted(a, off):
    """A copy of device tensor a that starts `off` elements into its allocation, guarded behind."""
    t = torch.full((a.numel() + off + 64,), 77, dtype=a.dtype, device=a.device)
    v = t[off:off + a.numel()]
    return v.copy_(a.reshape(-1)).view(a.shape), t


@pytest.mark.parametrize("op", ["framediff", "rgb2gray", "products", "threshold"])
@pytest.mark.parametrize("W,H,T", SIZES)
def test_alignment_and_edges(op, W, H, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(W * H + T)
    if op in ("framediff", "rgb2gray"):
        x = torch.randint(0, 256, (T, H, W, 3) if op == "rgb2gray" else (T, H, W), dtype=torch.uint8, device="cuda", generator=g)
        p = x.int()
        if op == "rgb2gray":
            ref = ((299 * p[..., 0] + 587 * p[..., 1] + 114 * p[..., 2] + 500) // 1000).to(torch.uint8)
        else:
            ref = (p - torch.cat([p[:1], p[:-1]])).abs().to(torch.uint8)
        shifts = [(i, o) for i in (0, 1, 2, 3, 7) for o in (0, 1, 2, 5)]
    elif op == "products":
        x = torch.randn((2, T, H, W), device="cuda", generator=g)
        ref = torch.stack([x[0] * x[0], x[0] * x[1], x[1] * x[1]])
        shifts = [(i, o) for i in (0, 1, 3) for o in (0, 1, 2)]
    else:
        x = torch.randn((1, T, H, W), device="cuda", generator=g) * 2e8
        ref = torch.where(x >= 1e8, x, torch.zeros_like(x))
        shifts = [(i, o) for i in (0, 1, 3) for o in (0, 1, 2)]
    plan = fz.Plan([op], W, H, T)
    assert plan.output_shape() == tuple(ref.shape)
    for i, o in shifts:
        y, whole = shifted(torch.zeros_like(ref), o)
        plan.run(shifted(x, i)[0], y)
        assert torch.equal(y, ref), (i, o)
        assert bool((whole[:o] == 77).all()) and bool((whole[o + ref.numel():] == 77).all())  # nothing past the buffer
