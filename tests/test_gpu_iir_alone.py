"""A lone IIR stage runs a kernel of its own: the frames it loads ahead must be in flight
together for both input types, so it is no slower than with a point stage behind it (which
the general kernel runs), and gives the same values."""
import pytest

from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def best_ms(run):
    times = []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times[2:])


@pytest.mark.parametrize("dtype", ["f32", "u8"])
@pytest.mark.parametrize("W,H,T", [(192, 432, 600), (640, 480, 203)])
def test_lone_iir_keeps_its_loads_in_flight(W, H, T, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randint(0, 256, (T, H, W), dtype=torch.uint8, device="cuda", generator=g)
    if dtype == "f32":
        x = x.float()[None].contiguous()
    one = fz.Plan([("iir", 0.3)], W, H, T, in_dtype=dtype)
    two = fz.Plan([("iir", 0.3), ("point", "affine", 1.0, 0.0)], W, H, T, in_dtype=dtype, partition=[])
    b1, b2 = one.alloc(), two.alloc()
    t1, t2 = best_ms(lambda: one.run(x, *b1)), best_ms(lambda: two.run(x, *b2))
    assert torch.equal(b1[0], b2[0])
    # (a quarter for the spread of two event-timed launches)
    assert t1 <= 1.25 * t2, (t1, t2)
