"""Streaming passes over long clips: the launch's grid (host arithmetic) and the pixels
of clips past one row of the grid, and past the 2^34 pixels that one grid dimension
could hold at 4 a thread."""
import pytest

from paper_1509_04394_amd import fz
from tests import hostcpp


@pytest.mark.parametrize("v", [4, 16])  # pixels a thread
def test_grid_stays_within_a_dimension(tmp_path, v):
    sizes = [1, 4, 1023, 1024, 1025, (1 << 30) - 1, 1 << 30, (1 << 30) + 1, 480000 * 35791, 1 << 34, (1 << 34) + 5, 1 << 40]
    out = hostcpp.run(tmp_path, ["fz_ops.h"], "".join(
        f'printf("%u %u %d\\n", stream_grid({n}ull, {v}).x, stream_grid({n}ull, {v}).y, BLOCK_THREADS);\n' for n in sizes))
    for n, line in zip(sizes, out):
        x, y, threads = map(int, line.split())
        assert 1 <= x <= 1 << 20 and 1 <= y and x * threads < 1 << 32  # threads a grid dimension can hold
        assert y == 1 or x == 1 << 20  # rows of one length, which the kernel multiplies by
        # the clip is covered, with less than a row to spare
        assert x * y * threads * v >= n and (x * (y - 1) if y > 1 else x - 1) * threads * v < n


@pytest.mark.gpu
@pytest.mark.parametrize("op,T", [("framediff", 2240), ("rgb2gray", 2240), ("framediff", 35800), ("rgb2gray", 35800)])
def test_pixels_past_one_row_of_the_grid(op, T):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    W, H, n = 799, 601, 40  # an odd frame size: every vector alignment
    C = 3 if op == "rgb2gray" else 1
    assert W * H * T > (1 << 34 if T > 10000 else 1 << 30)
    if torch.cuda.mem_get_info()[0] < 3 * C * W * H * T:
        pytest.skip("not enough device memory")
    g = torch.Generator(device="cuda").manual_seed(T)
    piece = torch.randint(0, 256, (n, H, W, 3) if C == 3 else (n, H, W), dtype=torch.uint8, device="cuda", generator=g)
    x = torch.empty((T, *piece.shape[1:]), dtype=torch.uint8, device="cuda")
    for t in range(0, T, n):
        x[t:t + n] = piece[:min(n, T - t)]
    out, _, _ = fz.Plan([op], W, H, T).run(x)
    if op == "rgb2gray":
        p = piece.int()
        ref = ((299 * p[..., 0] + 587 * p[..., 1] + 114 * p[..., 2] + 500) // 1000).to(torch.uint8)
    else:
        p = piece.int()
        ref = (p - p.roll(1, 0)).abs().to(torch.uint8)  # the frame before a piece's first is its last
    for t in range(0, T, n):
        a, b = out[t:t + n], ref[:min(n, T - t)]
        if t == 0 and op == "framediff":
            assert int(a[0].max()) == 0
            a, b = a[1:], b[1:]
        assert torch.equal(a, b), t
