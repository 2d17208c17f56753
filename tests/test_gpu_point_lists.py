"""Feature points of the row-marching kernels: lists that overflow, capacities below
the count, several frames and items per list.  The tile engine (one append per
group of points) is the reference: the point sets and outputs must be equal."""
import numpy as np
import pytest

from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
RGB7, GRAY7 = fz.RGB_HARRIS_CHAIN[:-1], fz.HARRIS_CHAIN[:-1]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def noise(W, H, T, C, seed):
    r = np.random.default_rng(seed)
    return r.integers(0, 256, (T, H, W, 3) if C == 3 else (T, H, W), dtype=np.uint8)


def run(ops, x, W, H, T, thr, cap, dev, **kw):
    plan = fz.Plan(ops, W, H, T, params={"threshold": thr}, **kw)
    out, pts, cnt, ws = plan.alloc(dev, point_capacity=cap)
    pts.fill_(-1)
    plan.run(x, out, pts, cnt, ws)
    torch.cuda.synchronize()
    n = int(cnt.item())
    p = pts.cpu().numpy()
    assert (p[min(n, cap):] == -1).all()
    p = p[:min(n, cap)]
    return out, n, p[np.lexsort(p.T[::-1])]


# chain, size, frames per item, band: dense noise fills a 64-entry list several
# times in a frame; 365 RGB columns take three columns a lane; a band of 250 rows
# passes 64 KB of LDS with the lists
@pytest.mark.parametrize("ops,W,H,T,tt,band", [
    (fz.HARRIS_CHAIN, 192, 60, 7, 3, 30), (fz.RGB_HARRIS_CHAIN, 365, 48, 4, 2, 20), (GRAY7, 130, 41, 5, 0, 16),
    (RGB7, 255, 33, 3, 0, 33), (fz.HARRIS_CHAIN, 128, 250, 3, 2, 250), (["threshold", "nms3"], 141, 37, 6, 0, 12),
    (["nms3", "framediff"], 141, 37, 6, 2, 12)])
@pytest.mark.parametrize("thr", [1.0, 1e8, 3e9])
def test_dense_points_equal_the_tile_engine(dev, ops, W, H, T, tt, band, thr):
    C = 3 if ops[0] == "rgb2gray" else 1
    if ops[0] in ("threshold", "nms3"):
        r = np.random.default_rng(W)
        x = torch.from_numpy(r.uniform(0, 6e9, (1, T, H, W)).astype(np.float32)).to(dev)
        if ops[0] == "nms3" and thr != 1.0:
            pytest.skip("no threshold stage")
    else:
        x = torch.from_numpy(noise(W, H, T, C, W + T)).to(dev)
    cap = W * H * T
    ref = run(ops, x, W, H, T, thr, cap, dev, partition=[], engine="tile")
    got = run(ops, x, W, H, T, thr, cap, dev, partition=[], engine="row", band_h=band, frames_per_block=tt)
    assert torch.equal(ref[0], got[0]) and ref[1] == got[1] and np.array_equal(ref[2], got[2])
    if ref[1] > 8:  # a capacity below the count: counted in full, the buffer filled, nothing past it
        cap = ref[1] // 3
        o, n, p = run(ops, x, W, H, T, thr, cap, dev, partition=[], engine="row", band_h=band, frames_per_block=tt)
        assert n == ref[1] and torch.equal(o, ref[0])
        every = {tuple(q) for q in ref[2]}
        assert len({tuple(q) for q in p}) == cap and all(tuple(q) in every for q in p)


def test_dense_points_in_a_batch(dev):
    bp = fz.Plan(fz.HARRIS_CHAIN, 200, 48, 9, params={"threshold": 1.0})
    keep, clips = [], []
    for i, (W, H, T) in enumerate([(200, 48, 9), (131, 70, 35), (128, 9, 1)]):
        x = torch.from_numpy(noise(W, H, T, 1, i)).to(dev)
        ref = run(fz.HARRIS_CHAIN, x, W, H, T, 1.0, W * H * T, dev, partition=[], engine="tile")
        out = torch.empty((T, H, W), dtype=torch.uint8, device=dev)
        pts = torch.empty((W * H * T, 4), dtype=torch.int32, device=dev)
        cnt = torch.zeros((1,), dtype=torch.int32, device=dev)
        keep.append((x, ref, out, pts, cnt))
        clips.append(fz.make_clip(x, out, pts, cnt, plan=bp))
    ws = fz.run_batch(bp, clips)
    for _ in range(2):
        fz.run_batch(bp, clips, ws)
        torch.cuda.synchronize()
        for x, ref, out, pts, cnt in keep:
            p = pts[:ref[1]].cpu().numpy()
            assert int(cnt.item()) == ref[1] and torch.equal(out, ref[0])
            assert np.array_equal(p[np.lexsort(p.T[::-1])], ref[2])


def test_frame_numbers_past_a_list_entry(dev):
    # one item of 65,600 frames: an entry holds 16 bits of the frame's number in its item
    W, H, T = 128, 8, 65600
    x = torch.zeros((T, H, W), dtype=torch.uint8, device=dev)
    for t in (0, 5, 65535, 65536, 65537, 65599):
        x[t, 2:5, 40:60] = 200
    cap = 4096
    ref = run(GRAY7, x, W, H, T, 1e6, cap, dev, partition=[], engine="tile")
    got = run(GRAY7, x, W, H, T, 1e6, cap, dev, partition=[], engine="row", band_h=8, frames_per_block=T)
    assert ref[1] > 0 and ref[1] == got[1] and np.array_equal(ref[2], got[2]) and torch.equal(ref[0], got[0])


# bands around the 15 rows of a packed mask word (5 with three columns a lane),
# runs that meet at every frame, the recomputing path beside the exchange
@pytest.mark.parametrize("ops,W,band", [(fz.HARRIS_CHAIN, 130, b) for b in (8, 14, 15, 16, 29, 30, 31, 44)] +
                         [(fz.RGB_HARRIS_CHAIN, 365, b) for b in (8, 9, 10, 11, 26)])
@pytest.mark.parametrize("tt", [1, 3])
def test_packed_masks_meet_at_run_boundaries(dev, ops, W, band, tt):
    H, T = 45, 8
    x = torch.from_numpy(noise(W, H, T, 3 if W == 365 else 1, band)).to(dev)
    ref = run(ops, x, W, H, T, 1e7, W * H * T, dev, partition=[], engine="tile")
    got = run(ops, x, W, H, T, 1e7, W * H * T, dev, partition=[], engine="row", band_h=band, frames_per_block=tt)
    assert torch.equal(ref[0], got[0]) and ref[1] == got[1] and np.array_equal(ref[2], got[2])


def test_static_run_recomputes_where_the_exchange_does_not_fit(dev):
    # 7 strips x 75 bands x 255 boundaries of 512 bytes: 69 MB of exchange words
    W, H, T = 800, 600, 256
    plan = fz.Plan(fz.HARRIS_CHAIN, W, H, T, partition=[], engine="row", band_h=8, frames_per_block=1)
    assert plan.workspace_bytes > fz.FZ_STATIC_WORKSPACE_BYTES
    x = torch.from_numpy(noise(W, H, 8, 1, 3)).to(dev).repeat(T // 8, 1, 1).contiguous()
    ref, rp, rc = plan.run(x, *plan.alloc(dev, point_capacity=1))
    out, pts, cnt, _ = plan.alloc(dev, point_capacity=1)
    plan.run_static(x, out, pts, cnt)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and int(cnt.item()) == int(rc.item())
