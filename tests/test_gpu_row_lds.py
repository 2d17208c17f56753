"""Row groups in LDS budgets that do not hold the feature-point lists: points appended
group by group, packed or byte masks alone.  The tile engine is the reference: equal
outputs and point sets."""
import numpy as np
import pytest

from paper_1509_04394_amd import fz

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run(ops, x, W, H, T, thr, cap, **kw):
    plan = fz.Plan(ops, W, H, T, params={"threshold": thr}, partition=[], **kw)
    out, pts, cnt, ws = plan.alloc(point_capacity=cap)
    pts.fill_(-1)
    for _ in range(2):  # the second run resets the count itself
        plan.run(x, out, pts, cnt, ws)
    torch.cuda.synchronize()
    n = int(cnt.item())
    p = pts.cpu().numpy()
    assert (p[min(n, cap):] == -1).all()
    p = p[:min(n, cap)]
    return plan, out, n, p[np.lexsort(p.T[::-1])]


# chain, size, frames per item, band, budget: two and three columns a lane, the
# exchange between runs, generic groups with byte masks, groups with no masks (0 bytes)
@pytest.mark.parametrize("ops,W,H,T,tt,band,budget", [
    (fz.HARRIS_CHAIN, 192, 60, 7, 3, 16, 4096), (fz.RGB_HARRIS_CHAIN, 365, 48, 4, 2, 20, 5120),
    (fz.RGB_HARRIS_CHAIN, 365, 48, 4, 1, 6, 1536), (fz.HARRIS_CHAIN, 141, 37, 5, 5, 0, 5000),
    (fz.HARRIS_CHAIN[:-1], 130, 41, 5, 0, 16, 64), (fz.RGB_HARRIS_CHAIN[:-1], 255, 33, 3, 0, 33, 64),
    (["threshold", "nms3"], 141, 37, 6, 0, 12, 64), (["nms3", "framediff"], 141, 37, 6, 2, 16, 4096)])
@pytest.mark.parametrize("thr", [1.0, 1e8])
def test_points_without_lists_equal_the_tile_engine(ops, W, H, T, tt, band, budget, thr):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = np.random.default_rng(W + T)
    if ops[0] in ("threshold", "nms3"):
        x = torch.from_numpy(r.uniform(0, 6e9, (1, T, H, W)).astype(np.float32)).cuda()
    else:
        x = torch.from_numpy(r.integers(0, 256, (T, H, W, 3) if ops[0] == "rgb2gray" else (T, H, W), dtype=np.uint8)).cuda()
    cap = W * H * T
    _, ref, n, pts = run(ops, x, W, H, T, thr, cap, engine="tile")
    plan, out, m, got = run(ops, x, W, H, T, thr, cap, engine="row", band_h=band, frames_per_block=tt, lds_budget=budget)
    assert plan.segment_info()[0].engine == fz.FZ_ENGINE_ROW
    assert torch.equal(out, ref) and m == n and np.array_equal(got, pts)
    if n > 8:  # a capacity below the count
        _, o, m, p = run(ops, x, W, H, T, thr, n // 3, engine="row", band_h=band, frames_per_block=tt, lds_budget=budget)
        every = {tuple(q) for q in pts}
        assert m == n and torch.equal(o, ref) and len({tuple(q) for q in p}) == n // 3 and all(tuple(q) in every for q in p)


@pytest.mark.parametrize("budget", [6000, 7000])  # clip by clip without lists; one launch with low bands
def test_batches_keep_to_the_budget(budget):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    keep, clips = [], []
    bp = fz.Plan(fz.HARRIS_CHAIN, 200, 48, 9, lds_budget=budget, partition=[])
    for i, (W, H, T) in enumerate([(200, 48, 9), (131, 70, 35), (128, 300, 5)]):
        x = torch.from_numpy(np.random.default_rng(i).integers(0, 256, (T, H, W), dtype=np.uint8)).cuda()
        _, ref, n, pts = run(fz.HARRIS_CHAIN, x, W, H, T, 1e8, W * H * T, engine="tile")
        out = torch.empty((T, H, W), dtype=torch.uint8, device="cuda")
        p = torch.empty((W * H * T, 4), dtype=torch.int32, device="cuda")
        cnt = torch.zeros((1,), dtype=torch.int32, device="cuda")
        keep.append((x, ref, n, pts, out, p, cnt))
        clips.append(fz.make_clip(x, out, p, cnt, plan=bp))
    ws = fz.run_batch(bp, clips)
    for _ in range(2):
        fz.run_batch(bp, clips, ws)
        torch.cuda.synchronize()
        for x, ref, n, pts, out, p, cnt in keep:
            q = p[:n].cpu().numpy()
            assert int(cnt.item()) == n and torch.equal(out, ref) and np.array_equal(q[np.lexsort(q.T[::-1])], pts)
