"""Batches on the host: what is checked before a launch, and the cost of sizing a batch."""
import time

import pytest

from paper_1509_04394_amd import fz


def clip(W, H, T):
    c = fz.fz_clip()
    c.width, c.height, c.frames = W, H, T
    c.d_in = c.d_out = 0x1000  # never dereferenced: the checks come first
    return c


@pytest.mark.parametrize("partition", ["optimal", "unfused"])
def test_workspace_is_checked_before_any_launch(partition):
    plan = fz.Plan(fz.HARRIS_CHAIN, 320, 240, 20, partition=partition)
    clips = [clip(320, 240, 20), clip(160, 120, 9)]
    need = fz.fz_batch_workspace_bytes(plan.handle, clips)
    assert need > 256
    for ws, size in ((0x1000, need - 1), (0x1000, 0), (None, need)):
        with pytest.raises(fz.FzError) as e:
            fz.fz_run_batch(plan.handle, clips, ws, size, None)
        assert e.value.code == fz.FZ_E_WORKSPACE


def test_sizing_a_batch_tries_each_band_once():
    # 32 clips of 4000 rows: some 120 different bands each, not the 1000 cuts of the frame
    plan = fz.Plan(fz.HARRIS_CHAIN, 800, 600, 100)
    one, many = [clip(800, 60, 100)] * 32, [clip(800, 4000, 100)] * 32

    def best(clips):
        fz.fz_batch_workspace_bytes(plan.handle, clips)
        t = []
        for _ in range(50):
            a = time.perf_counter()
            fz.fz_batch_workspace_bytes(plan.handle, clips)
            t.append(time.perf_counter() - a)
        return min(t)

    # (bands grow with the root of the height, 8 times; cuts with the height, 67 times)
    assert best(many) < 14 * best(one)
