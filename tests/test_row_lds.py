"""LDS of the row groups against the plan's budget: what the kernels hold (packed or byte
masks, point lists), not only the figure a plan states, has to fit."""
import itertools

import pytest

from paper_1509_04394_amd import fz
from tests import hostcpp

RGB, GRAY = fz.RGB_HARRIS_CHAIN, fz.HARRIS_CHAIN


def lists(k):
    return 4 * (256 * (2 + k) + 32) + 8


def masks(k, band):
    rows, pitch = (15, 20) if k == 2 else (5, 52)
    return 4 * -(-band // rows) * rows * pitch


def planned(ops, W, H, T, budget, **kw):
    try:
        return fz.Plan(ops, W, H, T, partition=[], lds_budget=budget, **kw).segment_info()[0]
    except fz.FzError as e:
        assert e.code == fz.FZ_E_LDS
        return None


def test_budget_below_what_the_kernel_holds_is_refused():
    # 16 rows of mask bytes (4096) are the least; a 4-row band was taken as "1024 bytes" and held 5432
    for budget in (256, 1024, 2048, 4095):
        assert planned(RGB, 320, 240, 4, budget) is None
    for budget in (4096, 5431, 5432, 8192, 65536):
        s = planned(RGB, 320, 240, 4, budget)
        k = s.tile_w // 64
        assert s.lds_bytes <= budget and masks(k, s.tile_h) <= budget


@pytest.mark.parametrize("ops,W,H,T", [(RGB, 800, 600, 1000), (GRAY, 800, 600, 1000), (RGB, 192, 432, 600),
                                       (RGB, 365, 300, 60), (GRAY, 150, 70, 100)])
def test_bands_follow_the_budget(ops, W, H, T):
    free = planned(ops, W, H, T, 0)
    taken = []
    for budget in (4096, 5000, 6144, 7000, 8192, 12000, 16384, 19200, 20000, 22016, 32768, 65536, 163840):
        s = planned(ops, W, H, T, budget)
        taken.append(s is not None)
        if s is None:
            continue
        k = s.tile_w // 64
        assert s.engine == fz.FZ_ENGINE_ROW and s.lds_bytes == 256 * s.tile_h <= budget and masks(k, s.tile_h) <= budget
        if budget >= 65536:
            assert (s.tile_w, s.tile_h, s.frames_per_block) == (free.tile_w, free.tile_h, free.frames_per_block)
    # a larger budget takes what a smaller one takes; 19,200 bytes (75 rows) are enough for the largest clip
    assert taken == sorted(taken) and all(taken[7:])


@pytest.mark.parametrize("ops,generic", [(["nms3", "framediff"], True), (RGB, False)])
def test_short_frames_at_every_budget(ops, generic):
    for H in (8, 15, 16, 17, 18, 31, 33, 40):
        taken = False
        for budget in range(2000, 10000, 97):
            s = planned(ops, 160, H, 6, budget)
            if s is None:
                assert not taken and budget < 256 * H
                continue
            taken = True
            held = 256 * s.tile_h if generic else masks(s.tile_w // 64, s.tile_h)
            assert 1 <= s.tile_h <= H and s.lds_bytes <= budget and held <= budget
        assert taken


def test_groups_without_masks_need_no_budget():
    # (their points are appended without lists below the lists' size)
    for budget in (64, 4000, 4232, 5256, 10000):
        for ops in (RGB[:8], GRAY[:7], ["threshold", "nms3"], ["nms3"]):
            s = planned(ops, 320, 240, 4, budget)
            assert s.engine == fz.FZ_ENGINE_ROW and s.lds_bytes == 0
    # every stage alone fits a small budget, so a plan exists
    fz.Plan(GRAY[:7], 320, 240, 4, lds_budget=512)


@pytest.mark.parametrize("W,band", [(800, 5), (800, 16), (800, 75), (800, 256), (365, 6), (365, 16), (365, 128), (192, 11)])
def test_requested_bands_are_kept_within_the_stated_bytes(W, band):
    # from five rows on, a requested band runs in its stated 256 bytes a row
    s = planned(RGB, W, 300, 10, 256 * band, engine="row", band_h=band)
    k = s.tile_w // 64
    assert s.tile_h == band and masks(k, band) <= 256 * band
    assert planned(RGB, W, 300, 10, 256 * band - 1, engine="row", band_h=band) is None


def test_header_counts_the_same_bytes(tmp_path):
    cases = list(itertools.product((2, 3), (1, 4, 5, 15, 16, 86, 256), (0, 1)))
    out = hostcpp.run(tmp_path, ["rowgeom.h"], "".join(
        f'printf("%d\\n", row_held_bytes(false, {k}, {b}, true, {l}));' for k, b, l in cases))
    assert [int(v) for v in out] == [masks(k, b) + (lists(k) if l else 0) for k, b, l in cases]


@pytest.mark.parametrize("W,H,T", [(365, 800, 10000), (729, 600, 10000), (192, 600, 20000), (365, 1000, 4000)])
@pytest.mark.parametrize("ops", [RGB, GRAY], ids=["rgb", "gray"])
def test_tall_bands_leave_room_for_the_wavefronts(ops, W, H, T):
    # four wavefronts a SIMD with three columns a lane, as the registers allow: the
    # sizing counts them, so four workgroups must fit a compute unit
    s = planned(ops, W, H, T, 0)
    k = s.tile_w // 64
    assert (4 if k == 3 else 6 if ops is GRAY else 5) * (masks(k, s.tile_h) + lists(k)) <= 163840
