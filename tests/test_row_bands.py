"""Bands of the generic row kernel on short clips: the last workgroups of a launch must
not land on a compute unit that already has its share when slightly taller bands avoid it."""
import pytest

from paper_1509_04394_amd import fz

HALO = {"gauss5": 2, "sobel3": 1, "boxsum5": 2, "nms3": 1}


def rows_in_turn(W, H, T, ops, band):
    strips = 1 + -(-(W - 128) // (128 - 2 * sum(HALO.get(o, 0) for o in ops)))
    workgroups = -(-strips * -(-H // band) * T // 4)
    return band * -(-workgroups // 256), strips * -(-H // band) * T


@pytest.mark.parametrize("ops", [fz.RGB_HARRIS_CHAIN[:4], fz.HARRIS_CHAIN[:2], fz.HARRIS_CHAIN[2:4], ["boxsum5"],
                                 ["threshold", "nms3"], fz.GRAD_CHAIN], ids="-".join)
@pytest.mark.parametrize("W,H,T", [(333, 251, 40), (192, 432, 64), (128, 96, 300), (150, 70, 60), (641, 479, 5),
                                   (320, 240, 4), (130, 9, 3), (203, 77, 33), (800, 600, 8)])
def test_short_clips_take_the_height_with_fewest_rows_in_turn(ops, W, H, T):
    s = fz.Plan(ops, W, H, T, partition=[]).segment_info()[0]
    assert s.engine == fz.FZ_ENGINE_ROW
    turn, _ = rows_in_turn(W, H, T, ops, s.tile_h)
    for rows in (14, 15, 16):
        even = -(-H // max(1, (H + rows // 2) // rows))
        assert turn <= rows_in_turn(W, H, T, ops, even)[0], (s.tile_h, even)


def test_a_third_workgroup_a_compute_unit_is_avoided():
    assert fz.Plan(fz.RGB_HARRIS_CHAIN[:4], 333, 251, 40, partition=[]).segment_info()[0].tile_h == 15
    # and where it is not the third, the shorter bands stay
    assert fz.Plan(fz.GRAD_CHAIN, 192, 432, 64).segment_info()[0].tile_h == 14
