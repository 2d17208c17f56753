"""Frame runs of a frame-difference group when its exchange words do not fit the
workspace (rowgeom.h: row_run)."""
import pytest

from tests import hostcpp

ROOM = 64 << 20


# a clip, its planned band and run, columns a lane, wavefronts at once; words that fit,
# words that do not, runs that reach the whole clip, a clip of a single run
@pytest.mark.parametrize("W,H,T,band,tt,K,slots", [
    (640, 480, 1000, 96, 1, 2, 6144), (640, 480, 400, 48, 1, 2, 6144), (800, 600, 700, 100, 1, 2, 5120),
    (800, 600, 1000, 86, 2, 2, 5120), (192, 432, 4000, 108, 1, 3, 4096), (1280, 720, 256, 72, 1, 2, 6144),
    (1920, 1080, 20000, 216, 8, 2, 6144), (128, 240, 33000, 240, 1, 2, 6144), (800, 600, 256, 8, 1, 2, 6144),
    (160, 100, 5, 100, 5, 2, 6144), (160, 100, 5, 20, 4, 2, 6144)])
@pytest.mark.parametrize("room", [ROOM, ROOM // 64, 0])
def test_run_that_fits_or_recomputes(tmp_path, W, H, T, band, tt, K, slots, room):
    span = 64 * K
    ns, nb = 1 + max(0, -(-(W - span) // (span - 12))), -(-H // band)
    out = hostcpp.run(tmp_path, ["rowgeom.h"], f"""
        const RowRun r = row_run({room}, {T}, {ns}, {nb}, {band}, {K}, {tt}, {slots});
        printf("%d %d %d\\n", r.tt, r.nchunks, (int)r.exchange);
        printf("%zu\\n", row_exchange_bytes({ns}, {nb}, {-(-T // tt)}, {band}, {K}));
        printf("%zu\\n", row_exchange_bytes({ns}, {nb}, r.nchunks, {band}, {K}));
        printf("%.17g\\n", row_time({band}, r.tt + (r.nchunks == 1 ? 0.0 : r.exchange ? 0.15 : 1.0),
                                    (double){ns} * {nb} * r.nchunks, {slots}));
        printf("%.17g\\n", row_time({band}, {tt} + 1.0, {ns * nb * -(-T // tt)}, {slots}));
    """)
    run, chunks, exchange = map(int, out[0].split())
    planned, used, modelled, recompute = int(out[1]), int(out[2]), float(out[3]), float(out[4])
    assert tt <= run <= T and chunks == -(-T // run)
    if planned <= room:
        assert run == tt and exchange == (T > tt)
    else:
        assert not exchange or used <= room
        # never the planned run recomputed where the model knows better
        assert modelled <= recompute
        if (W, H, T) == (640, 480, 1000) and room == ROOM:
            assert exchange and run == 2 and modelled < 0.7 * recompute
