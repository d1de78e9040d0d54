"""The plan that a call takes by default (CPU only: plans are chosen on the host)."""
import pytest

import paper_2001_07809_amd as sbs

SLOTS = 256 * 16   # wavefronts that the chip holds


def frame(W, H, C, block, dmax, n=None):
    return sbs.Frame(1, 1, W, H, C, W * C, 1, n or W * H // 5, block, dmax, 1, None)


def items(W, H, block, dmax, chunk, rows, tail=True):
    """(items, row steps) of a single frame: each item slides 2r rows and takes
    its own; the last 2048 items' worth of tiles has half the rows."""
    r = (block - 1) // 2
    lpad = (r + 4) & ~3
    cols = (256 - lpad - r) & ~3
    per = -(-W // cols) * ((dmax + chunk) // chunk)
    tiles = -(-H // rows)
    main = max(0, tiles - (-(-2048 // per))) if tail else tiles
    low = max(1, rows // 2)
    ntail = -(-max(H - main * rows, 0) // low)
    return per * (main + ntail), per * (main * (2 * r + rows) + ntail * (2 * r + low)) * chunk // 8


@pytest.mark.parametrize("W,H,dmax", [(640, 480, 127), (1390, 1110, 63), (1390, 1110, 255), (1920, 1080, 63), (4096, 2304, 127)])
@pytest.mark.parametrize("C", [1, 3])
@pytest.mark.parametrize("block", [33, 41, 47, 61, 81, 101, 127])
def test_window_starts_do_not_outweigh_the_rows(W, H, dmax, C, block):
    """Where 8-disparity items of 32 rows fill half of the chip, the plan of a
    large window slides over no more than 1.6 times their rows (grey, block 101,
    1390x1110: 2.9 times when the window's size did not count)."""
    p = sbs.get_plan(frame(W, H, C, block, dmax))
    ref, steps = items(W, H, block, dmax, 8, 32, tail=False)
    if ref >= SLOTS // 2:
        assert items(W, H, block, dmax, p["chunk"], p["tile_rows"])[1] <= 1.6 * steps, p


@pytest.mark.parametrize("W,H,dmax", [(384, 288, 15), (640, 480, 31), (1390, 1110, 63), (4096, 2304, 127), (4096, 2304, 15)])
def test_sums_that_do_not_pack_take_8_disparities(W, H, dmax):
    """RGB windows above 42 columns run 16 disparities as two passes of 8."""
    for block in (43, 63, 127):
        assert sbs.get_plan(frame(W, H, 3, block, dmax))["chunk"] == 8


def test_small_windows_by_launch_size():
    """Blocks up to 31: the smallest items for a launch that cannot fill the
    chip, taller ones as it grows."""
    rows = [sbs.get_plan(frame(W, H, C, b, d))["tile_rows"]
            for W, H, C, b, d in ((384, 288, 1, 15, 15), (1390, 1110, 3, 21, 63), (5000, 3000, 3, 31, 200), (8192, 4608, 3, 31, 127))]
    assert rows == [8, 16, 32, 64]


def test_plans_between_two_and_three_times_the_slots():
    """One frame: 16 disparities and 16 rows, but 8 x 32 for windows above 21
    whose last 16 disparities are half empty; several: 16 x 32."""
    def plan(*a):
        p = sbs.get_plan(frame(*a))
        return p["chunk"], p["tile_rows"]
    for C in (1, 3):
        assert plan(3072, 2304, C, 15, 74) == (16, 16)
        assert plan(3072, 2304, C, 15, 70) == (16, 16)
        assert plan(3072, 2304, C, 31, 74) == (16, 16)
        assert plan(2552, 1600, C, 31, 116) == (8, 32)
        assert plan(2552, 1600, C, 21, 116) == (16, 16)
        f = [frame(1390, 1110, C, 31, 63)] * 5
        p = sbs.Plan()
        arr = (sbs.Frame * len(f))(*f)
        import ctypes
        assert sbs.lib().sbs_get_plan_batched(arr, len(f), ctypes.byref(p)) == 0
        assert (p.chunk, p.tile_rows) == (16, 32)


@pytest.mark.parametrize("C", [1, 3])
def test_fewer_than_8_disparities_take_8(C):
    """Items of 16 disparities would be half empty."""
    for W, H in ((1390, 1110), (1920, 1080), (4096, 2304)):
        for block in (9, 31):
            for dmax in (0, 7):
                assert sbs.get_plan(frame(W, H, C, block, dmax))["chunk"] == 8
    assert sbs.get_plan(frame(4096, 2304, C, 31, 8))["chunk"] == 16
    assert sbs.get_plan(frame(384, 288, C, 127, 15))["tile_rows"] == 8


@pytest.mark.parametrize("C", [1, 3])
@pytest.mark.parametrize("block", [9, 21, 31, 33, 41])
def test_one_frame_s_tiles_are_low_enough_for_a_region(C, block):
    """The pixels of one region of the image lie in few tiles of 32 rows and more:
    frames of up to six times the slots take 24 rows at most, or 32 by 8
    disparities, as they did before plans went by size; large windows 32."""
    for W, H, dmax in ((1390, 1110, 255), (2902, 1473, 255), (4096, 2304, 127)):
        p = sbs.get_plan(frame(W, H, C, block, dmax))
        assert p["tile_rows"] <= (32 if p["chunk"] == 8 or block > 31 else 24), p
