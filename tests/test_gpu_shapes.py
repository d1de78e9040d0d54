"""Calls at the ends of the size ranges: results against the oracle, and times
against a call of about as much work and an ordinary shape, where an algorithm
that is serial along one axis of the image shows as a large factor."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def sbs():
    import paper_2001_07809_amd as m
    m.lib()
    return m


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def call_us(torch, fn, reps=10, rounds=5):
    """Microseconds per call, the best of some rounds of calls in a row."""
    for _ in range(2):
        fn()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            fn()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


def component_images():
    """Images whose boundary maps hold components as long as the image."""
    rng = np.random.default_rng(5)
    noise = lambda W, H: rng.integers(0, 256, (H, W), dtype=np.uint8)
    checks = lambda W, H: ((((np.arange(W) // 5)[None, :] ^ (np.arange(H) // 5)[:, None]) & 1) * 150).astype(np.uint8)
    ramp = lambda W, H: np.repeat((np.arange(W) * 255 // max(W - 1, 1)).astype(np.uint8)[None, :], H, 0)
    return [("noise 100000x20", noise(100000, 20), 10, 1),   # paper mode leaves the frame: two lines that meet at the ends
            ("ramp 3x20000", ramp(3, 20000), 10, 1),         # a ring of one column on either side
            ("checks 40x60000", checks(40, 60000), 4, 0),    # a grid all along the image
            ("checks 60000x40", checks(60000, 40), 4, 0),
            ("noise 65x20011", noise(65, 20011), 4, 0)]


@pytest.mark.parametrize("i", range(5))
def test_components_along_the_image(torch, sbs, i):
    what, img, K, mode = component_images()[i]
    got, kept, _ = sbs.boundaries(dev(torch, img), K=K, mode=mode, min_cc=20, with_maps=True)
    exp, exp_map = oracle.boundaries(img, K=K, mode=mode, min_cc=20, frac=-1.0, return_map=True)
    assert np.array_equal(kept.cpu().numpy(), exp_map), what
    assert np.array_equal(got.cpu().numpy().view(np.uint32), exp), what


def test_components_along_the_image_take_no_walk_of_it(torch, sbs):
    """Two lines of 1,563 tiles that meet at both ends, against noise of as many
    pixels in a square: 7.4 times the call when one thread walked a line, 1.2
    times when its tiles shorten the way together."""
    rng = np.random.default_rng(6)
    wide = dev(torch, rng.integers(0, 256, (20, 100000), dtype=np.uint8))
    square = dev(torch, rng.integers(0, 256, (1414, 1414), dtype=np.uint8))
    t = [call_us(torch, lambda: sbs.boundaries(img, K=10, mode=1)) for img in (wide, square)]
    assert t[0] < 3 * t[1], t


def check_reconstruct(torch, sbs, idx, disp, W, H, what):
    exp = oracle.reconstruct(idx, disp, W, H, 1)
    got = sbs.reconstruct(dev(torch, idx.view(np.int32)), dev(torch, disp), W, H, 1).cpu().numpy()
    assert np.array_equal(got, exp), f"{what}: {(got != exp).sum()} pixels differ"


@pytest.mark.parametrize("W,H", [(5, 40), (7, 2049), (40, 2500), (4096, 300)])
def test_reconstruct_rows_without_entries(torch, sbs, W, H):
    """Ordered lists with runs of empty rows around the length that one thread
    writes (32 rows), before the first entry, after the last one, and several
    long ones in one thread's and in one block's entries."""
    rng = np.random.default_rng(H)
    N = W * H
    lists = {"first": [0], "last": [N - 1], "ends": [0, N - 1], "past the image": [N // 2, N + 3, N + 4]}
    for step in (2, 31, 32, 33, 34, 300):
        lists[f"every {step} rows"] = np.arange(0, H, step) * W + W // 2
    lists["few"] = np.sort(rng.choice(N, 6, replace=False))
    lists["clusters"] = np.concatenate([np.arange(40) + at for at in (0, N // 3, N // 2, N - 40)])
    for what, lst in lists.items():
        idx = np.asarray(lst, dtype=np.uint32)
        check_reconstruct(torch, sbs, idx, rng.integers(0, 4, idx.size).astype(np.uint8), W, H, f"{W}x{H} {what}")


def test_reconstruct_rows_without_entries_are_written_by_many(torch, sbs):
    """One entry in 200,000 rows against an 18% list of the same image: 13 times
    the call when one thread wrote all rows' starts, less than it otherwise."""
    W, H = 64, 200000
    rng = np.random.default_rng(1)
    lists = [np.array([W * H - 1]), np.sort(rng.choice(W * H, W * H * 18 // 100, replace=False))]
    t = []
    for lst in lists:
        idx, disp = dev(torch, lst.astype(np.int32)), dev(torch, (lst % 60).astype(np.uint8))
        t.append(call_us(torch, lambda: sbs.reconstruct(idx, disp, W, H, 1)))
    assert t[0] < 2 * t[1], t


@pytest.mark.parametrize("W,H", [(3, 700), (64, 40), (255, 60), (256, 61), (1000, 33), (4096, 9)])
def test_reconstruct_rows_of_many_repeats(torch, sbs, W, H):
    """Ordered lists with one pixel repeated around the number of entries from
    which a row's list counts as one in no order (the row's width, at least 256,
    and 256 more), in the first, a middle and the last row; pixels repeated a
    few times all over a row; and entries past the image in such numbers."""
    rng = np.random.default_rng(W)
    N = W * H
    base = np.sort(rng.choice(N, max(N // 7, 3), replace=False))
    most = max(W, 256)
    for at in (0, N // 2, N - 1):
        for times in (2, 63, 64, 65, 511, 512, 513, most - 1, most + 1, most + 255, most + 256, most + 257, most + 1400):
            idx = np.sort(np.concatenate([base, np.full(times, at)])).astype(np.uint32)
            check_reconstruct(torch, sbs, idx, rng.integers(0, 3, idx.size).astype(np.uint8), W, H, f"{W}x{H} {at} {times} times")
    for times in (2, 3, 9):
        idx = np.repeat(np.arange(N // 2, min(N // 2 + W, N)), times).astype(np.uint32)
        check_reconstruct(torch, sbs, idx, rng.integers(0, 3, idx.size).astype(np.uint8), W, H, f"{W}x{H} a row {times} times")
    idx = np.concatenate([base, np.full(3000, N), np.full(3000, N + 5)]).astype(np.uint32)
    check_reconstruct(torch, sbs, idx, rng.integers(0, 3, idx.size).astype(np.uint8), W, H, f"{W}x{H} past the image")


def test_reconstruct_repeats_are_taken_by_many(torch, sbs):
    """A tenth as many entries on one pixel as the image has pixels, beside a 1%
    list, against that list: 25 times the call when one wavefront took them all."""
    W, H = 1390, 1110
    rng = np.random.default_rng(2)
    few = np.sort(rng.choice(W * H, W * H // 100, replace=False))
    lists = [np.sort(np.concatenate([few, np.full(W * H // 10, W * H // 2)])), few]
    t = []
    for lst in lists:
        idx, disp = dev(torch, lst.astype(np.int32)), dev(torch, (lst % 60).astype(np.uint8))
        t.append(call_us(torch, lambda: sbs.reconstruct(idx, disp, W, H, 1)))
    assert t[0] < 4 * t[1], t


@pytest.mark.parametrize("W,H", [(1560, 256), (1560, 257), (1555, 257), (400, 999), (392, 1023), (391, 1024), (391, 1023),
                                 (4096, 98), (2, 1500), (64, 17), (200, 16)])
def test_reconstruct_paths(torch, sbs, W, H):
    """Images around the sizes from which a list is checked (400,000 pixels, 257
    rows), a row goes to one wavefront whatever the list (1,024 rows) and a
    column's segments to several (17 of 16 rows), with lists in order and not, of
    at most half of the pixels and of more."""
    rng = np.random.default_rng(W * H)
    N = W * H
    for n in (N * 18 // 100, N // 2, N // 2 + 1, N):
        idx = np.sort(rng.choice(N, n, replace=False)).astype(np.uint32)
        lists = {"in order": idx, "in no order": rng.permutation(idx)}
        one = idx.copy()
        one[[n // 3, n // 3 + 1]] = one[[n // 3 + 1, n // 3]]
        lists["one descent"] = one
        for what, lst in lists.items():
            check_reconstruct(torch, sbs, lst, rng.integers(0, 4, n).astype(np.uint8), W, H, f"{W}x{H}, {n} entries {what}")


def test_reconstruct_few_long_rows_take_no_longer_than_an_image(torch, sbs):
    """All pixels of 4000x100, and a shuffled 18% of them, against an ordered 18%
    of 640x480: 1.5 times the call when a wavefront took a row of either."""
    rng = np.random.default_rng(3)
    t = []
    for W, H, share, shuffle in ((640, 480, 0.18, False), (4000, 100, 1.0, False), (4000, 100, 0.18, True)):
        lst = rng.choice(W * H, int(W * H * share), replace=False)
        lst = lst if shuffle else np.sort(lst)
        idx, disp = dev(torch, lst.astype(np.int32)), dev(torch, (lst % 60).astype(np.uint8))
        t.append(call_us(torch, lambda: sbs.reconstruct(idx, disp, W, H, 1), reps=30))
    assert max(t[1:]) < 1.3 * t[0], t


def search_inputs(torch, W, H, seed):
    rng = np.random.default_rng(seed)
    left = rng.integers(0, 256, (H, W, 3), dtype=np.uint8)
    idx = np.sort(rng.choice(W * H, W * H * 18 // 100, replace=False)).astype(np.uint32)
    return left, np.roll(left, -4, axis=1), idx


def test_per_frame_launches_take_each_frame_s_plan(torch, sbs):
    """Frames of one, two and three sizes launched one by one: the results are
    the single calls', and the time does not depend on which frame comes first
    (1.25 times when the first frame's plan was all frames')."""
    big, small, mid = search_inputs(torch, 4096, 2304, 1), search_inputs(torch, 200, 150, 2), search_inputs(torch, 640, 480, 3)
    params = {id(big): (21, 127), id(small): (15, 15), id(mid): (61, 31)}
    t = []
    for frames in ([big, small], [small, big], [small, mid, big, mid]):
        args = [(dev(torch, L), dev(torch, R), dev(torch, i.view(np.int32)), *params[id(f)]) for f in frames for L, R, i in [f]]
        runner = sbs.BatchRunner(args)
        runner.run_per_frame()
        torch.cuda.synchronize()
        for k, a in enumerate(args):
            d, c = sbs.sad_disparity(*a)
            assert torch.equal(runner.disp[k], d) and torch.equal(runner.cost[k], c), k
        t.append(call_us(torch, runner.run_per_frame))
    assert t[1] < 1.15 * t[0], t


def test_tuned_plan_is_no_slower_than_the_default(torch, sbs, tmp_path):
    """A small frame, whose default plan has lower items than 32 rows, tuned: the
    tuner has such items among its plans and the default plan itself, so a call
    on the stored plan takes no longer than one before."""
    left, right, idx = search_inputs(torch, 392, 296, 4)
    args = [dev(torch, left[:, :, 0].copy()), dev(torch, right[:, :, 0].copy()), dev(torch, idx.view(np.int32)), 15, 15]
    d, c = (x.clone() for x in sbs.sad_disparity(*args))
    before = call_us(torch, lambda: sbs.sad_disparity(*args), reps=40)
    out = torch.empty_like(d)
    frame = sbs.make_frame(*args, out, None)
    assert sbs.get_plan(frame)["tile_rows"] == 8
    sbs.tune([frame], str(tmp_path / "tuning.json"))
    assert sbs.get_plan(frame)["tile_rows"] < 32
    after = call_us(torch, lambda: sbs.sad_disparity(*args), reps=40)
    d1, c1 = sbs.sad_disparity(*args)
    assert torch.equal(d, d1) and torch.equal(c, c1) and torch.equal(out, d)
    assert after < 1.15 * before, (before, after)


@pytest.mark.parametrize("W,H", [(8192, 5), (8193, 5), (9001, 7), (20011, 3)])
def test_fraction_control_of_wide_rows(torch, sbs, W, H):
    """Fractions that end far from every boundary pixel, on rows that are
    searched in LDS (up to 8,192 pixels) and in memory, flat and with a region."""
    img = np.full((H, W), 40, np.uint8)
    region = img.copy()
    region[:, W // 3: W // 3 + 50] = 210
    for what, im in (("flat", img), ("region", region)):
        for frac in (0.01, 0.3, 0.77, 0.999):
            got = sbs.boundaries(dev(torch, im), K=2, mode=0, min_cc=1, frac=frac, seed=5).cpu().numpy().view(np.uint32)
            exp = oracle.boundaries(im, K=2, mode=0, min_cc=1, frac=frac, seed=5)
            assert np.array_equal(got, exp), f"{W}x{H} {what} {frac}"


@pytest.mark.parametrize("H", [1, 7, 8, 9, 16, 17, 33, 130])
@pytest.mark.parametrize("rows", [8, 16, 128, 256])
def test_lists_in_no_order_in_stacked_tiles(torch, sbs, H, rows):
    """Reversed and shuffled lists in items of 16 disparities, which take two
    tiles one above the other by 8 disparities each: odd and even numbers of
    tile rows, main and tail tiles, an odd number of 8-disparity chunks, sums
    that pack and not, a frame on its own and in a batch."""
    rng = np.random.default_rng(H * rows)
    for W, C, block, dmax in ((37, 3, 5, 15), (260, 1, 9, 23), (50, 3, 45, 18)):
        left = rng.integers(0, 256, (H, W, 3) if C == 3 else (H, W), dtype=np.uint8)
        right = np.roll(left, -3, axis=1)
        idx = np.sort(rng.choice(W * H, max(W * H // 4, 1), replace=False)).astype(np.uint32)
        lists = [idx[::-1].copy(), rng.permutation(idx), np.concatenate([idx, idx[:idx.size // 2]])]
        sbs.set_plan(cols_per_lane=4, chunk=16, tile_rows=rows)
        try:
            args = [(dev(torch, left), dev(torch, right), dev(torch, i.view(np.int32)), block, dmax) for i in lists]
            runner = sbs.BatchRunner(args)
            runner.run()
            for k, i in enumerate(lists):
                ed, ec, _ = oracle.sad(left, right, i, block, dmax)
                for d, c in (sbs.sad_disparity(*args[k]), (runner.disp[k], runner.cost[k])):
                    assert np.array_equal(d.cpu().numpy(), ed) and np.array_equal(c.cpu().numpy().view(np.uint32), ec), (W, C, k)
        finally:
            sbs.set_plan()


def test_main_and_tail_tiles_of_lists_in_no_order(torch, sbs):
    """Enough items for main tiles above the tail ones, odd numbers of both."""
    W = 24
    for H in (9000, 9009, 9020):
        rng = np.random.default_rng(H)
        left = rng.integers(0, 256, (H, W), dtype=np.uint8)
        idx = rng.permutation(W * H)[:W * H // 6].astype(np.uint32)
        sbs.set_plan(chunk=16, tile_rows=8)
        try:
            d, c = sbs.sad_disparity(dev(torch, left), dev(torch, np.roll(left, -2, 1)), dev(torch, idx.view(np.int32)), 5, 31)
        finally:
            sbs.set_plan()
        ed, ec, _ = oracle.sad(left, np.roll(left, -2, 1), idx, 5, 31)
        assert np.array_equal(d.cpu().numpy(), ed) and np.array_equal(c.cpu().numpy().view(np.uint32), ec), H


def test_lists_in_no_order_run_as_in_8_disparity_items(torch, sbs):
    """A reversed list on the default plan against items of 8 disparities and 32
    rows, in which it runs in one pass: 1.4 times the call when an item of 16
    disparities was two passes one after another."""
    left, right, idx = search_inputs(torch, 1000, 800, 6)
    args = (dev(torch, left), dev(torch, right), dev(torch, idx[::-1].copy().view(np.int32)), 31, 47)
    t = [call_us(torch, lambda: sbs.sad_disparity(*args))]
    sbs.set_plan(cols_per_lane=4, chunk=8, tile_rows=32)
    try:
        t.append(call_us(torch, lambda: sbs.sad_disparity(*args)))
    finally:
        sbs.set_plan()
    assert t[0] < 1.2 * t[1], t


def test_batches_of_few_tiles(torch, sbs):
    """Frames of one to nine tiles, some with empty lists, more and fewer of them
    than queues: the results are the oracle's."""
    rng = np.random.default_rng(9)
    host, args = [], []
    for t, (W, H, n) in enumerate([(4, 13, 9), (300, 3, 50), (30, 70, 0), (500, 40, 900), (1, 1, 1), (9, 9, 0), (9, 9, 20),
                                   (260, 20, 300), (2, 90, 40), (700, 9, 100), (20, 5, 30)] * 2):
        left = rng.integers(0, 256, (H, W, 3), dtype=np.uint8)
        idx = np.sort(rng.choice(W * H, min(n, W * H), replace=False)).astype(np.uint32)
        host.append((left, np.roll(left, -1, 1), idx))
        args.append((*(dev(torch, a) for a in host[-1][:2]), dev(torch, idx.view(np.int32)), 5, (255, 31)[t % 2]))
    for some in (slice(0, 22), slice(0, 3), slice(2, 6), slice(5, 14)):
        runner = sbs.BatchRunner(args[some])
        for _ in range(2):
            runner.run()
        for k, (L, R, idx) in enumerate(host[some]):
            if not idx.size:
                continue
            ed, ec, _ = oracle.sad(L, R, idx, 5, args[some][k][4])
            assert np.array_equal(runner.disp[k].cpu().numpy(), ed), (some, k)
            assert np.array_equal(runner.cost[k].cpu().numpy().view(np.uint32), ec), (some, k)


def test_batches_of_few_tiles_fill_all_queues(torch, sbs):
    """20 frames of one or two tiles with 256 disparities against the same with
    8: 2.3 times the call when all their items were in the first two queues, 1.6
    times over all of them."""
    rng = np.random.default_rng(10)
    left = dev(torch, rng.integers(0, 256, (13, 4), dtype=np.uint8))
    idx = dev(torch, np.arange(0, 52, 2).astype(np.int32))
    t = []
    for dmax in (255, 7):
        runner = sbs.BatchRunner([(left, left, idx, 9, dmax)] * 20)
        t.append(call_us(torch, runner.run, reps=40))
    assert t[0] < 2 * t[1], t


@pytest.mark.parametrize("W,H", [(37, 4500), (4200, 2100), (9000, 1500)])
def test_row_bits_of_large_arrays(torch, sbs, W, H):
    """Lists in no order on images whose row bits are set in memory (more than
    4,096 words): ordered but for one descent, reversed, shuffled, sparse,
    entries past the image among them."""
    rng = np.random.default_rng(W)
    left = rng.integers(0, 256, (H, W), dtype=np.uint8)
    right = np.roll(left, -2, 1)
    dl, dr = dev(torch, left), dev(torch, right)
    idx = np.sort(rng.choice(W * H, W * H // 40, replace=False)).astype(np.uint32)
    for what, lst in {"one descent": np.concatenate([idx, idx[:100]]), "reversed": idx[::-1].copy(), "shuffled": rng.permutation(idx),
                      "sparse": rng.permutation(idx)[:300], "past": np.concatenate([idx[::-1], [W * H, 2 ** 32 - 1, 5]]).astype(np.uint32)}.items():
        d, c = sbs.sad_disparity(dl, dr, dev(torch, lst.view(np.int32)), 3, 7)
        ed, ec, _ = oracle.sad(left, right, np.minimum(lst, W * H - 1), 3, 7)
        out = lst >= W * H
        ed[out], ec[out] = 255, 0xFFFFFFFF
        assert np.array_equal(d.cpu().numpy(), ed) and np.array_equal(c.cpu().numpy().view(np.uint32), ec), what


def test_row_bits_of_dense_lists_take_no_atomic_each(torch, sbs):
    """A dense list with one descent on an image whose row bits do not fit the
    LDS, against one of as many pixels whose do: 2.2 times the call when every
    entry set its bit by itself."""
    t = []
    for W, H in ((365, 4750), (444, 3905)):
        rng = np.random.default_rng(H)
        left = rng.integers(0, 256, (H, W), dtype=np.uint8)
        idx = np.sort(rng.choice(W * H, W * H * 5 // 6, replace=False))
        args = (dev(torch, left), dev(torch, left), dev(torch, np.concatenate([idx, idx[:idx.size // 2]]).astype(np.int32)), 5, 31)
        t.append(call_us(torch, lambda: sbs.sad_disparity(*args)))
    assert t[0] < 1.4 * t[1], t


@pytest.mark.parametrize("K", [1, 2, 4, 5, 6, 17, 33, 63, 64])
def test_label_images_of_many_clusters(torch, sbs, K):
    """The label image after open and close at numbers of clusters around groups
    of four planes and the largest, widths of every remainder of four pixels."""
    rng = np.random.default_rng(K)
    for W, H in ((61, 60), (64, 56), (130, 107), (67, 9), (3, 70)):
        img = np.kron(rng.integers(0, 256, (H // 4 + 1, W // 5 + 1)), np.ones((4, 5)))[:H, :W].astype(np.uint8)
        _, _, labels = sbs.boundaries(dev(torch, img), K=K, mode=0, min_cc=5, with_maps=True)
        lab = oracle.label_open_close(oracle.label_pixels(img, oracle.kmeans_bins(oracle.histogram(img), K)[0]))
        assert np.array_equal(labels.cpu().numpy(), lab), (W, H)


def test_label_image_of_many_clusters_is_written_once(torch, sbs):
    """64 clusters with the label image asked for and without: 3 times the
    call when a label was read back and written for every four clusters."""
    rng = np.random.default_rng(8)
    img = dev(torch, np.kron(rng.integers(0, 256, (60, 80)), np.ones((8, 8))).astype(np.uint8))
    t = [call_us(torch, lambda: sbs.boundaries(img, K=64, with_maps=maps)) for maps in (True, False)]
    assert t[0] < 2 * t[1], t


def test_fraction_control_of_a_large_ring(torch, sbs):
    """A list that ends among 2.4 million pixels at one distance: over 1,536 of
    their hashes fall in one bin, more than are ranked in LDS."""
    W, H = 4096, 2304
    img = np.repeat((((np.arange(W) // 8) & 1) * 150).astype(np.uint8)[None, :], H, 0)
    for frac in (0.26, 0.4):
        got = sbs.boundaries(dev(torch, img), K=2, mode=0, min_cc=1, frac=frac, seed=11).cpu().numpy().view(np.uint32)
        exp = oracle.boundaries(img, K=2, mode=0, min_cc=1, frac=frac, seed=11)
        assert np.array_equal(got, exp), frac


@pytest.mark.parametrize("nframes,rows", [(2, 64), (7, 96)])
def test_default_plans_of_tall_tiles(torch, sbs, nframes, rows):
    """Batches that take 64 and 96 rows without a plan set."""
    W, H = 4096, 2304
    rng = np.random.default_rng(rows)
    left = rng.integers(0, 256, (H, W), dtype=np.uint8)
    right = np.roll(left, -9, 1)
    dl, dr = dev(torch, left), dev(torch, right)
    lists = [np.sort(rng.choice(W * H, 4000, replace=False)).astype(np.uint32) for _ in range(nframes)]
    lists[0] = (np.arange(4000) + 1000 * W - 77).astype(np.uint32)
    runner = sbs.BatchRunner([(dl, dr, dev(torch, i.view(np.int32)), 9, 255) for i in lists])
    assert runner.plan()["tile_rows"] == rows and runner.plan()["chunk"] == 16
    runner.run()
    for k, i in enumerate(lists):
        ed, ec, _ = oracle.sad(left, right, i, 9, 255)
        assert np.array_equal(runner.disp[k].cpu().numpy(), ed), k
        assert np.array_equal(runner.cost[k].cpu().numpy().view(np.uint32), ec), k
