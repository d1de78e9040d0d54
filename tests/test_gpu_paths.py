"""GPU parity at the edges of dispatch rules and of kernels' tiles: the HIP path
against the oracle, bit for bit (whole numbers) at the sizes where a path
begins, ends or leaves a remainder."""
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


def pair(rng, W, H, C, levels=256):
    shape = (H, W) if C == 1 else (H, W, C)
    L = (rng.integers(0, levels, shape) * (256 // levels)).astype(np.uint8)
    R = np.roll(L, -5, axis=1)
    R[::3] = rng.integers(0, 256, R[::3].shape, dtype=np.uint8)
    return L, R


def check_search(torch, sbs, L, R, idx, block, dmax, what):
    d, c = sbs.sad_disparity(dev(torch, L), dev(torch, R), dev(torch, idx.astype(np.uint32).view(np.int32)), block, dmax)
    torch.cuda.synchronize()
    ed, ec, _ = oracle.sad(L, R, idx.astype(np.uint32), block, dmax)
    gd, gc = d.cpu().numpy(), c.cpu().numpy().view(np.uint32)
    bad = np.flatnonzero((gd != ed) | (gc != ec))
    assert bad.size == 0, f"{what}: {bad.size} of {idx.size} differ, first at entry {bad[:3]}"


@pytest.mark.parametrize("run", [1, 3, 255, 256, 257, 1024, 5000])
def test_lists_ordered_in_runs(torch, sbs, run):
    """Lists made of ascending runs in a shuffled order, with some entries
    repeated far apart: wavefronts of the order check that see a descent lie
    beside ones that see none, down to a single descent in the whole list."""
    rng = np.random.default_rng(100 + run)
    W, H = 331, 97
    L, R = pair(rng, W, H, 3)
    idx = np.sort(rng.choice(W * H, 7013, replace=False))
    cuts = [idx[i:i + run] for i in range(0, idx.size, run)]
    order = np.roll(np.arange(len(cuts)), 1) if len(cuts) < 3 else rng.permutation(len(cuts))
    lst = np.concatenate([cuts[i] for i in order] + [idx[:40]])
    check_search(torch, sbs, L, R, lst, 9, 33, f"runs of {run}")


@pytest.mark.parametrize("H", [1, 4096, 4097])
def test_unordered_lists_tall_images(torch, sbs, H):
    """The row bits of an unordered list gathered in LDS (up to 4096 words:
    one per row here) and, one row more, set in memory."""
    rng = np.random.default_rng(H)
    W = 40
    L, R = pair(rng, W, H, 1)
    lst = rng.choice(W * H, max(W * H // 9, 20))
    check_search(torch, sbs, L, R, lst, 5, 11, f"{W}x{H}")


@pytest.mark.parametrize("C,block", [(1, 15), (1, 17), (3, 9), (3, 11), (1, 1), (3, 1)])
@pytest.mark.parametrize("chunk", [8, 16])
def test_narrow_windows(torch, sbs, C, block, chunk):
    """Windows whose sums just fit 16 bits (15x15 grey, 9x9 RGB) and the next
    larger blocks, with sums up to the largest (black against white), largest
    disparities around the chunks' ends, and widths around a tile's."""
    rng = np.random.default_rng(7 * block + C)
    sbs.set_plan(cols_per_lane=4, chunk=chunk, tile_rows=16)
    try:
        for W, H, dmax, white in [(241, 37, 15, True), (240, 20, 16, False), (530, 33, 33, True), (60, 9, 0, True)]:
            L, R = pair(rng, W, H, C)
            if white:
                L[: H // 2] = 0
                R[: H // 2] = 255
                L[:, : W // 3] = 255
                R[:, : W // 3] = 0
            idx = np.sort(rng.choice(W * H, W * H // 3, replace=False))
            check_search(torch, sbs, L, R, idx, block, dmax, f"{W}x{H}x{C} block {block} dmax {dmax}")
    finally:
        sbs.set_plan()


@pytest.mark.parametrize("nframes,W,H,wpc", [(1, 40, 20, 16), (3, 90, 33, 16), (9, 250, 130, 16), (2, 700, 300, 1)])
def test_queue_starts(torch, sbs, nframes, W, H, wpc):
    """Batched launches with fewer work items than queues, about as many as
    workgroups, and several items for each workgroup."""
    rng = np.random.default_rng(nframes)
    sbs.set_plan(waves_per_cu=wpc, tile_rows=8 if wpc == 1 else 0)
    try:
        host, frames = [], []
        for t in range(nframes):
            L, R = pair(rng, W, H, 3)
            idx = np.sort(rng.choice(W * H, W * H // 5, replace=False)).astype(np.uint32)
            host.append((L, R, idx))
            frames.append((dev(torch, L), dev(torch, R), dev(torch, idx.view(np.int32)), 7, 40))
        runner = sbs.BatchRunner(frames)
        for rep in range(2):
            runner.run()
        torch.cuda.synchronize()
        for t, (L, R, idx) in enumerate(host):
            ed, ec, _ = oracle.sad(L, R, idx, 7, 40)
            assert np.array_equal(runner.disp[t].cpu().numpy(), ed), t
            assert np.array_equal(runner.cost[t].cpu().numpy().view(np.uint32), ec), t
    finally:
        sbs.set_plan()


@pytest.mark.parametrize("H", [1, 3, 4, 5, 7, 8, 9, 130])
def test_tail_tiles(torch, sbs, H):
    """Images that are all tail tiles (half of the plan's rows each), of fewer
    rows than a tile, one row more, and several tiles."""
    rng = np.random.default_rng(H)
    W = 30
    L, R = pair(rng, W, H, 1)
    idx = np.unique(np.concatenate([rng.choice(W * H, W * H // 4, replace=False), np.arange(min(W, W * H)),
                                    np.arange(max(0, W * H - 2 * W), W * H)]))
    for tile_rows, chunk in ((8, 8), (9, 16), (0, 0)):
        sbs.set_plan(chunk=chunk, tile_rows=tile_rows)
        try:
            check_search(torch, sbs, L, R, idx, 3, 15, f"H {H} tile rows {tile_rows}")
        finally:
            sbs.set_plan()


@pytest.mark.parametrize("H", [9000, 9009])
def test_main_and_tail_tiles(torch, sbs, H):
    """Enough items for main tiles above the tail ones (8 rows, two chunks of
    one tile column: 1,125 and 1,127 tile rows, the last 1,024 of them tail)."""
    rng = np.random.default_rng(H)
    W = 24
    L, R = pair(rng, W, H, 1)
    idx = np.sort(rng.choice(W * H, W * H // 6, replace=False))
    sbs.set_plan(chunk=8, tile_rows=8)
    try:
        check_search(torch, sbs, L, R, idx, 5, 15, f"H {H}")
    finally:
        sbs.set_plan()


def check_front(torch, sbs, dimg, img, K, mode, min_cc, what):
    lst, refined, labels = sbs.boundaries(dimg, K=K, mode=mode, min_cc=min_cc, with_maps=True)
    exp_list, exp_map = oracle.boundaries(img, K=K, mode=mode, min_cc=min_cc, frac=-1.0, return_map=True)
    L8 = oracle.lightness(img)
    lab = oracle.label_pixels(L8, oracle.kmeans_bins(oracle.histogram(L8), K)[0])
    if mode == 0:
        lab = oracle.label_open_close(lab)
    assert np.array_equal(labels.cpu().numpy(), lab), f"{what}: labels"
    assert np.array_equal(refined.cpu().numpy(), exp_map), f"{what}: kept map"
    assert np.array_equal(lst.cpu().numpy().view(np.uint32), exp_list), f"{what}: list"
    assert np.array_equal(sbs.boundaries(dimg, K=K, mode=mode, min_cc=min_cc).cpu().numpy().view(np.uint32), exp_list), what


def blotches(rng, W, H, levels=9):
    """A grey image of flat patches a few pixels wide, with specks."""
    img = np.kron(rng.integers(0, levels, (H // 5 + 1, W // 7 + 1)), np.ones((5, 7)))[:H, :W] * (255 // levels)
    img[rng.random((H, W)) < 0.02] = 255
    return img.astype(np.uint8)


@pytest.mark.parametrize("W,H", [(63, 54), (64, 55), (65, 58), (68, 59), (127, 64), (130, 109), (200, 117), (20, 3), (35, 240)])
def test_refinement_tiles(torch, sbs, W, H):
    """Images around the refinement's tiles (64 columns; 54 rows configured,
    58 in paper mode), rows of whole words and not, images at odd addresses,
    and numbers of clusters at the edges of a group of planes."""
    rng = np.random.default_rng(W * H)
    img = blotches(rng, W, H)
    for off in (0, 1):
        buf = torch.zeros(W * H + 8, dtype=torch.uint8, device="cuda")
        view = buf[off:off + W * H].view(H, W)
        view.copy_(dev(torch, img))
        for mode, Ks in ((0, (2, 5, 6, 9)), (1, (2, 4, 16, 17))):
            for K in Ks:
                check_front(torch, sbs, view, img, K, mode, 5, f"{W}x{H} offset {off} mode {mode} K {K}")


def check_fraction(torch, sbs, img, K, mode, min_cc, frac, seed, what):
    got = sbs.boundaries(dev(torch, img), K=K, mode=mode, min_cc=min_cc, frac=frac, seed=seed).cpu().numpy().view(np.uint32)
    exp = oracle.boundaries(img, K=K, mode=mode, min_cc=min_cc, frac=frac, seed=seed)
    assert np.array_equal(got, exp), f"{what}: {got.size} and {exp.size} pixels, {np.setdiff1d(got, exp).size} differ"


@pytest.mark.parametrize("W,H", [(300, 260), (128, 98), (129, 99), (700, 40)])
def test_fraction_control_levels(torch, sbs, W, H):
    """Fractions that end at every distance a small scene has: the levels of
    both dilation launches (1 .. 15 and 16 .. 30), their last and first ones,
    and the distance passes beyond, on maps around the dilation's tiles (128
    columns, 98 rows)."""
    img = np.full((H, W), 40, np.uint8)
    img[H // 3:H // 3 + 14, W // 2:W // 2 + 20] = 210
    _, kept = oracle.boundaries(img, K=2, mode=0, min_cc=1, frac=-1.0, return_map=True)
    base = kept.astype(bool)
    base[:, 0] = base[:, -1] = True
    from scipy.ndimage import distance_transform_cdt
    dist = distance_transform_cdt(~base, metric="chessboard")
    for d in sorted({1, 2, 14, 15, 16, 17, 29, 30, 31, 32, 40, int(dist.max())}):
        inside, ring = int((dist < d).sum()), int((dist == d).sum())
        for k in {1, ring // 2, ring}:
            if ring and k:
                check_fraction(torch, sbs, img, 2, 0, 1, (inside + k) / (W * H), 77 + d, f"{W}x{H} distance {d} rank {k}")


def test_fraction_control_levels_many_blocks(torch, sbs):
    """A list that ends within the first level of the second dilation launch,
    on an image whose blocks do not all run at once: those that start late
    have the counts of the others before them."""
    W, H = 64, 200000
    img = np.full((H, W), 40, np.uint8)
    check_fraction(torch, sbs, img, 1, 0, 1, (32 * H + H // 9) / (W * H), 7, f"{W}x{H}")


@pytest.mark.parametrize("W,H", [(64, 33), (131, 70), (4200, 4096)])
def test_fraction_control_component_sizes(torch, sbs, W, H):
    """Fractions that end among the kept pixels: within a component size that
    many components share (ties by raster order), at the largest and at the
    smallest, and on an image of 2^24 pixels and more (a third digit)."""
    rng = np.random.default_rng(W)
    img = np.zeros((H, W), np.uint8)
    for k in range(W * H // 500 if W < 1000 else 400):
        y, x, r = int(rng.integers(0, H)), int(rng.integers(0, W)), int(rng.integers(3, 8))
        img[y:y + r, x:x + r] = 200
    _, kept = oracle.boundaries(img, K=2, mode=0, min_cc=1, frac=-1.0, return_map=True)
    n1, n0 = int(kept[:, 1:-1].sum()), 2 * H
    for share in ((0.5,) if W > 1000 else (0.0, 0.1, 0.33, 0.5, 0.77, 1.0)):
        check_fraction(torch, sbs, img, 2, 0, 1, (n0 + 1 + share * (n1 - 1)) / (W * H), 3, f"{W}x{H} share {share}")


@pytest.mark.parametrize("C", [1, 3])
def test_lightness_rows(torch, sbs, C):
    """Rows of every remainder of the groups that a thread takes (4 RGB pixels,
    16 grey ones), with and without gaps, at odd addresses; the histogram taken
    on the way gives the same labels."""
    rng = np.random.default_rng(C)
    for W in (1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 65):
        for H, pad, off in ((1, 0, 0), (7, 0, 1), (7, 1, 0), (9, 4, 2), (40, 13, 3)):
            pitch = W * C + pad
            buf = rng.integers(0, 256, off + H * pitch, dtype=np.uint8)
            img = np.ascontiguousarray(buf[off:].reshape(H, pitch)[:, :W * C].reshape((H, W, C) if C == 3 else (H, W)))
            d = dev(torch, buf)
            view = torch.as_strided(d, (H, W, C) if C == 3 else (H, W), (pitch, C, 1) if C == 3 else (pitch, 1), off)
            what = f"{W}x{H}x{C} pitch {pitch} offset {off}"
            assert np.array_equal(sbs.lightness(view).cpu().numpy(), oracle.lightness(img)), what
            check_front(torch, sbs, view, img, 4, 0, 2, what)


@pytest.mark.parametrize("K", [1, 2, 9, 10, 33, 64])
def test_kmeans_level_ranges(torch, sbs, K):
    """Ranges of grey levels just below, at and above the number of clusters
    (equal first centres below it), few and many occupied levels, clusters that
    stay empty, and midpoints that fall on a level."""
    rng = np.random.default_rng(K)
    for span in sorted({1, max(K - 1, 1), K, K + 1, 2 * K, 200, 256}):
        for levels in {1, 2, 5, span}:
            lo = int(rng.integers(0, 256 - span + 1))
            used = np.unique(np.concatenate([[0, span - 1], rng.integers(0, span, min(levels, span))])) + lo
            img = used[rng.integers(0, used.size, (40, 70))].astype(np.uint8)
            img[0, :2] = lo, lo + span - 1
            check_front(torch, sbs, dev(torch, img), img, K, 0, 5, f"K {K}, {used.size} levels of {span} from {lo}")


@pytest.mark.parametrize("W,H,n", [(1, 9, 5), (64, 5, 40), (65, 7, 1024), (4095, 6, 5000), (4096, 300, 1100000)])
def test_reconstruct_lists_in_order_and_not(torch, sbs, W, H, n):
    """Lists in raster order, with repeats and entries past the image, and the
    same ones with a single descent: at the start, at the end, at the edges of
    the 1024 entries a block checks at a time and where blocks meet."""
    rng = np.random.default_rng(n)
    idx = np.sort(rng.integers(0, W * H + 3, n)).astype(np.uint32)
    disp = rng.integers(0, 3, n).astype(np.uint8)
    at = [None] + [k for k in (1, 1023, 1024, 2048, n - 1) if 0 < k < n]
    for k in at:
        p = idx.copy()
        if k is not None:
            p[k - 1], p[k] = max(int(p[k - 1]), 1), 0
        exp = oracle.reconstruct(p, disp, W, H, 1)
        got = sbs.reconstruct(dev(torch, p.view(np.int32)), dev(torch, disp), W, H, 1).cpu().numpy()
        assert np.array_equal(got, exp), f"{W}x{H}, {n} entries, descent at {k}: {(got != exp).sum()} pixels differ"


@pytest.mark.parametrize("C", [1, 3])
def test_blur_edge_tiles(torch, sbs, C):
    """Images narrower than a group of four pixels, than a tile, and around the
    widths where a tile becomes an interior one, at odd addresses and pitches:
    every column of the edge tiles' clamped groups."""
    rng = np.random.default_rng(C)
    for W in (1, 2, 3, 4, 5, 9, 63, 66, 72, 73, 76, 77, 135, 140):
        for H, pad, off in ((1, 0, 0), (35, 1, 1), (40, 4, 3)):
            pitch = W * C + pad
            buf = rng.integers(0, 256, off + H * pitch, dtype=np.uint8)
            rows = buf[off:].reshape(H, pitch)[:, :W * C].reshape((H, W, C) if C == 3 else (H, W))
            depth = rng.integers(0, 4, (H, W)).astype(np.uint8)
            d = dev(torch, buf)
            view = torch.as_strided(d, (H, W, C) if C == 3 else (H, W), (pitch, C, 1) if C == 3 else (pitch, 1), off)
            got = sbs.selective_blur(view, dev(torch, depth), [(1, 1)], 2.0).cpu().numpy()
            exp = oracle.blur(np.ascontiguousarray(rows), depth, [(1, 1)], 2.0)
            assert np.abs(got - exp).max() <= 1e-3, f"{W}x{H}x{C} pitch {pitch} offset {off}"


@pytest.mark.parametrize("W,H", [(24, 40000), (1024, 2048), (1031, 2035)])
def test_single_frame_preparation(torch, sbs, W, H):
    """Single frames at and past the size up to which the pixel map is cleared
    with the copies (2^21 pixels), and one whose list check has fewer words for
    its blocks than entries to fill them: ordered lists, one descent, lists in
    no order, and entries past the image, the first of them anywhere."""
    rng = np.random.default_rng(W)
    L, R = pair(rng, W, H, 1)
    N = W * H
    base = np.sort(rng.choice(N, min(N // 2, 400000), replace=False))
    n = base.size
    lists = {"ordered": base, "in no order": rng.permutation(base)[:30000]}
    for k in (1, n // 2, n - 1):
        one = base.copy()
        one[k - 1], one[k] = one[k], one[k - 1]
        lists[f"descent at {k}"] = one
    past = base.copy()
    past[-3:] = N + 5, N + 6, N + 9
    lists["ordered, ends past the image"] = past
    mixed = rng.permutation(base)[:30000]
    mixed[[7, 12345]] = N
    lists["in no order, past the image"] = mixed
    sbs.check_indices()   # (reads and clears the error word)
    for what, idx in lists.items():
        check_search(torch, sbs, L, R, idx, 3, 9, f"{W}x{H} {what}")
        assert sbs.check_indices() == (5 if idx.max() >= N else 0), what
