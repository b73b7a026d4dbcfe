"""The two-level binning (supertiles of 8 x 8 tiles) at the sizes where it
can go wrong: remainders of the supertile grid, the largest grid it serves and
the first one binned by rows, lists of many chunks, and chunks longer than what
is counted and staged at once.  Pair lists and ranges are bit-exact."""
import numpy as np
import pytest
import torch

from gpu_helpers import ctx, say
from oracle import binning as obn
from paper_2412_13547_amd import api, scenes

pytestmark = pytest.mark.gpu
F64 = torch.float64


def _lists(view, dev):
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    return view.pair_vals().cpu().to(torch.int64), view.ranges().cpu().to(torch.int64)


def _oracle(view, g):
    r32 = view.records().cpu()
    bits, r = r32.view(torch.int32), r32.to(F64)
    return obn.bin_gaussians(r[:, 0], r[:, 1], r[:, 9], bits[:, 10].to(torch.int64),
                             (bits[:, 11] & 8) != 0, g)


# (n, width, height, stride, tile): one tile; one supertile; a tile past it in
# x, in y; ragged ones; many Gaussians on few tiles (lists of many chunks and
# blocks); 1024 supertiles (the most), 1056 (by rows)
@pytest.mark.parametrize("n,w,h,d,tile", [
    (1, 8, 8, 1, 8), (63, 64, 64, 1, 8), (513, 65, 64, 1, 8), (512, 64, 65, 1, 8),
    (1500, 333, 201, 2, 8), (20_000, 40, 24, 1, 8), (9_001, 130, 70, 1, 16),
    (300, 2048, 2048, 1, 8), (300, 2049, 2048, 1, 8),
])
def test_pair_lists_at_the_supertile_edges(n, w, h, d, tile):
    sc, cam = scenes.small_scene(900 + n, n, w, h, sh_degree=0)
    say(f"[gpu] binning n={n} {w}x{h} d={d} T={tile}")
    view = api.View(ctx(), sc.n, cam, d, tile=tile)
    vals, ranges = _lists(view, api.DeviceScene.from_scene(sc))
    o = _oracle(view, obn.grid(w, h, d, 0, 0, tile))
    assert torch.equal(vals, o["vals"])
    assert torch.equal(ranges, o["ranges"])


def test_needle_and_point_splats_against_the_rows():
    """The same Gaussians on a grid binned in two levels and, as its upper-left
    part, on a wider one binned by rows: the shared tiles' lists are equal."""
    sc, cam = scenes.small_scene(77, 4000, 2048, 512, sh_degree=0)
    sc.scales[1:, ::3] *= 1e-3
    sc.scales[:, 1::3] *= 1e-3
    wide = scenes.Camera(8192, 4352, cam.fx, cam.fy, cam.cx, cam.cy, cam.w2c)
    dev = api.DeviceScene.from_scene(sc)
    a, b = api.View(ctx(), sc.n, cam, tile=8), api.View(ctx(), sc.n, wide, tile=8)
    assert int(b.sizes.num_tiles) > 64 * 1024
    # the field-of-view guard depends on the image size, so compare lists of
    # Gaussians whose rectangles agree where both grids have the tile
    va, ra = _lists(a, dev)
    vb, rb = _lists(b, dev)
    same = torch.equal(a.records()[:, :6], b.records()[:, :6])
    gxa, gya, gxb = int(a.sizes.grid_x), int(a.sizes.grid_y), int(b.sizes.grid_x)
    moved = (a.records()[:, :6] != b.records()[:, :6]).any(1).cpu()
    checked = 0
    for ty in range(0, gya, 3):
        for tx in range(0, gxa, 5):
            s, e = ra[ty * gxa + tx].tolist()
            s2, e2 = rb[ty * gxb + tx].tolist()
            la, lb = va[s:e], vb[s2:e2]
            assert torch.equal(la[~moved[la]], lb[~moved[lb]]), (ty, tx)
            checked += int(la.numel())
    assert checked > 1000 and (same or int(moved.sum()) < sc.n // 2)


def test_long_chunks_hold_every_gaussian_in_depth_order():
    """133,001 Gaussians that each cover the whole 1024 x 1 tile grid: every
    tile's list is the depth order.  The 17 M list entries make chunks of more
    than 2048 entries."""
    n = 133_001
    rng = np.random.default_rng(5)
    z = rng.uniform(2.0, 3.0, n).astype(np.float32)
    z[1000:1100] = z[0]                                        # ties: ascending index
    f = lambda a: np.ascontiguousarray(a, np.float32)
    sc = scenes.Scene(f(np.stack([np.zeros(n), np.zeros(n), z])), f(np.full((3, n), 100.0)),
                      f(np.stack([np.ones(n), np.zeros(n), np.zeros(n), np.zeros(n)])),
                      f(np.full(n, 0.01)), f(np.zeros((1, 3, n))), 0)
    cam = scenes.identity_camera(8192, 8, 8192.0)
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), n, cam, tile=8, pair_capacity=1024 * n)
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    assert view.pair_count() == 1024 * n
    want = torch.sort(torch.as_tensor(z).cuda(), stable=True).indices.to(torch.int32)
    got = view.pair_vals().view(1024, n)
    assert bool((got == want[None]).all())
    starts = torch.arange(1024, dtype=torch.int32, device="cuda") * n
    assert torch.equal(view.ranges(), torch.stack([starts, starts + n], 1))


# one block's sort up to 4096 and 8192 keys, tiles of 4096 keys, and of 8192
# above 512 x 4096; around a wavefront's and a round's keys
@pytest.mark.parametrize("n", [1, 2, 64, 65, 256, 257, 1023, 1025, 4096, 4097, 8191, 8192, 8193,
                               12_289, 512 * 4096, 512 * 4096 + 1])
@pytest.mark.parametrize("ties", [False, True])
def test_depth_order_is_the_stable_order(n, ties):
    """The ids of the Gaussians with tiles by depth bits, equal depths by id."""
    sc, cam = scenes.small_scene(7, n, 96, 80, sh_degree=0)
    if ties:
        sc.means[2] = np.round(sc.means[2], 1)
    say(f"[gpu] depth order n={n} ties={ties}")
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), n, cam, 1, 0, 0, 16, (0.0, 0.0, 0.0))
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    z = view.records()[:, 9].contiguous().view(torch.int32).cpu().numpy().view(np.uint32)
    ids = np.flatnonzero(view.tiles_touched().cpu().numpy())
    want = ids[np.argsort(z[ids], kind="stable")]
    assert np.array_equal(view.depth_order().cpu().numpy(), want)


# views of few Gaussians and tiles are binned directly (up to 32 M tests of one
# against the other): parts of the depth order and their remainders, tiles
# past a block's 16, the last direct size of 64 tiles and the first of the two
# levels, and two-level grids with a remainder of tiles in both directions
@pytest.mark.parametrize("n,w,h,tile", [
    (1, 8, 8, 8), (1023, 136, 8, 8), (1025, 128, 64, 8), (2049, 129, 127, 8), (5000, 250, 250, 16),
    (9000, 640, 360, 8), (500_000, 64, 64, 8), (500_001, 64, 64, 8), (40_000, 333, 201, 8),
])
def test_pair_lists_around_the_direct_binning(n, w, h, tile):
    sc, cam = scenes.small_scene(77 + n, n, w, h, sh_degree=0)
    if n > 100_000:
        sc.scales[:] = sc.scales * np.float32(0.2)
    say(f"[gpu] direct binning n={n} {w}x{h} T={tile}")
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), n, cam, 1, 0, 0, tile, (0.0, 0.0, 0.0))
    vals, ranges = _lists(view, dev)
    o = _oracle(view, obn.grid(w, h, 1, 0, 0, tile))
    assert torch.equal(vals, o["vals"])
    assert torch.equal(ranges, o["ranges"])


@pytest.mark.parametrize("n", [300, 4097, 9000])
def test_binning_again_gives_the_same_lists(n):
    """A second bin/sort of one preprocess (culled Gaussians included) finds its
    keys as the first did."""
    sc, cam = scenes.small_scene(9, n, 96, 80, sh_degree=0)
    sc.means[2, ::3] = -4.0
    say(f"[gpu] binning again n={n}")
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), n, cam, 1, 0, 0, 16, (0.0, 0.0, 0.0))
    vals, ranges = _lists(view, dev)
    order = view.depth_order().cpu()
    assert 0 < len(order) < n
    for _ in range(2):
        view.bin_sort(dev)
        assert torch.equal(view.depth_order().cpu(), order)
        assert torch.equal(view.pair_vals().cpu().to(torch.int64), vals)
        assert torch.equal(view.ranges().cpu().to(torch.int64), ranges)
