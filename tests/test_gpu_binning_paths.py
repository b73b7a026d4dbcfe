"""The binning in two levels and by rows at the sizes where each can go wrong,
alone, in a batch, in a replayed graph and past the capacity.  Pair lists and
ranges are bit-exact against the oracle."""
import pytest
import torch

import binning_cases as bc
from gpu_helpers import ctx, say
from oracle import binning as obn
from paper_2412_13547_amd import api, scenes

pytestmark = pytest.mark.gpu
F64 = torch.float64


def _view(case, **kw):
    sc, cam = bc.scene(case)
    _n, cap, _w, _h, d, ox, oy, tile = case[:8]
    view = api.View(ctx(), sc.n, cam, d, ox, oy, tile, (0.3, 0.2, 0.1), pair_capacity=cap, **kw)
    return view, api.DeviceScene.from_scene(sc)


def _check_lists(view, w, h, d, ox, oy, tile):
    r32 = view.records().cpu()
    bits, r = r32.view(torch.int32), r32.to(F64)
    o = obn.bin_gaussians(r[:, 0], r[:, 1], r[:, 9], bits[:, 10].to(torch.int64),
                          (bits[:, 11] & 8) != 0, obn.grid(w, h, d, ox, oy, tile))
    assert torch.equal(view.pair_vals().cpu().to(torch.int64), o["vals"])
    assert torch.equal(view.ranges().cpu().to(torch.int64), o["ranges"])
    return int(o["vals"].numel())


@pytest.mark.parametrize("name", list(bc.TWO_LEVELS) + list(bc.ROWS))
def test_pair_lists(name):
    case = bc.TWO_LEVELS.get(name) or bc.ROWS[name]
    view, dev = _view(case)
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    pairs = _check_lists(view, *case[2:8])
    say(f"[gpu] {name}: {pairs} pairs")
    assert int(view.state.pair_capacity) == case[1]          # (not grown: still the path it names)
    assert pairs > case[0] // 4


@pytest.mark.parametrize("name", list(bc.OVERFLOW))
def test_an_overflow_on_the_device_renders_the_background(name):
    """Asynchronous: no pair is written, every range is empty, the count is
    reported later; the next binning of fewer pairs is whole."""
    case = bc.OVERFLOW[name]
    view, dev = _view(case, sync_check=False)
    small = bc.scene(case)[0]
    small.scales *= 0.02
    small = api.DeviceScene.from_scene(small)
    for _ in range(2):
        say(f"[gpu] overflow {name}")
        view.preprocess_fwd(small)
        view.bin_sort(small)
        assert _check_lists(view, *case[2:8]) <= case[1]
        before = view.pair_vals().clone()
        view.preprocess_fwd(dev)
        view.bin_sort(dev)
        image = torch.full(view.image_shape, float("nan"), device="cuda")
        view.raster_fwd(image)
        view.raster_bwd(torch.ones_like(image))
        assert not bool(view.ranges().any())
        assert not bool(view.grad2d().any())
        want = torch.tensor([0.3, 0.2, 0.1], device="cuda")[:, None, None].expand_as(image)
        assert torch.equal(image, want)
        vals = view._view(view.state.off_pair_vals, before.numel(), torch.int32)
        assert torch.equal(vals, before)
        with pytest.raises(api.TgsError) as e:
            view.pair_count()
        assert e.value.status == api.TGS_ERR_CAPACITY and int(view.state.pair_count) > case[1]


def test_a_batch_in_two_levels_eager_and_replayed():
    """Five views on the caller's and the auxiliary streams; then the same from
    a captured graph, replayed with other Gaussians and eager work between."""
    specs = bc.BATCH_VIEWS
    sc, cams = scenes.small_multiview(11, bc.BATCH_N, [(w, h) for w, h, *_ in specs], sh_degree=0)
    sc.scales[:] = sc.scales * 0.15
    other = sc.means.copy()
    other[:, ::2] = other[:, ::2] * 0.9
    dev = api.DeviceScene.from_scene(sc)
    views = [(cams[k], d, ox, oy) for k, (_w, _h, d, ox, oy) in enumerate(specs)]
    b = api.Batch(ctx(), sc.n, views, tile=bc.BATCH_TILE, pair_capacity=bc.BATCH_CAPACITY)

    def check(images):
        counts = b.pair_counts()
        for k, (w, h, d, ox, oy) in enumerate(specs):
            assert _check_lists(b.views[k], w, h, d, ox, oy, bc.BATCH_TILE) == counts[k] > bc.BATCH_N // 4
            assert int(b.states[k].pair_capacity) == bc.BATCH_CAPACITY
            if images is not None:
                assert torch.equal(b.images[k], images[k]), k
        return [t.clone() for t in b.images]

    means = [torch.as_tensor(x).cuda() for x in (sc.means, other)]
    eager = []
    for m in means:
        dev.means.copy_(m)
        b.forward(dev)
        eager.append(check(None))
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        b.forward(dev)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.forward(dev)
    for r in range(4):
        say(f"[gpu] two-level batch, replay {r}")
        dev.means.copy_(means[r % 2])
        graph.replay()
        torch.cuda.synchronize()
        check(eager[r % 2])
        dev.means.copy_(means[(r + 1) % 2])                  # eager work of the other Gaussians
        b.forward(dev)
        check(eager[(r + 1) % 2])
