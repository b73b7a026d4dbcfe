"""What a bin/sort leaves in a state is what the raster stages ask of it."""
import pytest
import torch

from gpu_helpers import ctx, say
from paper_2412_13547_amd import api, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sync", [False, True])
def test_a_view_moved_to_another_tile_grid_is_refused(sync):
    """640 x 65 at stride 2: 20 x 2 tiles of the odd rows, 20 x 3 of the even
    ones.  Each call is refused on the host, and the view's own grid still works."""
    sc, cam = scenes.small_scene(3, 2000, 640, 65, sh_degree=0)
    say(f"[gpu] moved view sync={sync}")
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), sc.n, cam, 2, 0, 1, 16, sync_check=sync)
    image = view.forward(dev)
    dL = torch.ones_like(image)
    view.raster_bwd(dL)
    want = view.grad2d().clone()
    view.set_offsets(0, 0)
    wider = torch.zeros(view.image_shape, device="cuda")
    assert wider.shape != image.shape
    for call in (lambda: view.raster_fwd(wider), lambda: view.raster_bwd(wider)):
        with pytest.raises(api.TgsError) as e:
            call()
        assert e.value.status == api.TGS_ERR_INVALID_ARG
    view.set_offsets(0, 1)
    again = torch.empty_like(image)
    view.raster_fwd(again)
    view.raster_bwd(dL)
    torch.cuda.synchronize()
    assert torch.equal(again, image)
    assert torch.allclose(view.grad2d(), want, rtol=1e-4, atol=1e-6)
    # another phase with the same tile grid takes the same lists
    view.set_offsets(1, 1)
    view.raster_fwd(again)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(again).all())


# binned directly, in two levels and by rows
@pytest.mark.parametrize("n,w,h,tile", [(3000, 320, 200, 16), (9000, 1016, 640, 8), (3000, 2049, 2048, 8)])
def test_a_synchronous_overflow_leaves_the_needed_count_on_the_device(n, w, h, tile):
    """The word at off_pair_count is the count that did not fit, not that of the
    binning before (tgs_bin_sort reads the count back, reports it and stops)."""
    sc, cam = scenes.small_scene(5, n, w, h, sh_degree=0)
    say(f"[gpu] synchronous overflow n={n} {w}x{h} T={tile}")
    dev = api.DeviceScene.from_scene(sc)
    view = api.View(ctx(), n, cam, tile=tile, pair_capacity=400 * n)
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    few = view.pair_count()
    wide = api.DeviceScene.from_scene(sc)
    wide.scales *= 3.0
    view.preprocess_fwd(wide)
    view.bin_sort(wide)
    need = view.pair_count()
    assert need > few + 1000
    view.reserve(few + 64)
    view.preprocess_fwd(dev)
    view.bin_sort(dev)
    word = view._view(view.state.off_pair_count, 1, torch.int32)
    assert int(word.item()) == few
    view.preprocess_fwd(wide)
    with pytest.raises(api.TgsError) as e:
        view.bin_sort(wide, grow=False)
    assert e.value.status == api.TGS_ERR_CAPACITY
    assert int(view.state.pair_count) == need
    assert int(view._view(view.state.off_pair_count, 1, torch.int32).item()) == need
