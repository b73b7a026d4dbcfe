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
