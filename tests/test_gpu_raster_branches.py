"""The rasterizers' tests per splat are left out where they cannot matter (an
exponent that is never positive, an alpha below its clamp, an entry before
every pixel's last blend).  Scenes that mix splats on both sides of each of
those rules, for every tile size and work split, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import grad_close, records_to_oracle, run_gpu, say
from oracle import backward as obw
from oracle import raster as ors
from paper_2412_13547_amd import scenes

pytestmark = pytest.mark.gpu
F64 = torch.float64


def _mixed(kind):
    """A third of the splats off the rule: opacities around the clamp and 1,
    needles (nearly singular conics), or both among nearly opaque layers that
    end pixels' walks at very different entries."""
    sc, cam = scenes.small_scene(41, 400, 96, 80, sh_degree=0)
    rng = np.random.default_rng(6)
    pick = np.arange(sc.n) % 3 == 0
    if kind in ("clamp", "layers"):
        edge = np.array([0.9898, 0.98995, 0.99, 0.9901, 0.999, 1.0], np.float32)
        sc.opacities[pick] = edge[rng.integers(0, len(edge), int(pick.sum()))]
    if kind in ("needles", "layers"):
        sc.scales[1:, pick] = sc.scales[:1, pick] * np.float32(1e-5)
    if kind == "layers":
        sc.scales[:, 1::3] *= np.float32(0.3)
    return sc, cam


@pytest.mark.parametrize("tile,ppt", [(8, 1), (16, 1), (16, 2), (16, 4), (32, 2), (32, 4)])
@pytest.mark.parametrize("kind", ["clamp", "needles", "layers"])
def test_both_sides_of_the_splat_rules(kind, tile, ppt):
    sc, cam = _mixed(kind)
    tgt = scenes.target_image(cam.width, cam.height, 541)
    bg = (0.3, 0.1, 0.2)
    say(f"[gpu] {kind} T={tile} P={ppt}")
    g = run_gpu(sc, cam, 1, 0, 0, tile, bg, target=tgt, pixels_per_thread=ppt)
    rec = records_to_oracle(g["records"])
    vals, ranges = g["pair_vals"].to(torch.int64), g["ranges"].to(torch.int64)
    o = ors.raster_forward(rec, vals, ranges, g["grid"], bg=bg)
    keep = ~o["flag"]
    assert float(o["flag"].float().mean()) < 0.05
    for k in ("last_contrib", "n_eval", "n_blend"):
        assert torch.equal(g[k].to(torch.int64)[keep], o[k][keep]), k
    assert float((g["image"].to(F64) - o["image"]).abs()[:, keep].max()) <= 1e-4
    dL = g["dL"].to(F64) * keep.to(F64)[None]
    view = g["_view"]
    view.raster_bwd(dL.to(torch.float32).cuda())
    torch.cuda.synchronize()
    got = view.grad2d().cpu()
    want = obw.raster_backward(rec, vals, ranges, g["grid"], dL, bg=bg)
    for c, nm in enumerate(("u", "v", "A", "B", "C", "opacity", "r", "g", "b")):
        grad_close(got[:, c], want[:, c], name=f"{kind} T={tile} P={ppt} d{nm}")


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 68, 127, 129, 255, 256, 257, 300, 513])
@pytest.mark.parametrize("kind", ["all", "some", "stops"])
def test_listed_walk_at_the_edges_of_pairs_words_and_rounds(kind, n):
    """With one pixel a lane a wavefront lists the entries it visits and takes
    them in pairs, four at a time; with four it scans their bits one by one.
    The arithmetic of a pixel is the same, so the forward's outputs are equal
    bit by bit, for every number of entries around a pair, a word of 64 and a
    round; the backward's sums differ in their order (the gradient bar), also
    where it is given the bits of the other split."""
    sc, cam = scenes.small_scene(43, n, 24, 20, sh_degree=0)
    sc.scales[:] = sc.scales * np.float32(0.3 if kind == "some" else 40.0)
    sc.opacities[:] = np.float32(0.5 if kind == "stops" else 0.015)
    tgt = scenes.target_image(cam.width, cam.height, 77)
    want = run_gpu(sc, cam, 1, 0, 0, 16, (0.1, 0.2, 0.3), target=tgt, pixels_per_thread=4)
    for batch in (64, 128, 256):
        say(f"[gpu] {kind} n={n} B={batch}")
        g = run_gpu(sc, cam, 1, 0, 0, 16, (0.1, 0.2, 0.3), target=tgt, pixels_per_thread=1,
                    lds_batch=batch)
        for k in ("image", "t_final", "last_contrib", "n_eval", "n_blend"):
            assert torch.equal(g[k], want[k]), (batch, k)
        grad_close(g["grad2d"], want["grad2d"], name=f"{kind} n={n} B={batch}")
        view = g["_view"]
        view.opt.pixels_per_thread = view.opt_sync.pixels_per_thread = 4
        view.forward(g["_dev"], g["_image"])
        view.opt.pixels_per_thread = 1
        view.raster_bwd(g["dL"].cuda())
        torch.cuda.synchronize()
        grad_close(view.grad2d().cpu(), want["grad2d"], name=f"{kind} n={n} B={batch} other bits")


# the last launch handed out in row order, the first with an order, one share
# and a tile more, three and a tile less, ragged shares of many buckets
@pytest.mark.parametrize("gx,gy", [(32, 16), (27, 19), (32, 32), (41, 25), (59, 26), (67, 61)])
def test_every_tile_is_taken_once(gx, gy):
    """The order of the tiles only decides when each is rendered: from the
    weights of the forward before, and from its own, every pixel comes out as
    in row order, and the gradients' sums differ in their order alone."""
    w, h = 8 * gx - 3, 8 * gy - 1
    sc, cam = scenes.small_scene(47, 900, w, h, sh_degree=0)
    sc.scales[:, ::3] *= np.float32(6.0)
    tgt = torch.as_tensor(scenes.target_image(w, h, 78)).cuda()
    say(f"[gpu] tile order {gx}x{gy}")
    first = run_gpu(sc, cam, 1, 0, 0, 8, (0.2, 0.1, 0.0), target=tgt.cpu().numpy())
    view, dev = first["_view"], first["_dev"]
    for _ in range(2):
        image = torch.full(view.image_shape, float("nan"), device="cuda")
        view.forward(dev, image)
        dL, _loss = view.l1_grad(image, tgt)
        view.raster_bwd(dL)
        torch.cuda.synchronize()
        assert torch.equal(image.cpu(), first["image"])
        grad_close(view.grad2d().cpu(), first["grad2d"], name=f"{gx}x{gy}")
