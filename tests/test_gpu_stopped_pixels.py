"""A Gaussian behind what ends every pixel's walk takes no part in the image,
whatever its colour: one whose spherical harmonics overflow to infinity (times a
weight of 0 that is not 0) is not looked at any more."""
import numpy as np
import pytest
import torch

from gpu_helpers import ctx, say
from paper_2412_13547_amd import api, scenes

pytestmark = pytest.mark.gpu


def _layers(thin, behind):
    """`thin` faint layers, three opaque ones that end every walk, then
    `behind` more, all far larger than the image."""
    n = thin + 3 + behind
    f = lambda a: np.ascontiguousarray(a, np.float32)
    means = np.zeros((3, n))
    means[2] = 2.0 + 0.01 * np.arange(n)
    opac = np.r_[np.full(thin, 0.02), np.full(3, 1.0), np.full(behind, 0.5)]
    quats = np.zeros((4, n))
    quats[0] = 1.0
    sh = np.random.default_rng(thin).uniform(-0.1, 0.1, (16, 3, n))
    return scenes.Scene(f(means), f(np.full((3, n), 60.0)), f(quats), f(opac), f(sh), 3)


@pytest.mark.parametrize("tile,ppt", [(8, 1), (16, 1), (16, 2), (16, 4), (32, 2), (32, 4)])
@pytest.mark.parametrize("thin", [0, 1, 2, 3, 60, 61, 62, 63])
def test_an_infinite_colour_behind_every_walk(thin, tile, ppt):
    sc, cam = _layers(thin, 5), scenes.identity_camera(72, 40, 72.0)
    say(f"[gpu] infinite colour behind {thin + 3} layers T={tile} P={ppt}")

    def image():
        view = api.View(ctx(), sc.n, cam, tile=tile, pixels_per_thread=ppt, bg=(0.1, 0.2, 0.3))
        out = view.forward(api.DeviceScene.from_scene(sc)).cpu()
        return out, view.records().cpu()

    want, _ = image()
    assert bool(torch.isfinite(want).all())
    sc.sh[:, :, thin + 3:] = 3.4e38                            # (each finite, their sum not)
    got, rec = image()
    assert bool(torch.isinf(rec[thin + 3:, 6:9]).any(1).all())
    assert torch.equal(got, want)
