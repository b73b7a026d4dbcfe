"""Views for the tests of the binnings, with the binning each takes: directly, in
two levels (supertiles) or by rows.  The sizes are where each can go wrong; that
they are what the library's rules send there is checked without a GPU."""
import numpy as np

from paper_2412_13547_amd import scenes

# n, capacity, width, height, stride, off_x, off_y, tile, scale of the splats,
# share of the Gaussians behind the camera
TWO_LEVELS = {
    "a tile past a supertile in x": (450_001, 4_000_000, 65, 64, 1, 0, 0, 8, 0.02, 0.0),
    "a tile past a supertile in y": (450_001, 4_000_000, 64, 65, 1, 0, 0, 8, 0.02, 0.5),
    "many chunks of part of a supertile": (1_100_003, 12_000_000, 48, 40, 1, 0, 0, 8, 0.02, 0.0),
    "ragged, strided, whole blocks": (66_560, 8_000_000, 641, 479, 2, 1, 0, 8, 0.2, 0.0),
    "ragged, strided, a Gaussian more": (66_561, 8_000_000, 643, 478, 2, 0, 1, 8, 0.2, 0.3),
    "stride 3 at tile 16": (100_003, 8_000_000, 1237, 822, 3, 2, 1, 16, 0.3, 0.1),
    "tile 32": (40_000, 4_000_000, 1037, 901, 1, 0, 0, 32, 0.3, 0.0),
    "one block on many tiles": (64, 1_000_000, 1040, 1016, 1, 0, 0, 8, 1.0, 0.0),
    "1024 supertiles, 8 wide": (5_000, 8_000_000, 512, 8192, 1, 0, 0, 8, 0.3, 0.0),
    "1024 supertiles, 128 wide": (5_000, 24_000_000, 8192, 512, 1, 0, 0, 8, 0.3, 0.0),
    "large splats on 1023 supertiles": (2_000, 40_000_000, 2111, 1983, 1, 0, 0, 8, 2.0, 0.0),
}
ROWS = {
    "1056 supertiles, many blocks and slices": (60_000, 40_000_000, 2049, 2048, 1, 0, 0, 8, 0.3, 0.2),
    "a capacity without room for the tables": (1_000_000, 1_200_000, 2048, 2048, 1, 0, 0, 8, 0.002, 0.7),
}
# views of one batch, all in two levels: n, capacity of each, tile, then the views
BATCH_N, BATCH_CAPACITY, BATCH_TILE = 40_000, 3_000_000, 8
BATCH_VIEWS = [(333, 201, 1, 0, 0), (640, 360, 2, 1, 0), (1024, 512, 3, 2, 1), (520, 300, 1, 0, 0),
               (400, 400, 1, 0, 0)]
# more pairs than the capacity
OVERFLOW = {
    "direct": (3_000, 20_000, 320, 200, 1, 0, 0, 16, 1.0, 0.0),
    "two levels": (40_000, 500_000, 640, 360, 1, 0, 0, 8, 1.0, 0.0),
    "rows": (20_000, 3_000_000, 2049, 2048, 1, 0, 0, 8, 1.0, 0.0),
}


def layout_request(case):
    return case[:8]


def scene(case, seed=5):
    n, _cap, w, h = case[:4]
    sc, cam = scenes.small_scene(seed, n, w, h, sh_degree=0)
    sc.scales[:] = sc.scales * np.float32(case[8])
    behind = np.random.default_rng(seed).permutation(n)[:int(case[9] * n)]
    centre = -cam.w2c[:, :3].T @ cam.w2c[:, 3]
    sc.means[:, behind] = (2.0 * centre[:, None] - sc.means[:, behind]).astype(np.float32)
    return sc, cam
