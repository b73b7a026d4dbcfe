"""The raster stages refuse a state that was binned for another tile grid or
capacity before any device work, and take one of the same.  The states are
filled as a bin/sort leaves them; a NULL context ends the calls that pass the
check."""
import ctypes as C

import pytest

from layout_probe import layouts
from paper_2412_13547_amd import api

N = 200_000


def _cam(w, h):
    c = api.tgs_camera()
    c.width, c.height = w, h
    c.fx = c.fy = 300.0
    c.cx, c.cy = w / 2, h / 2
    for k in (0, 5, 10):
        c.world_to_cam[k] = 1.0
    c.near_z = 0.2
    return c


def _key_bits(tiles):
    b = 1
    while (1 << b) < tiles:
        b += 1
    return b


def _grid(w, h, d, ox, oy, tile):
    return -(-(-(-(w - ox) // d)) // tile), -(-(-(-(h - oy) // d)) // tile)


def _state(view, cap, pending, tag):
    L = layouts([(N, cap) + view])[0]
    st = api.tgs_state()
    st.workspace, st.workspace_bytes, st.pair_capacity = 1 << 20, L["total"] + (1 << 20), cap
    st.pair_count = api.PAIR_COUNT_PENDING if pending else min(cap, 100)
    gx, gy = _grid(*view)
    st.key_bits = _key_bits(gx * gy)
    st.reserved = (gx | gy << 16) if tag else 0
    for k, v in L.items():
        if k.startswith("off_"):
            setattr(st, k, v)
    return st


def _calls(st, view):
    w, h, d, ox, oy, tile = view
    lib, cam, dil = api.lib(), _cam(w, h), api.dilation_struct(d, ox, oy)
    opt = api.options_struct(tile)
    io = (api.tgs_view_io * 1)()
    io[0].image = io[0].dL_dimage = 1 << 20
    one = (C.byref(cam), C.byref(dil), C.byref(opt), C.byref(st), N)
    many = (N, 1, C.byref(cam), C.byref(dil), C.byref(opt), C.byref(st), io, None)
    yield lib.tgs_raster_fwd(None, *one, 1 << 20, None, None, None, None, None)
    yield lib.tgs_raster_bwd(None, *one, 1 << 20, None)
    yield lib.tgs_batch_raster_fwd(None, *many)
    yield lib.tgs_batch_raster_bwd(None, *many)


def _refused(st, view):
    msgs = []
    for r in _calls(st, view):
        assert r == api.TGS_ERR_INVALID_ARG
        msg = api.lib().tgs_last_error()
        assert b"binned" in msg or b"do not match its layout" in msg or b"context is NULL" in msg, msg
        msgs.append(b"context" not in msg)
    assert len(set(msgs)) == 1, msgs
    return msgs[0]


A = (640, 65, 2, 0, 1, 16)                   # 20 x 2 tiles


@pytest.mark.parametrize("pending", [False, True])
@pytest.mark.parametrize("tag", [False, True])
@pytest.mark.parametrize("binned,cap,used,used_cap", [
    (A, 1_000_000, (640, 65, 2, 0, 0, 16), 1_000_000),                        # a row more
    ((640, 65, 2, 0, 0, 16), 1_000_000, A, 1_000_000),                        # a row less
    (A, 1_000_000, A, 500_000),                                               # less capacity
    (A, 1_000_000, A, 1_000_064),                                             # a little more
    ((1920, 1080, 1, 0, 0, 16), 30_000_000, (1936, 1080, 1, 0, 0, 16), 30_000_000),   # a column more
    ((1025, 800, 1, 0, 0, 16), 8_000_000, (800, 1025, 1, 0, 0, 16), 8_000_000),       # turned
])
def test_another_grid_or_capacity_is_refused(binned, cap, used, used_cap, pending, tag):
    st = _state(binned, cap, pending, tag)
    assert not _refused(st, binned)
    st.pair_capacity = used_cap
    assert _refused(st, used)


@pytest.mark.parametrize("binned,used", [
    ((641, 64, 2, 0, 0, 16), (641, 64, 2, 1, 0, 16)),                         # 21 and 20 columns
    ((65, 33, 1, 0, 0, 8), (64, 33, 1, 0, 0, 8)),
])
def test_a_column_that_the_alignment_hides_is_refused(binned, used):
    st = _state(binned, 1000, False, True)
    assert not _refused(st, binned)
    assert _refused(st, used)


@pytest.mark.parametrize("cap", [1000, 5_000_000])
def test_another_phase_of_the_same_tile_grid_passes(cap):
    """The lists do not depend on the phase, so an image of another phase may
    be made from them (413 and 412 columns of pixels, 26 of tiles)."""
    st = _state((1237, 822, 3, 0, 0, 16), cap, False, True)
    for ox, oy in ((0, 0), (2, 1), (1, 2)):
        assert not _refused(st, (1237, 822, 3, ox, oy, 16))
