"""The densification workspace holds what the selection uses: the candidate
count, keys and positions twice, and the sort's work area (four passes of 256
digit totals and states per 4096 keys, and eight words).  No GPU."""
import ctypes as C

import pytest

from paper_2412_13547_amd import api


@pytest.mark.parametrize("n", [0, 1, 63, 64, 4096, 4097, 1_000_003, 3_000_000])
def test_workspace_is_what_the_buffers_take(n):
    up = lambda x: (x + 255) // 256 * 256
    got = C.c_uint64()
    assert api.lib().tgs_densify_query(n, C.byref(got)) == api.TGS_OK
    words = 4 * 256 + 8 + 4 * 256 * -(-n // 4096)
    assert got.value == 256 + 4 * up(4 * n) + up(4 * words)
