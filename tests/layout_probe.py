"""The workspace layout of a view as the library computes it (a small host
program linked against libtgs.so; no GPU): what a test needs to fill a state as
a bin/sort leaves it, and to know which of the binnings a view takes."""
from __future__ import annotations

import functools
import os
import shutil
import subprocess
import tempfile

import pytest

from paper_2412_13547_amd import api, build

FIELDS = ("off_records", "off_tiles_touched", "off_pair_vals", "off_ranges", "off_grad2d",
          "off_pair_count", "off_tile_work", "off_t_final", "off_last_contrib",
          "off_nonfinite_count", "total", "path")
PROGRAM = r"""
#include <cinttypes>
#include <cstdio>
#include "common.hpp"
int main() {
    long long n;
    unsigned long long cap;
    int w, h, d, ox, oy, t;
    while (std::scanf("%lld %llu %d %d %d %d %d %d", &n, &cap, &w, &h, &d, &ox, &oy, &t) == 8) {
        tgs_camera cam{};
        cam.width = w;
        cam.height = h;
        const tgs::Grid g = tgs::make_grid(cam, tgs_dilation{d, ox, oy}, t);
        const tgs::Layout L = tgs::make_layout(n, cap, g);
        const int path = L.super.supers == 0 ? 0 : L.super.direct == 0 ? 1 : 2;
        const uint64_t v[] = {L.records, L.tiles_touched, L.pair_vals, L.ranges, L.grad2d,
                              L.row_start + 4 * uint64_t(g.gy), L.tile_work, L.pix_tfinal,
                              L.pix_last, L.nonfinite, L.total, uint64_t(path)};
        for (const uint64_t x : v) std::printf("%" PRIu64 " ", x);
        std::printf("\n");
    }
    return 0;
}
"""
PATHS = ("rows", "two levels", "direct")
_TMP = tempfile.TemporaryDirectory(prefix="tgs_layout")      # (removed when the tests end)


@functools.lru_cache(maxsize=1)
def _program() -> str:
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    api.lib()
    src, exe = os.path.join(_TMP.name, "layout.cpp"), os.path.join(_TMP.name, "layout")
    with open(src, "w") as f:
        f.write(PROGRAM)
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    r = subprocess.run([cxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-isystem",
                        os.path.join(rocm, "include"), f"-I{build.CSRC}",
                        f"-I{os.path.join(build.ROOT, 'include')}", src, api.LIB_PATH,
                        f"-Wl,-rpath,{os.path.dirname(api.LIB_PATH)}:{os.path.join(rocm, 'lib')}",
                        f"-L{os.path.join(rocm, 'lib')}", "-lamdhip64", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def layouts(requests) -> list[dict]:
    """requests: (n, capacity, width, height, stride, off_x, off_y, tile) each."""
    text = "".join(" ".join(str(int(x)) for x in r) + "\n" for r in requests)
    out = subprocess.run([_program()], input=text, capture_output=True, text=True, check=True).stdout
    rows = [dict(zip(FIELDS, map(int, line.split()))) for line in out.splitlines()]
    assert len(rows) == len(requests)
    for r in rows:
        r["path"] = PATHS[r["path"]]
    return rows
