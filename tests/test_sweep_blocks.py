"""The host side of the face-flux pass' block shapes: the tiles cover every cell
once, no shape is chosen that takes more threads than the large one, and a tile
asked for names a shape."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2110_10191_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include "common.h"
int main() {
  int n1, n2, n3, recon, mixed, stx, sty;
  while (scanf("%d %d %d %d %d %d %d", &n1, &n2, &n3, &recon, &mixed, &stx, &sty) == 7) {
    Dims d{};
    d.n1 = n1, d.n2 = n2, d.n3 = n3;
    SweepBlocks b;
    b.add(d, recon, mixed != 0);
    set_sweep_shape(d, sweep_shape(stx, sty, b, recon, mixed != 0), recon, mixed != 0);
    printf("%d %d %d %d %d\n", d.sbx, d.sby, sweep_tiles_x1(n1, d.sbx), sweep_tiles_x2(n2, d.sby), (int)sweep_grid(d, d.sbx, d.sby));
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    """{(n1, n2, n3, recon, mixed, tile)} -> (bx, by, tiles in x1, tiles in x2, blocks), in one run of the library's rule"""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    d = tmp_path_factory.mktemp("blocks")
    (d / "blocks.hip").write_text(SOURCE)
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-w", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    str(d / "blocks.hip"), "-o", str(d / "blocks")], check=True, capture_output=True)

    def run(cases):
        text = "".join("%d %d %d %d %d %d %d\n" % (*c[:5], *c[5]) for c in cases)
        out = subprocess.run([str(d / "blocks")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]
    return run


AUTO, LARGE, SMALL, NARROW = (64, 8), (128, 4), (32, 8), (16, 8)
MODES = [(r, m) for r in (0, 1) for m in (0, 1)]


def test_tiles_cover_every_cell_with_no_tile_to_spare(shapes):
    cases = [(n1, n2, 5, r, m, t) for r, m in MODES for t in (AUTO, LARGE, SMALL, NARROW)
             for n1, n2 in [(n, 1 + n % 37) for n in range(1, 200)]]
    for (n1, n2, *_), (bx, by, t1, t2, _) in zip(cases, shapes(cases)):
        # divergences of columns 1..bx-2 and rows 0..by-2 of a tile (from cell -1), edges of cell n
        # in the last tile's last column and row at the latest
        assert t1 * (bx - 2) >= n1 > (t1 - 1) * (bx - 2)
        assert t2 * (by - 1) >= n2 + 1 > (t2 - 1) * (by - 1)


def test_the_grid_decides_for_the_default_tile_only(shapes):
    grids = [(8, 256, 128), (14, 14, 14), (15, 256, 128), (30, 200, 100), (62, 7, 900), (400, 4, 400), (64, 64, 1),
             (131, 67, 45), (288, 128, 128)]
    cases = [(*g, r, m, t) for g in grids for r, m in MODES for t in (AUTO, LARGE, SMALL, NARROW)]
    got = dict(zip(cases, shapes(cases)))
    for g in grids:
        for r, m in MODES:
            auto, large, small, narrow = (got[(*g, r, m, t)] for t in (AUTO, LARGE, SMALL, NARROW))
            assert large[:2] == ((32, 16) if (r, m) == (1, 0) else (64, 8))
            assert small[:2] == (32, 8) and narrow[:2] == (16, 8)
            threads = lambda s: s[0] * s[1] * s[4]
            assert auto in (large, small, narrow)
            assert auto[4] < 1024 or threads(auto) <= threads(large)
            if g[0] <= 14:
                assert auto == narrow
            if g == (288, 128, 128):
                assert auto == large
            # no more threads than tiles of 64 x 8 cells would take, but for the rows that overlap
            assert threads(auto) <= 1.5 * 512 * -(-(g[0] + 2) // 64) * -(-(g[1] + 2) // 8) * -(-(g[2] + 2) // 8) * 8
