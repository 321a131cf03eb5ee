"""The launch-time arithmetic of the operator's tiles (tile.h), compiled with the host
compiler: the place of a launch's j-th tile without divisions is that of the walk's tile,
for every tile of a set of boxes (slabs of several heights, a short last slab); and a plan
is marked wide exactly when a byte offset from a tile's first node, as the operator forms
it, can pass 32 bits."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2202_12477_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <initializer_list>
#include "tile.h"
using namespace hb;
static long places = 0;
static int check_places(int N, int nx, int ny, int nz, int kx, int ky, int kz) {
    const TilePlan p = make_plan(N, nx, ny, nz, false, false, kx, ky, kz);
    for (int j = 0; j < p.tiles(); ++j, ++places) {
        const TilePlace a = place_in_walk(p, j), b = tile_place(p, walk_tile(p.walk, j));
        if (a.x != b.x || a.y != b.y || a.z != b.z) return 1;
    }
    return 0;
}
// the farthest offset, by the operator's expressions, over the tile's corner columns
static int check_wide(int N, int nx, int ny, int nz, bool mask, int kx, int ky, int kz) {
    const TilePlan p = make_plan(N, nx, ny, nz, mask, false, kx, ky, kz);
    int64_t far = 0;
    for (int lx : {0, kx - 1}) for (int ly : {0, ky - 1}) for (int lz : {0, kz - 1})
        for (int a : {0, N}) for (int b : {0, N}) {
            if (lx >= nx || ly >= ny || lz >= nz) continue;
            const int64_t o = (int64_t)lx * N + a + (int64_t)p.sx * (ly * N + b) + (int64_t)p.sxy * (lz * N) + (mask ? p.sxy : 0);
            if (o > far) far = o;
        }
    const bool need = 8 * far >= (int64_t{1} << 32);
    return need && !p.wide ? 1 : (!need && p.wide && nx >= kx && ny >= ky && nz >= kz) ? 2 : 0;
}
int main() {
    int bad = 0;
    for (int nx : {1, 2, 5, 16, 33}) for (int ny : {1, 3, 8, 9, 17, 40}) for (int nz : {1, 2, 7, 20})
        for (int kx : {1, 4}) for (int ky : {1, 2}) for (int kz : {1, 3})
            if (check_places(2, nx, ny, nz, kx, ky, kz)) { printf("place %d %d %d %d%d%d\n", nx, ny, nz, kx, ky, kz); ++bad; }
    for (bool mask : {false, true}) {
        // flat boxes on either side of 2^29 DOFs between a tile's ends
        for (int n : {5000, 13376, 13377, 13378, 13379, 13380, 13400})
            for (int kz : {1, 2}) if (int e = check_wide(3, n / 3, n / 3, 2, mask, 4, 2, kz)) { printf("wide %d %d %d: %d\n", n, kz, mask, e); ++bad; }
        for (int n : {11583, 11584, 11585, 11586, 11587, 11588, 11589})
            if (int e = check_wide(1, n, n, 4, mask, 8, 2, 4)) { printf("wide1 %d %d: %d\n", n, mask, e); ++bad; }
        for (int n : {67108800, 67108863, 67108864, 100000000}) if (int e = check_wide(2, n, 1, 1, mask, 28, 1, 1)) { printf("strip %d %d: %d\n", n, mask, e); ++bad; }
        if (check_wide(7, 32, 32, 32, mask, 4, 1, 1) || make_plan(7, 32, 32, 32, mask, false, 4, 1, 1).wide) { printf("ordinary\n"); ++bad; }
    }
    printf("%ld places, %d bad\n", places, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_places_and_wide_plans(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


WIDE_BOXES = [(1, 5_000_000, 4, 3, 0), (1, 1_650_000, 2, 7, 1)]  # nx, ny, nz, N, masked: as in test_gpu_wide.py

WIDE = r"""
#include <cstdio>
#include <cstdlib>
#include "tile.h"
using namespace hb;
int main(int argc, char **argv) {
    const int nx = atoi(argv[1]), ny = atoi(argv[2]), nz = atoi(argv[3]), N = atoi(argv[4]), mask = atoi(argv[5]);
    const int np2 = (N + 1) * (N + 1);
    const TilePlan a = plan_tiles(N, nx, ny, nz, mask, false, 256 / np2), b = plan_tiles(N, nx, ny, nz, mask, false, 64 / np2);
    printf("%d %d\n", a.wide, b.wide);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("box", WIDE_BOXES)
def test_boxes_wide_in_one_shape_only(tmp_path, box):
    """The boxes of the GPU test of wide tiles are wide with 256-thread workgroups and not
    with one-wave ones."""
    src, exe = tmp_path / "wide.cpp", tmp_path / "wide"
    src.write_text(WIDE)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), *map(str, box)], capture_output=True, text=True, timeout=60)
    assert r.stdout.split() == ["1", "0"]
