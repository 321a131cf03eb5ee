"""The operator's tiles (tile.h): host-side checks of the very header the kernels
include, compiled with the host compiler.  For every tile shape of a set of boxes
(plain and masked, short last tiles, one-element tiles), each tile's node sums are
stored as the kernel stores them -- to y if the tile owns the node, else to the
halo -- and every y entry and halo position must have one writer, and y plus
halo_sum (or halo_add over the halo's entries) must be the sum over all tiles that
touch the node (integers, exact).
FastDiv is checked against / at the edges of its range."""
import os
import shutil
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2202_12477_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "tile.h"
using namespace hb;
static int check(const TilePlan &p) {
    const int lx = p.gx, ly = p.gy, lz = p.gz;
    const long nd = (long)(lx - 2 * p.mask) * (ly - 2 * p.mask) * (lz - 2 * p.mask);
    std::vector<double> y(nd, 0), h(p.halo + 1, 0), ref((size_t)lx * ly * lz, 0);
    std::vector<int> wy(nd, 0), wh(p.halo + 1, 0), seen(p.tiles(), 0);
    for (int b = 0; b < p.tiles(); ++b) {
        const uint32_t t = walk_tile(p.walk, b);
        if ((int)t >= p.tiles() || seen[t]++) return 1;
        const int row = t / p.ntx, tx = t - row * p.ntx, tz = row / p.nty, ty = row - tz * p.nty;
        const int ex = p.nx - tx * p.kx < p.kx ? p.nx - tx * p.kx : p.kx;
        const int ey = p.ny - ty * p.ky < p.ky ? p.ny - ty * p.ky : p.ky;
        const int ez = p.nz - tz * p.kz < p.kz ? p.nz - tz * p.kz : p.kz;
        if (ex < 1 || ey < 1 || ez < 1) return 2;
        for (int k = 0; k <= ez * p.N; ++k)
            for (int j = 0; j <= ey * p.N; ++j)
                for (int i = 0; i <= ex * p.N; ++i) {
                    const int I = tx * p.kx * p.N + i, J = ty * p.ky * p.N + j, K = tz * p.kz * p.N + k;
                    const double v = rand() % 1000 + 1;
                    ref[I + (size_t)lx * (J + (size_t)ly * K)] += v;
                    const bool hx = i == ex * p.N && tx < p.ntx - 1, hy = j == ey * p.N && ty < p.nty - 1,
                               hz = k == ez * p.N && tz < p.ntz - 1;
                    if (hx | hy | hz) {
                        const uint32_t at = hx ? p.hx_at(tx, ty, tz, k, j) : hy ? p.hy_at(ty, tz, k, I) : p.hz_at(tz, J, I);
                        if (at >= p.halo || wh[at]++) return 3;
                        h[at] = v;
                    } else if (!(p.mask && (I == 0 || J == 0 || K == 0 || I == lx - 1 || J == ly - 1 || K == lz - 1))) {
                        const long at = (long)p.off + I + (long)p.sx * J + (long)p.sxy * K;
                        if (at < 0 || at >= nd || wy[at]++) return 4;
                        y[at] = v;
                    }
                }
    }
    for (long g = 0; g < nd; ++g) {
        const Node n = dof_node(p, (uint32_t)g);
        if (!wy[g] || (long)p.off + n.I + (long)p.sx * n.J + (long)p.sxy * n.K != g) return 5;
        if (halo_sum(p, h, n.I, n.J, n.K) != halo_sum(p, h, (uint32_t)g)) return 7;
        if (y[g] + halo_sum(p, h, (uint32_t)g) != ref[n.I + (size_t)lx * (n.J + (size_t)ly * n.K)]) return 6;
    }
    for (uint32_t n = 0; n < p.halo + 3; ++n) halo_add(p, h.data(), y.data(), n);
    for (long g = 0; g < nd; ++g) {
        const Node n = dof_node(p, (uint32_t)g);
        if (y[g] != ref[n.I + (size_t)lx * (n.J + (size_t)ly * n.K)]) return 8;
    }
    return 0;
}
int main() {
    const uint32_t ns[] = {0, 1, 2, 3, 5, 127, 128, 65535, 65536, 1000003, 2147483646u, 2147483647u};
    for (uint32_t d = 1; d < 5000; ++d) {
        const FastDiv f = fast_div(d);
        for (uint32_t n : ns) if (f(n) != n / d) { printf("div %u %u\n", n, d); return 1; }
        for (uint32_t k = 1; k < 40; ++k) for (int o = -1; o <= 1; ++o) {
            const uint64_t n = (uint64_t)d * ((2147483647ull / d) / k) + o;
            if (n < 2147483648ull && f((uint32_t)n) != n / d) { printf("div %lu %u\n", (unsigned long)n, d); return 1; }
        }
    }
    for (uint32_t d : {2147483647u, 1u << 30, (1u << 30) + 1, 99999999u})
        for (uint32_t n : ns) if (fast_div(d)(n) != n / d) { printf("div %u %u\n", n, d); return 1; }
    long cases = 0;
    const int boxes[][3] = {{1,1,1},{2,1,1},{1,3,1},{1,1,4},{3,2,2},{5,3,4},{4,4,4},{7,1,3}};
    for (int N = 1; N <= 4; ++N)
        for (auto &b : boxes)
            for (int mask = 0; mask <= 1; ++mask) {
                if (mask && (b[0] * N < 2 || b[1] * N < 2 || b[2] * N < 2)) continue;
                for (int kx = 1; kx <= b[0]; ++kx) for (int ky = 1; ky <= b[1]; ++ky) for (int kz = 1; kz <= b[2]; ++kz, ++cases) {
                    const int r = check(make_plan(N, b[0], b[1], b[2], mask, false, kx, ky, kz));
                    if (r) { printf("N=%d box %dx%dx%d tile %dx%dx%d mask %d: %d\n", N, b[0], b[1], b[2], kx, ky, kz, mask, r); return 1; }
                }
                for (int epb : {1, 2, 4, 7, 16, 64}) {
                    const TilePlan p = plan_tiles(N, b[0], b[1], b[2], mask, false, epb);
                    if (p.kx * p.ky * p.kz > epb || check(p)) { printf("plan N=%d epb %d\n", N, epb); return 1; }
                }
            }
    printf("ok %ld\n", cases);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_tiles_cover_every_node_once():
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "t.cpp"), os.path.join(d, "t")
        with open(src, "w") as f:
            f.write(HARNESS)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, src, "-o", exe], check=True)
        out = subprocess.run([exe], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout
        assert out.stdout.startswith("ok")
