// Tiles of the operator on a box mesh, and the assembly of their outputs
// without atomics.
//
// A tile is kx x ky x kz neighbouring elements of the box, worked on by one
// workgroup, which sums the elements' shared nodes in LDS.  Of the tile's
// (kx N + 1)(ky N + 1)(kz N + 1) nodes it owns all but the last plane in each
// direction (the last tile of a direction owns that plane too), so every DOF
// has one owner, which stores its sum to y.  The nodes of the last planes
// belong to neighbouring tiles: their sums go to the halo, three families of
// planes that each have one writer per entry:
//   HZ [tz][J][I]        the last z plane of tile layer tz, whole DOF rows;
//   HY [ty][tz][c][I]    the last y plane of tile row ty, c = 0 .. kz N;
//   HX [tx][ty][tz][c][j] the last x plane, j = 0 .. ky N
// (an edge or corner node goes to HX if it lies on the last x plane, else to HY
// if on the last y plane, else to HZ; I, J, K number the box's nodes, masked
// ones included).  Whoever consumes y next adds the halo: the residual step of
// CG as it reads Ap, or the finishing kernel of hb_ax.  Every sum has a fixed
// order, so results are the same from run to run.
//
// Plain arithmetic for host and device: the host plans tiles, tests check the
// ownership and the halo against brute force.
#pragma once

#include <cstdint>

#include "walk.h"

#if defined(__HIP__) || defined(__HIPCC__)
#define HB_HD __host__ __device__
#else
#define HB_HD
#endif

namespace hb {

// Division of 0 <= n < 2^31 by a fixed d >= 1: multiply high and shift.
// m = ceil(2^(32+s) / d) with 2^s < d <= 2^(s+1): the error of m d against
// 2^(32+s) is below 2^(s+1), which times n < 2^31 stays below 2^(32+s).
struct FastDiv {
    uint32_t d = 1, m = 0, s = 0;
    HB_HD uint32_t operator()(uint32_t n) const
    {
        if (d == 1) return n;
        return static_cast<uint32_t>((static_cast<uint64_t>(n) * m) >> 32) >> s;
    }
};
inline FastDiv fast_div(uint32_t d)
{
    FastDiv f;
    f.d = d;
    if (d <= 1) return f;
    uint32_t s = 0;
    while ((uint64_t{1} << (s + 1)) < d) ++s;
    f.s = s;
    f.m = static_cast<uint32_t>(((uint64_t{1} << (32 + s)) + d - 1) / d);
    return f;
}

struct TilePlan {
    int32_t N = 1;
    int32_t nx = 1, ny = 1, nz = 1;     // elements of the box
    int32_t kx = 1, ky = 1, kz = 1;     // elements of a full tile
    int32_t ntx = 1, nty = 1, ntz = 1;  // tiles (the last of a direction may be short)
    int32_t gx = 2, gy = 2, gz = 2;     // nodes of the box
    int32_t sx = 2, sxy = 4;            // DOF strides of y and z
    int32_t off = 0;                    // DOF of node (I,J,K): off + I + sx J + sxy K (off < 0 on a masked box)
    int32_t mask = 0;                   // 1: the box's boundary nodes carry no DOF
    int32_t invdeg = 0;                 // mass coefficient 1 / multiplicity
    int32_t wide = 0;                   // a tile's DOFs lie 2^32 bytes or more apart (offsets take 64 bits)
    uint32_t hy = 0, hx = 0;            // starts of HY and HX in the halo (HZ starts at 0)
    uint32_t halo = 0;                  // entries of the halo
    TileWalk walk;                      // the order in which a launch visits the tiles
    FastDiv row, plane;                 // DOF -> row, row -> plane of DOFs
    FastDiv px, py, pz;                 // node -> tile (division by kx N, ky N, kz N)
    FastDiv ex, exy;                    // element slot of a tile -> its place (division by kx, kx ky)
    FastDiv tx, ty;                     // tile -> row of tiles -> plane of tiles
    FastDiv gxd, gyd, tz, cy, cz;       // division by gx, gy, ntz, ky N + 1, kz N + 1
    FastDiv slab, level, level1;        // tiles of a slab of the walk, of one z in it, of one z in the last slab

    HB_HD int32_t tiles() const { return ntx * nty * ntz; }
    HB_HD uint32_t hz_at(int32_t tz, int32_t J, int32_t I) const
    {
        return (static_cast<uint32_t>(tz) * gy + J) * gx + I;
    }
    HB_HD uint32_t hy_at(int32_t ty, int32_t tz, int32_t c, int32_t I) const
    {
        return hy + (static_cast<uint32_t>(ty * ntz + tz) * (kz * N + 1) + c) * gx + I;
    }
    HB_HD uint32_t hx_at(int32_t tx, int32_t ty, int32_t tz, int32_t c, int32_t j) const
    {
        return hx + (static_cast<uint32_t>((tx * nty + ty) * ntz + tz) * (kz * N + 1) + c) * (ky * N + 1) + j;
    }
};

// The halo entries of node (I,J,K): up to seven, none where its owner is the only
// tile that touches it.  load() fetches them and sum() adds them in a fixed order,
// so that several nodes' loads can be in flight together: as they are in memory, since
// a conversion would wait for its load inside the branch (FP32 operator, 13^3 N = 7 28.4 us
// an iteration of CG against 26.6).  The two of a corner, which few nodes have, arrive as
// one in FP64, to hold fewer registers.  The branches are nested by how
// often a wave of consecutive nodes takes them: in a residual step of CG at 32^3 N = 7
// 50.0 us against 51.7 with one branch to an entry, at 11x10x9 N = 11 10.0 against
// 11.1; 54.9 and 11.6 with the entries of the three faces read unconditionally.
// T: the halo's type; h: anything indexable by a halo position.
template <typename T>
struct HaloNode {
    static constexpr bool apart = sizeof(T) == 4;  // a corner's two entries
    T v[apart ? 7 : 6];
    template <typename H>
    HB_HD void load(const TilePlan &p, const H &h, int32_t I, int32_t J, int32_t K)
    {
        const int32_t tx = static_cast<int32_t>(p.px(I)), ty0 = static_cast<int32_t>(p.py(J)),
                      tz0 = static_cast<int32_t>(p.pz(K));
        const int32_t wx = p.kx * p.N, wy = p.ky * p.N, wz = p.kz * p.N;
        // on the first plane of a tile with a neighbour below it (the box's last
        // plane is in the last tile, never on the first plane of one)
        const bool ax = I == tx * wx && tx > 0 && tx < p.ntx;
        const bool ay = J == ty0 * wy && ty0 > 0 && ty0 < p.nty;
        const bool az = K == tz0 * wz && tz0 > 0 && tz0 < p.ntz;
        const int32_t ty = ty0 < p.nty ? ty0 : p.nty - 1, tz = tz0 < p.ntz ? tz0 : p.ntz - 1;
        const int32_t c = K - tz * wz, j = J - ty * wy;
        for (T &x : v) x = T(0);
        if (ax) v[2] = h[p.hx_at(tx - 1, ty, tz, c, j)];
        if (ay | az) {
            if (az) {
                v[0] = h[p.hz_at(tz - 1, J, I)];
                if (ax) v[3] = h[p.hx_at(tx - 1, ty, tz - 1, wz, j)];
            }
            if (ay) {
                v[1] = h[p.hy_at(ty - 1, tz, c, I)];
                if (ax) v[4] = h[p.hx_at(tx - 1, ty - 1, tz, c, wy)];
                if (az) {
                    v[5] = h[p.hy_at(ty - 1, tz - 1, wz, I)];
                    if (ax) {
                        const T last = h[p.hx_at(tx - 1, ty - 1, tz - 1, wz, wy)];
                        if constexpr (apart)
                            v[6] = last;
                        else
                            v[5] += last;
                    }
                }
            }
        }
    }
    HB_HD double sum()
    {
#if defined(__HIP_DEVICE_COMPILE__)
        // here, and not before the loads of other nodes: the compiler would convert each
        // value in the branch that loads it
        if constexpr (apart)
            for (T &x : v) asm volatile("" : "+v"(x));
#endif
        double s = 0.0;
        for (int k = 0; k < 5; ++k) s += static_cast<double>(v[k]);
        double corner = static_cast<double>(v[5]);
        if constexpr (apart) corner += static_cast<double>(v[6]);
        return s + corner;
    }
};
template <typename H>
HB_HD inline double halo_sum(const TilePlan &p, const H &h, int32_t I, int32_t J, int32_t K)
{
    HaloNode<decltype(+h[0])> n;
    n.load(p, h, I, J, K);
    return n.sum();
}

// Node of DOF g.
struct Node {
    int32_t I, J, K;
};
HB_HD inline Node dof_node(const TilePlan &p, uint32_t g)
{
    const uint32_t r = p.row(g), k = p.plane(r);
    const int32_t sy = static_cast<int32_t>(p.plane.d);
    return Node{static_cast<int32_t>(g - r * p.row.d) + p.mask, static_cast<int32_t>(r) - static_cast<int32_t>(k) * sy + p.mask,
                static_cast<int32_t>(k) + p.mask};
}
template <typename H>
HB_HD inline double halo_sum(const TilePlan &p, const H &h, uint32_t g)
{
    const Node n = dof_node(p, g);
    return halo_sum(p, h, n.I, n.J, n.K);
}

// y += the halo: entry n of the halo, if it is the first of its node (in the order
// HZ, HY, HX), adds the node's whole sum.
template <typename T>
HB_HD inline void halo_add(const TilePlan &p, const T *halo, T *y, uint32_t n)
{
    if (n >= p.halo) return;
    const int32_t wx = p.kx * p.N, wy = p.ky * p.N, wz = p.kz * p.N;
    int32_t I, J, K;
    if (n < p.hy) {
        const uint32_t r = p.gxd(n), q = p.gyd(r);
        I = static_cast<int32_t>(n - r * p.gx);
        J = static_cast<int32_t>(r - q * p.gy);
        K = static_cast<int32_t>(q + 1) * wz;
    } else if (n < p.hx) {
        n -= p.hy;
        const uint32_t r = p.gxd(n), q = p.cz(r), ty = p.tz(q);
        const int32_t c = static_cast<int32_t>(r - q * (wz + 1)), tz = static_cast<int32_t>(q - ty * p.ntz);
        I = static_cast<int32_t>(n - r * p.gx);
        J = static_cast<int32_t>(ty + 1) * wy;
        K = tz * wz + c;
        if ((c == 0 && tz > 0) || (c == wz && tz < p.ntz - 1) || K >= p.gz) return;  // on a z plane of the halo
    } else {
        n -= p.hx;
        const uint32_t r = p.cy(n), q = p.cz(r), v = p.tz(q), tx = p.ty(v);
        const int32_t j = static_cast<int32_t>(n - r * (wy + 1)), c = static_cast<int32_t>(r - q * (wz + 1));
        const int32_t tz = static_cast<int32_t>(q - v * p.ntz), ty = static_cast<int32_t>(v - tx * p.nty);
        I = static_cast<int32_t>(tx + 1) * wx;
        J = ty * wy + j;
        K = tz * wz + c;
        if ((c == 0 && tz > 0) || (c == wz && tz < p.ntz - 1) || K >= p.gz) return;
        if ((j == 0 && ty > 0) || (j == wy && ty < p.nty - 1) || J >= p.gy) return;  // on a y plane of the halo
    }
    if (p.mask && (I == 0 || J == 0 || K == 0 || I == p.gx - 1 || J == p.gy - 1 || K == p.gz - 1)) return;
    T &out = y[static_cast<int64_t>(p.off) + I + static_cast<int64_t>(p.sx) * J + static_cast<int64_t>(p.sxy) * K];
    out = static_cast<T>(static_cast<double>(out) + halo_sum(p, halo, I, J, K));
}

// A tile's place in the tile grid.
struct TilePlace {
    int32_t x, y, z;
};
HB_HD inline TilePlace tile_place(const TilePlan &p, uint32_t tile)
{
    const uint32_t row = p.tx(tile), z = p.ty(row);
    return TilePlace{static_cast<int32_t>(tile - row * p.tx.d), static_cast<int32_t>(row - z * p.ty.d),
                     static_cast<int32_t>(z)};
}
// tile_place of walk_tile(walk, j), without its divisions.
HB_HD inline TilePlace place_in_walk(const TilePlan &p, uint32_t j)
{
    const uint32_t s = p.slab(j), r = j - s * p.slab.d, y0 = s * p.walk.ys;
    const bool full = y0 + p.walk.ys <= p.walk.ny;
    const FastDiv level{full ? p.level.d : p.level1.d, full ? p.level.m : p.level1.m, full ? p.level.s : p.level1.s};
    const uint32_t z = level(r), r2 = r - z * level.d, y = p.tx(r2);
    return TilePlace{static_cast<int32_t>(r2 - y * p.tx.d), static_cast<int32_t>(y0 + y), static_cast<int32_t>(z)};
}

// The plan with the given tile shape.
inline TilePlan make_plan(int N, int nx, int ny, int nz, bool mask, bool invdeg, int kx, int ky, int kz)
{
    TilePlan p;
    p.N = N;
    p.nx = nx;
    p.ny = ny;
    p.nz = nz;
    p.kx = kx;
    p.ky = ky;
    p.kz = kz;
    p.ntx = (nx + kx - 1) / kx;
    p.nty = (ny + ky - 1) / ky;
    p.ntz = (nz + kz - 1) / kz;
    p.gx = nx * N + 1;
    p.gy = ny * N + 1;
    p.gz = nz * N + 1;
    p.mask = mask ? 1 : 0;
    p.invdeg = invdeg ? 1 : 0;
    p.sx = mask ? p.gx - 2 : p.gx;
    const int sy = mask ? p.gy - 2 : p.gy;
    p.sxy = p.sx * sy;
    p.off = mask ? -(1 + p.sx + p.sxy) : 0;
    // the farthest node read from a tile's first, less the layer of a column (a masked
    // node's column starts one layer up)
    const int64_t reach = static_cast<int64_t>(kx) * N + static_cast<int64_t>(p.sx) * (static_cast<int64_t>(ky) * N) +
                          static_cast<int64_t>(p.sxy) * (static_cast<int64_t>(kz - 1) * N + p.mask);
    p.wide = 8 * reach >= int64_t{1} << 32 ? 1 : 0;
    p.hy = static_cast<uint32_t>(static_cast<int64_t>(p.ntz - 1) * p.gy * p.gx);
    p.hx = p.hy + static_cast<uint32_t>(static_cast<int64_t>(p.nty - 1) * p.ntz * (kz * N + 1) * p.gx);
    p.halo = p.hx + static_cast<uint32_t>(static_cast<int64_t>(p.ntx - 1) * p.nty * p.ntz * (kz * N + 1) * (ky * N + 1));
    p.walk = make_walk(p.ntx, p.nty, p.ntz, 1);
    p.slab = fast_div(p.walk.txn * p.walk.ys * p.walk.nz);
    p.level = fast_div(p.walk.txn * p.walk.ys);
    const uint32_t last = p.walk.ny % p.walk.ys;
    p.level1 = fast_div(p.walk.txn * (last ? last : p.walk.ys));
    p.row = fast_div(p.sx > 0 ? p.sx : 1);
    p.plane = fast_div(sy > 0 ? sy : 1);
    p.tx = fast_div(p.ntx);
    p.ty = fast_div(p.nty);
    p.gxd = fast_div(p.gx);
    p.gyd = fast_div(p.gy);
    p.tz = fast_div(p.ntz);
    p.cy = fast_div(ky * N + 1);
    p.cz = fast_div(kz * N + 1);
    p.ex = fast_div(kx);
    p.exy = fast_div(kx * ky);
    p.px = fast_div(kx * N);
    p.py = fast_div(ky * N);
    p.pz = fast_div(kz * N);
    return p;
}

// Tile shape for workgroups of `epb` elements: of all kx ky kz <= epb the one
// with the least modelled cost, (element slots)(N+1)^3 + 2 (halo entries) + 4 per
// row of nodes a tile stores (a row is a run of consecutive DOFs: short runs
// leave most of a memory request empty).
inline TilePlan plan_tiles(int N, int nx, int ny, int nz, bool mask, bool invdeg, int epb)
{
    TilePlan best;
    double best_cost = -1.0;
    for (int kz = 1; kz <= epb && kz <= nz; ++kz)
        for (int ky = 1; ky * kz <= epb && ky <= ny; ++ky) {
            int kx = epb / (ky * kz);
            if (kx > nx) kx = nx;
            const double tiles = static_cast<double>((nx + kx - 1) / kx) * ((ny + ky - 1) / ky) * ((nz + kz - 1) / kz);
            const double n1 = N + 1;
            const double gx = static_cast<double>(nx) * N + 1, gy = static_cast<double>(ny) * N + 1;
            const double ntx = (nx + kx - 1) / kx, nty = (ny + ky - 1) / ky, ntz = (nz + kz - 1) / kz;
            const double halo = (ntz - 1) * gy * gx + (nty - 1) * ntz * (kz * N + 1) * gx +
                                (ntx - 1) * nty * ntz * (kz * N + 1.0) * (ky * N + 1.0);
            const double cost = tiles * epb * n1 * n1 * n1 + 2.0 * halo + 4.0 * tiles * (ky * N + 1.0) * (kz * N + 1.0);
            if (best_cost < 0.0 || cost < best_cost) {
                best_cost = cost;
                best = make_plan(N, nx, ny, nz, mask, invdeg, kx, ky, kz);
            }
        }
    return best;
}

}  // namespace hb
