// Mesh setup on the device: vertex jitter, the elements' trilinear maps, and for the
// export the scatter map Z, the geometric factors G (NekBone section: the symmetric 3x3
// block of diagonal matrices of metric terms combined with GLL weights) and the mass
// coefficient c; the diagonal for the Jacobi preconditioner; plus the pseudo-random
// forcing kernel of the HipBone section.
//
// Random numbers: splitmix64 (Steele, Lea & Flood, OOPSLA 2014).  A stream's
// start state is the generator's output number `stream` from state `seed`;
// value number i of the stream is the generator's output number i from that
// start state.  Output number i from state s is finalise(s + (i+1) * gamma).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "common.h"

namespace hb {
namespace {

__host__ __device__ inline uint64_t sm64(uint64_t state, uint64_t i)
{
    uint64_t z = state + (i + 1) * 0x9E3779B97F4A7C15ULL;
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ULL;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}

__device__ inline double unit_uniform(uint64_t stream_start, uint64_t i)
{
    return static_cast<double>(sm64(stream_start, i) >> 11) * 0x1.0p-53;
}

__global__ void rhs_kernel(int64_t n, uint64_t start, double *__restrict__ b)
{
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x)
        b[g] = 2.0 * unit_uniform(start, static_cast<uint64_t>(g)) - 1.0;
}

// Vertex coordinates [(nx+1)(ny+1)(nz+1)][3]; interior vertices are jittered.
__global__ void vertex_kernel(int nx, int ny, int nz, double jitter, uint64_t sx, uint64_t sy, uint64_t sz,
                              double *__restrict__ V)
{
    const int64_t nv = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const int i = static_cast<int>(v % (nx + 1));
    const int j = static_cast<int>((v / (nx + 1)) % (ny + 1));
    const int k = static_cast<int>(v / ((int64_t)(nx + 1) * (ny + 1)));
    double c[3] = {(double)i / nx, (double)j / ny, (double)k / nz};
    const bool interior = i > 0 && i < nx && j > 0 && j < ny && k > 0 && k < nz;
    if (interior && jitter != 0.0) {
        const uint64_t st[3] = {sx, sy, sz};
        const int n[3] = {nx, ny, nz};
        for (int d = 0; d < 3; ++d)
            c[d] += (jitter / n[d]) * (2.0 * unit_uniform(st[d], static_cast<uint64_t>(v)) - 1.0);
    }
    V[3 * v + 0] = c[0];
    V[3 * v + 1] = c[1];
    V[3 * v + 2] = c[2];
}

// One thread per local node of elements e0 .. e0 + ne - 1: the Jacobian of the trilinear
// map, which has to be positive everywhere (*bad); STORE: the row of Z, G and c.
// Nothing of this is kept with the mesh: the operator recomputes it (ax_impl.h), and so
// does the export, in pieces.  Storing 60 bytes per node and their allocation were most
// of the time of creating a mesh (32^3 N = 7: 1.40 ms, of which 0.28 ms this kernel).
template <bool STORE>
__global__ __launch_bounds__(256) void geometry_kernel(int nx, int ny, int nz, int N, int64_t e0, int64_t ne,
                                                       const double *__restrict__ V, const double *__restrict__ xw,
                                                       int mass_invdeg, int dirichlet, int32_t *__restrict__ map,
                                                       double *__restrict__ geo, int *__restrict__ bad)
{
    const int n1 = N + 1;
    const int64_t np3 = (int64_t)n1 * n1 * n1;
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= ne * np3) return;
    const int64_t el = t / np3, e = e0 + el;
    const int n = static_cast<int>(t - el * np3);
    const int a = n % n1, b = (n / n1) % n1, c = n / (n1 * n1);
    const int ex = static_cast<int>(e % nx), ey = static_cast<int>((e / nx) % ny), ez = static_cast<int>(e / ((int64_t)nx * ny));
    // Trilinear map x(r) = sum over corners of X_corner * prod_d (1 +- r_d)/2.
    const double r = xw[2 * a], s = xw[2 * b], tt = xw[2 * c];
    const double lo[3] = {0.5 * (1.0 - r), 0.5 * (1.0 - s), 0.5 * (1.0 - tt)};
    const double hi[3] = {0.5 * (1.0 + r), 0.5 * (1.0 + s), 0.5 * (1.0 + tt)};
    double jac[3][3] = {{0.0}};  // jac[i][d] = d x_i / d r_d
    for (int corner = 0; corner < 8; ++corner) {
        const int dx = corner & 1, dy = (corner >> 1) & 1, dz = corner >> 2;
        const int64_t v = (ex + dx) + (int64_t)(nx + 1) * ((ey + dy) + (int64_t)(ny + 1) * (ez + dz));
        const double fx = dx ? hi[0] : lo[0], fy = dy ? hi[1] : lo[1], fz = dz ? hi[2] : lo[2];
        const double gxr = (dx ? 0.5 : -0.5) * fy * fz;
        const double gys = fx * (dy ? 0.5 : -0.5) * fz;
        const double gzt = fx * fy * (dz ? 0.5 : -0.5);
        for (int i = 0; i < 3; ++i) {
            const double X = V[3 * v + i];
            jac[i][0] += X * gxr;
            jac[i][1] += X * gys;
            jac[i][2] += X * gzt;
        }
    }
    // cofactors: inv[d][i] = d r_d / d x_i = cof[i][d] / J
    const double c00 = jac[1][1] * jac[2][2] - jac[1][2] * jac[2][1];
    const double c01 = jac[1][2] * jac[2][0] - jac[1][0] * jac[2][2];
    const double c02 = jac[1][0] * jac[2][1] - jac[1][1] * jac[2][0];
    const double c10 = jac[0][2] * jac[2][1] - jac[0][1] * jac[2][2];
    const double c11 = jac[0][0] * jac[2][2] - jac[0][2] * jac[2][0];
    const double c12 = jac[0][1] * jac[2][0] - jac[0][0] * jac[2][1];
    const double c20 = jac[0][1] * jac[1][2] - jac[0][2] * jac[1][1];
    const double c21 = jac[0][2] * jac[1][0] - jac[0][0] * jac[1][2];
    const double c22 = jac[0][0] * jac[1][1] - jac[0][1] * jac[1][0];
    const double J = jac[0][0] * c00 + jac[0][1] * c01 + jac[0][2] * c02;
    if (!(J > 0.0)) atomicOr(bad, 1);
    if constexpr (STORE) {
        const int64_t gx = (int64_t)nx * N + 1, gy = (int64_t)ny * N + 1, gz = (int64_t)nz * N + 1;
        const int64_t gi = (int64_t)ex * N + a, gj = (int64_t)ey * N + b, gk = (int64_t)ez * N + c;
        const bool edge = gi == 0 || gj == 0 || gk == 0 || gi == gx - 1 || gj == gy - 1 || gk == gz - 1;
        const bool dof = !dirichlet || !edge;
        if (!dof)
            map[t] = -1;  // boundary node: no DOF
        else if (dirichlet)
            map[t] = static_cast<int32_t>((gi - 1) + (gx - 2) * ((gj - 1) + (gy - 2) * (gk - 1)));
        else
            map[t] = static_cast<int32_t>(gi + gx * (gj + gy * gk));
        const double invJ = 1.0 / J;
        // rows of the inverse Jacobian: grad r, grad s, grad t
        const double gr[3] = {c00 * invJ, c10 * invJ, c20 * invJ};
        const double gs[3] = {c01 * invJ, c11 * invJ, c21 * invJ};
        const double gt[3] = {c02 * invJ, c12 * invJ, c22 * invJ};
        const double wJ = xw[2 * a + 1] * xw[2 * b + 1] * xw[2 * c + 1] * J;
        auto dot3 = [](const double *u, const double *v) { return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]; };
        double *g = geo + el * np3 * kGeo + n;  // [element][factor][node]
        g[0 * np3] = wJ * dot3(gr, gr);
        g[1 * np3] = wJ * dot3(gr, gs);
        g[2 * np3] = wJ * dot3(gr, gt);
        g[3 * np3] = wJ * dot3(gs, gs);
        g[4 * np3] = wJ * dot3(gs, gt);
        g[5 * np3] = wJ * dot3(gt, gt);
        // elements that share the node: two in each direction in which it is on a face
        // between elements
        const bool sx = (a == 0 && ex > 0) || (a == N && ex < nx - 1), sy = (b == 0 && ey > 0) || (b == N && ey < ny - 1),
                   sz = (c == 0 && ez > 0) || (c == N && ez < nz - 1);
        g[6 * np3] = !mass_invdeg ? wJ : dof ? (sx ? 0.5 : 1.0) * (sy ? 0.5 : 1.0) * (sz ? 0.5 : 1.0) : 0.0;
    }
}

// Coefficients of the element's trilinear map in powers of (r, s, t), one thread
// per element: C_100, C_010, C_001, C_110, C_101, C_011, C_111, three components
// each, from the differences along the element's edges (exact, or rounded at the
// size of the edge rather than of the coordinates).
__global__ void coef_kernel(int nx, int ny, int nz, const double *__restrict__ V, double *__restrict__ coef)
{
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)nx * ny * nz) return;
    const int ex = static_cast<int>(e % nx), ey = static_cast<int>((e / nx) % ny), ez = static_cast<int>(e / ((int64_t)nx * ny));
    auto X = [&](int dx, int dy, int dz, int i) {
        return V[3 * ((ex + dx) + (int64_t)(nx + 1) * ((ey + dy) + (int64_t)(ny + 1) * (ez + dz))) + i];
    };
    double *C = coef + 21 * e;
    for (int i = 0; i < 3; ++i) {
        // edges along r at (s,t) corners, along s at (r,t), along t at (r,s)
        double r[2][2], s[2][2], t[2][2];
        for (int u = 0; u < 2; ++u)
            for (int v = 0; v < 2; ++v) {
                r[u][v] = X(1, u, v, i) - X(0, u, v, i);
                s[u][v] = X(u, 1, v, i) - X(u, 0, v, i);
                t[u][v] = X(u, v, 1, i) - X(u, v, 0, i);
            }
        C[0 + i] = 0.125 * ((r[0][0] + r[1][0]) + (r[0][1] + r[1][1]));
        C[3 + i] = 0.125 * ((s[0][0] + s[1][0]) + (s[0][1] + s[1][1]));
        C[6 + i] = 0.125 * ((t[0][0] + t[1][0]) + (t[0][1] + t[1][1]));
        C[9 + i] = 0.125 * ((r[1][0] - r[0][0]) + (r[1][1] - r[0][1]));
        C[12 + i] = 0.125 * ((r[0][1] - r[0][0]) + (r[1][1] - r[1][0]));
        C[15 + i] = 0.125 * ((s[0][1] - s[0][0]) + (s[1][1] - s[1][0]));
        C[18 + i] = 0.125 * ((r[1][1] - r[0][1]) - (r[1][0] - r[0][0]));
    }
}

// Elements of a workgroup of the kernel below: those of the operator's workgroup shape
// (variant_epb); its threads: up to eight element nodes each on the large tiles of
// N <= 7 (50^3 N = 7 1091 us against 1165 with four), else up to four (16^3 N = 15
// 385 us against 488 with sixteen).
constexpr int diag_elements(int N, int v)
{
    const int np2 = (N + 1) * (N + 1), n = (v == 1 && np2 <= 64 ? 64 : 256) / np2;
    return n > 0 ? n : 1;
}
constexpr int diag_threads(int N, int v)
{
    if (v == 0 && N <= 7) return 256;
    return ((diag_elements(N, v) * (N + 1) * (N + 1) * (N + 1) + 3) / 4 + 63) / 64 * 64;
}

// Diagonal of the assembled operator: at node (a,b,c) of an element, (D^T G D +
// lambda C)_ii = sum_m D[m][a]^2 G_rr(m,b,c) + sum_m D[m][b]^2 G_ss(a,m,c)
// + sum_m D[m][c]^2 G_tt(a,b,m) + 2 (D_aa D_bb G_rs + D_aa D_cc G_rt + D_bb D_cc G_st)(i)
// + lambda c(i) (the cross terms meet only at the node itself).  A workgroup works on a
// tile of the operator: it forms its elements' factors from the trilinear maps,
// puts the three it sums along lines into LDS, sums each element's diagonal, and then the
// copies of each node of the tile, in a fixed order, into diag (the nodes the tile owns) or
// the halo, as the operator does (tile.h).  An element's own terms wait in registers.
// 50^3 N = 7 masked 1091 us, 20^3 N = 11 238, 64^3 N = 1 33; 1094, 273 and 43 with a
// workgroup per element and atomic addition, whose sums of four and eight elements came
// in any order; 2241 (50^3 N = 7) with a thread per node reading 3 (N + 1) stored factors.
template <int N, int V>
__global__ __launch_bounds__(diag_threads(N, V)) void jacobi_diag_kernel(TilePlan p, const double *__restrict__ coef,
                                                                   const double *__restrict__ xw,
                                                                   const double *__restrict__ Dm, double lambda,
                                                                   double *__restrict__ diag,
                                                                   double *__restrict__ halo)
{
    extern __shared__ double lines[];
    constexpr int n1 = N + 1, np2 = n1 * n1, np3 = np2 * n1, epb = diag_elements(N, V), threads = diag_threads(N, V);
    constexpr int per = (epb * np3 + threads - 1) / threads;  // element nodes of a thread
    const TilePlace at = tile_place(p, blockIdx.x);
    // the tile's first element, and its elements (the last tile of a direction may be short)
    const int tx = at.x * p.kx, ty = at.y * p.ky, tz = at.z * p.kz;
    const int ex = min(p.kx, p.nx - tx), ey = min(p.ky, p.ny - ty), ez = min(p.kz, p.nz - tz);
    const int nn = ex * ey * ez * np3;
    double *Gr = lines, *Gs = Gr + epb * np3, *Gt = Gs + epb * np3, *D2 = Gt + epb * np3;  // D2: D's entries squared
    for (int t = threadIdx.x; t < np2; t += threads) D2[t] = Dm[t] * Dm[t];
    auto dot3 = [](const double *u, const double *v) { return u[0] * v[0] + u[1] * v[1] + u[2] * v[2]; };
    double sum[per];
#pragma unroll
    for (int q = 0; q < per; ++q) {
        const int t = threadIdx.x + q * threads;
        if (t >= nn) continue;
        const int el = epb == 1 ? 0 : t / np3, n = t - el * np3, a = n % n1, b = (n / n1) % n1, c = n / np2;
        const int lz = el / (ex * ey), ly = (el - lz * ex * ey) / ex, lx = el - (lz * ey + ly) * ex;
        const int gx = tx + lx, gy = ty + ly, gz = tz + lz;  // the element in the box
        const double *C = coef + 21 * (gx + (int64_t)p.nx * (gy + (int64_t)p.ny * gz));
        // cofactor rows, determinant, and weight over the determinant, at the node
        const double r = xw[2 * a], s = xw[2 * b], z = xw[2 * c], w = xw[2 * a + 1] * xw[2 * b + 1] * xw[2 * c + 1];
        double xr[3], xs[3], xt[3], cr[3], cs[3], ct[3];
        for (int i = 0; i < 3; ++i) {
            xr[i] = C[i] + s * C[9 + i] + z * (C[12 + i] + s * C[18 + i]);
            xs[i] = C[3 + i] + r * C[9 + i] + z * (C[15 + i] + r * C[18 + i]);
            xt[i] = C[6 + i] + r * C[12 + i] + s * (C[15 + i] + r * C[18 + i]);
        }
        for (int i = 0; i < 3; ++i) {
            const int j = (i + 1) % 3, k = (i + 2) % 3;
            cr[i] = xs[j] * xt[k] - xs[k] * xt[j];
            cs[i] = xt[j] * xr[k] - xt[k] * xr[j];
            ct[i] = xr[j] * xs[k] - xr[k] * xs[j];
        }
        const double J = xt[0] * ct[0] + xt[1] * ct[1] + xt[2] * ct[2], k = w / J;
        Gr[t] = k * dot3(cr, cr);
        Gs[t] = k * dot3(cs, cs);
        Gt[t] = k * dot3(ct, ct);
        double mass = w * J;
        if (p.invdeg) {
            mass = 1.0;
            if ((a == 0 && gx > 0) || (a == N && gx < p.nx - 1)) mass *= 0.5;
            if ((b == 0 && gy > 0) || (b == N && gy < p.ny - 1)) mass *= 0.5;
            if ((c == 0 && gz > 0) || (c == N && gz < p.nz - 1)) mass *= 0.5;
        }
        const double Daa = Dm[a * n1 + a], Dbb = Dm[b * n1 + b], Dcc = Dm[c * n1 + c];
        sum[q] = 2.0 * k * (Daa * Dbb * dot3(cr, cs) + Daa * Dcc * dot3(cr, ct) + Dbb * Dcc * dot3(cs, ct)) + lambda * mass;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < per; ++q) {
        const int t = threadIdx.x + q * threads;
        if (t >= nn) continue;
        const int n = epb == 1 ? t : t % np3, a = n % n1, b = (n / n1) % n1, c = n / np2;
        double s = 0.0;
        for (int m = 0; m < n1; ++m) {
            s += D2[m * n1 + a] * Gr[t + (m - a)];
            s += D2[m * n1 + b] * Gs[t + (m - b) * n1];
            s += D2[m * n1 + c] * Gt[t + (m - c) * np2];
        }
        sum[q] += s;
    }
    __syncthreads();  // every line has been read
#pragma unroll
    for (int q = 0; q < per; ++q) {
        const int t = threadIdx.x + q * threads;
        if (t < nn) Gr[t] = sum[q];
    }
    __syncthreads();
    const int wx = ex * N + 1, wy = ey * N + 1, wz = ez * N + 1;
    for (int t = threadIdx.x; t < wx * wy * wz; t += threads) {
        const int row = t / wx, i = t - row * wx, k = row / wy, j = row - k * wy;
        // the elements of the tile that have the node: up to two in each direction
        const int x1 = min(i / N, ex - 1), y1 = min(j / N, ey - 1), z1 = min(k / N, ez - 1);
        const int x0 = i > 0 && i == x1 * N ? x1 - 1 : x1, y0 = j > 0 && j == y1 * N ? y1 - 1 : y1,
                  z0 = k > 0 && k == z1 * N ? z1 - 1 : z1;
        double v = 0.0;
        for (int z = z0; z <= z1; ++z)
            for (int y = y0; y <= y1; ++y)
                for (int x = x0; x <= x1; ++x)
                    v += Gr[(x + ex * (y + ey * z)) * np3 + (i - x * N) + n1 * ((j - y * N) + n1 * (k - z * N))];
        const int I = tx * N + i, J = ty * N + j, K = tz * N + k;
        if (i == wx - 1 && at.x < p.ntx - 1)
            halo[p.hx_at(at.x, at.y, at.z, k, j)] = v;
        else if (j == wy - 1 && at.y < p.nty - 1)
            halo[p.hy_at(at.y, at.z, k, I)] = v;
        else if (k == wz - 1 && at.z < p.ntz - 1)
            halo[p.hz_at(at.z, J, I)] = v;
        else if (!(p.mask && (I == 0 || J == 0 || K == 0 || I == p.gx - 1 || J == p.gy - 1 || K == p.gz - 1)))
            diag[p.off + I + (int64_t)p.sx * J + (int64_t)p.sxy * K] = v;
    }
}

__global__ __launch_bounds__(256) void invert_kernel(int64_t n, double *__restrict__ v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v[i] = 1.0 / v[i];
}

inline unsigned blocks_for(int64_t n, int threads) { return static_cast<unsigned>((n + threads - 1) / threads); }

}  // namespace

hb_status launch_rhs(int64_t n, uint64_t seed, double *b, hipStream_t s)
{
    if (n == 0) return HB_OK;
    const int threads = 256;
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>(blocks_for(n, threads), 8192));
    rhs_kernel<<<grid, threads, 0, s>>>(n, sm64(seed, 0), b);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

namespace {

// The vertices of the mesh, into V.
void enqueue_vertices(const hb_mesh_desc &d, double *V, hipStream_t s)
{
    const int64_t nv = (int64_t)(d.nx + 1) * (d.ny + 1) * (d.nz + 1);
    vertex_kernel<<<blocks_for(nv, 256), 256, 0, s>>>(d.nx, d.ny, d.nz, d.jitter, sm64(d.seed, 1), sm64(d.seed, 2),
                                                      sm64(d.seed, 3), V);
}

}  // namespace

// What the operator reads: one allocation, with the tables (layout: struct Line in
// ax_impl.h) copied in one piece, the elements' maps, and a halo, whose place first holds
// the vertices.  One wait in all (for the Jacobian's check).
hb_status build_mesh(hb_mesh_s *m, hipStream_t s)
{
    const hb_mesh_desc &d = m->desc;
    const int N = m->N, n1 = N + 1, h = n1 / 2;
    const bool fp32 = (d.flags & HB_MESH_FP32) != 0, mask = (d.flags & HB_MESH_DIRICHLET) != 0;
    size_t halo = 0;
    for (int v = 0; v < 2; ++v) {
        m->plan[v] = plan_tiles(N, d.nx, d.ny, d.nz, mask, d.mass == HB_MASS_INVDEG, variant_epb(N, v));
        halo = std::max<size_t>(halo, m->plan[v].halo);
    }
    m->halo_len = halo;
    std::vector<double> tab;
    for (int tr = 0; tr < 2; ++tr) {
        auto D = [&](int i, int j) { return tr ? m->h_D[j * n1 + i] : m->h_D[i * n1 + j]; };
        for (int i = 0; i < h; ++i) {
            for (int j = 0; j < h; ++j) tab.push_back(0.5 * (D(i, j) - D(i, N - j)));
            for (int j = 0; j < h; ++j) tab.push_back(0.5 * (D(i, j) + D(i, N - j)));
            if (n1 % 2) {
                tab.push_back(D(i, h));
                tab.push_back(D(h, i));
            }
        }
    }
    const size_t nt = tab.size(), nv = (size_t)(d.nx + 1) * (d.ny + 1) * (d.nz + 1);
    // the tables, in a multiple of 256 bytes each: tab, xw, D, a flag (zero), tab32
    size_t bytes = 0;
    auto place = [&](size_t b) {
        const size_t at = bytes;
        bytes += (b + 255) / 256 * 256;
        return at;
    };
    const size_t at_tab = place(8 * nt), at_xw = place(16 * n1), at_D = place(8 * n1 * n1), at_bad = place(sizeof(int)),
                 at_tab32 = place(4 * nt), tables = bytes;
    const size_t at_coef = place(sizeof(double) * 21 * m->E), at_halo = place(sizeof(double) * halo);
    bytes = std::max(bytes, at_halo + sizeof(double) * 3 * nv);
    hb_status st;
    if ((st = dev_alloc(&m->mem, bytes, &m->device_bytes))) return st;
    std::vector<unsigned char> host(tables, 0);
    std::memcpy(host.data() + at_tab, tab.data(), 8 * nt);
    for (int i = 0; i < n1; ++i) {
        std::memcpy(host.data() + at_xw + 16 * i, &m->h_xi[i], 8);
        std::memcpy(host.data() + at_xw + 16 * i + 8, &m->h_w[i], 8);
    }
    std::memcpy(host.data() + at_D, m->h_D, 8 * n1 * n1);
    const std::vector<float> tab32(tab.begin(), tab.end());  // rounded to nearest
    std::memcpy(host.data() + at_tab32, tab32.data(), 4 * nt);
    auto f64 = [&](size_t at) { return reinterpret_cast<double *>(m->mem + at); };
    m->tab = f64(at_tab);
    m->xw = f64(at_xw);
    m->D = f64(at_D);
    m->coef = f64(at_coef);
    m->own_halo = f64(at_halo);
    m->call_halo.resize(1);
    m->call_halo[0].mem = m->own_halo;
    if (fp32) m->tab32 = reinterpret_cast<float *>(m->mem + at_tab32);
    int *const bad = reinterpret_cast<int *>(m->mem + at_bad);
    double *const V = m->own_halo;
    int h_bad = 0;
    hipError_t e = hipMemcpyAsync(m->mem, host.data(), tables, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        enqueue_vertices(d, V, s);
        coef_kernel<<<blocks_for(m->E, 256), 256, 0, s>>>(d.nx, d.ny, d.nz, V, m->coef);
        geometry_kernel<false><<<blocks_for(m->NL, 256), 256, 0, s>>>(d.nx, d.ny, d.nz, N, 0, m->E, V, m->xw, 0, 0,
                                                                      nullptr, nullptr, bad);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&h_bad, bad, sizeof(int), hipMemcpyDeviceToHost, s);
    const hipError_t w = hipStreamSynchronize(s);  // also on an error: the host tables go out of scope
    if (e != hipSuccess || w != hipSuccess) return hip_fail(e != hipSuccess ? e : w, "hb_mesh_create: setup");
    if (h_bad) return fail(HB_ERR_INVALID_ARG, "hb_mesh_create: non-positive Jacobian (jitter too large?)");
    return HB_OK;
}

// Z and the geometric factors, computed and copied out by pieces of elements.
hb_status export_geometry(const hb_mesh_s *m, double *host_geo, int32_t *host_map)
{
    const hb_mesh_desc &d = m->desc;
    const int64_t np3 = (int64_t)(m->N + 1) * (m->N + 1) * (m->N + 1);
    const int64_t piece = std::min<int64_t>(m->E, std::max<int64_t>(1, (int64_t{1} << 21) / np3));
    const size_t nv = (size_t)(d.nx + 1) * (d.ny + 1) * (d.nz + 1);
    unsigned char *mem = nullptr;
    const size_t geo_b = sizeof(double) * kGeo * piece * np3, V_b = sizeof(double) * 3 * nv;
    if (hipMalloc(&mem, geo_b + V_b + sizeof(int32_t) * (piece * np3 + 1)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(HB_ERR_OUT_OF_MEMORY, "hb_mesh_export: device allocation failed");
    }
    double *geo = reinterpret_cast<double *>(mem), *V = reinterpret_cast<double *>(mem + geo_b);
    int32_t *map = reinterpret_cast<int32_t *>(mem + geo_b + V_b), *bad = map + piece * np3;
    enqueue_vertices(d, V, nullptr);
    hipError_t e = hipGetLastError();
    for (int64_t e0 = 0; e0 < m->E && e == hipSuccess; e0 += piece) {
        const int64_t ne = std::min(piece, m->E - e0);
        geometry_kernel<true><<<blocks_for(ne * np3, 256), 256>>>(d.nx, d.ny, d.nz, m->N, e0, ne, V, m->xw,
                                                                  d.mass == HB_MASS_INVDEG,
                                                                  (d.flags & HB_MESH_DIRICHLET) != 0, map, geo, bad);
        e = hipGetLastError();
        if (e == hipSuccess && host_geo)
            e = hipMemcpy(host_geo + e0 * np3 * kGeo, geo, sizeof(double) * kGeo * ne * np3, hipMemcpyDeviceToHost);
        if (e == hipSuccess && host_map)
            e = hipMemcpy(host_map + e0 * np3, map, sizeof(int32_t) * ne * np3, hipMemcpyDeviceToHost);
    }
    (void)hipFree(mem);
    return e == hipSuccess ? HB_OK : hip_fail(e, "hb_mesh_export");
}

hb_status launch_jacobi_inverse(const hb_mesh_s *m, double lambda, double *inv, double *halo, hipStream_t s)
{
    if (m->NG == 0) return HB_OK;
    // small tiles where the large ones are fewer than the compute units (4^3 N = 7: 16 us
    // with the large, 10 with the small)
    const int n2 = (m->N + 1) * (m->N + 1), v = n2 <= 64 && m->plan[0].tiles() < kSmallLaunch ? 1 : 0;
    const TilePlan &p = m->plan[v];
    const unsigned grid = static_cast<unsigned>(p.tiles());
    const size_t lds = sizeof(double) * (3 * diag_elements(m->N, v) * n2 * (m->N + 1) + n2);
    auto launch = [&](auto NN, auto VV) {
        constexpr int N = decltype(NN)::value, V = decltype(VV)::value;
        jacobi_diag_kernel<N, V><<<grid, diag_threads(N, V), lds, s>>>(p, m->coef, m->xw, m->D, lambda, inv, halo);
    };
    auto pick = [&](auto NN) {
        if constexpr (decltype(NN)::value <= 7)
            if (v == 1) return launch(NN, std::integral_constant<int, 1>{});
        launch(NN, std::integral_constant<int, 0>{});
    };
    switch (m->N) {
#define HB_DIAG(n) \
    case n: pick(std::integral_constant<int, n>{}); break;
        HB_DIAG(1) HB_DIAG(2) HB_DIAG(3) HB_DIAG(4) HB_DIAG(5) HB_DIAG(6) HB_DIAG(7) HB_DIAG(8)
        HB_DIAG(9) HB_DIAG(10) HB_DIAG(11) HB_DIAG(12) HB_DIAG(13) HB_DIAG(14) HB_DIAG(15)
#undef HB_DIAG
    default: return fail(HB_ERR_INVALID_ARG, "unsupported degree N");
    }
    HB_HIP(hipGetLastError());
    const hb_status st = launch_halo_add(p, halo, inv, s);
    if (st) return st;
    invert_kernel<<<blocks_for(m->NG, 512), 256, 0, s>>>(m->NG, inv);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

}  // namespace hb
