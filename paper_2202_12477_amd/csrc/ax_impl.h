// The fused assembled screened-Poisson operator y = Z^T (S_L + lambda C) Z x
// (eq. poisson and eq. stiffness; the fused gather of the Poisson Operator
// section, with the Z^T assembly in the same kernel).
//
// Nothing about the mesh is streamed: the map Z of a box is index arithmetic,
// and the geometric factors are recomputed at every node from the element's
// trilinear map (21 doubles per element), so the kernel reads x once and writes
// y once.  What bounds it is then FP64 arithmetic and LDS, and both are cut by
// the line form of the contractions:
//   - a thread owns one (a,b) column of one element (its nodes along t), one
//     r line and one s line.  Each derivative is one (N+1)x(N+1) product on a
//     whole line in registers, with D's entries in scalar registers, and data
//     changes hands through LDS: 15 LDS accesses per node instead of the
//     4(N+1) + 3 of reading every product's operand from an LDS slice;
//   - D is centro-antisymmetric (D[i][j] = -D[N-i][N-j]), so a line's product
//     splits into the products of its even and odd parts with half-size
//     matrices: (N+1)^2/2 + 2(N+1) operations instead of (N+1)^2;
//   - along a column the map's Jacobian columns are linear in t, so the cofactor
//     rows and the determinant are polynomials in t whose coefficients are
//     formed once per column.  With c_d the rows of the cofactor matrix and J
//     the determinant, f_d = w/J c_d . (c_r q_r + c_s q_s + c_t q_t).
// Outputs go to their owners with plain stores and to the halo (tile.h); no atomics
// and no vector to clear first.
//
// y = A x, complete, FP64, against the form this replaced (streamed map and factors,
// 60 bytes per node; atomic assembly into a cleared vector): 32^3 N = 7 237 -> 113 us,
// 61x83x47 N = 2 masked 94 -> 62 us, 16^3 N = 15 328 -> 130 us; FP32 26^3 N = 9 188 ->
// 128 us.  Bounds at 32^3 N = 7 (102 us without the halo's addition): about 100 FP64
// and 40 other vector instructions per node keep the vector units 58% busy (the
// card's FP64 rate would allow 56 us), LDS is 47% busy, and three waves per SIMD do
// not hide the rest of the phases' latency.  Measured on the way, same kernel: atomics
// cost 50-65 us more than plain stores; assembling through merged rows in LDS 22 us
// more than by columns; D read again from memory-cached scalars at each use 7 us.
//
// T is the arithmetic type of the contractions: double (the method's FP64
// operator) or float (the FP32 operator of the mixed-precision solver: x
// rounded to FP32 on load, FP32 contractions and output; the geometric factors
// are formed and applied in FP64, so they carry no more error than stored
// factors rounded once to FP32).  x is FP64 in both.
#pragma once

#include <type_traits>

#include "common.h"
#include "reduce.h"
#include "tile.h"

namespace hb {

// Pointers into device (global) memory.  The tile routine takes them in the
// global address space explicitly: callers that read pointers from a table in
// memory would otherwise hand the compiler generic pointers, and every access
// would become a flat access (which also waits on the LDS counter).
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
// Read-only data at uniform positions: scalar loads.
template <typename T>
using cptr = const __attribute__((address_space(4))) T *;

template <typename T>
__device__ inline gptr<T> to_global(T *p)
{
    return (gptr<T>)p;
}
template <typename T>
__device__ inline cptr<T> to_const(const T *p)
{
    return (cptr<T>)p;
}

// The tables of one degree, one array per precision (build_operator fills it): the
// half matrices of D, P[i][j] = (D[i][j] - D[i][N-j])/2 and M[i][j] =
// (D[i][j] + D[i][N-j])/2 for i, j < h, then those of D^T.  Row i holds P[i][.] and
// M[i][.] next to each other, and for an odd number of nodes the middle column's
// and middle row's entries D[i][h] and D[h][i] after them.
template <int N>
struct Line {
    static constexpr int n1 = N + 1, np2 = n1 * n1, np3 = np2 * n1, h = n1 / 2;
    static constexpr bool odd = (n1 & 1) != 0;
    static constexpr int row = 2 * h + (odd ? 2 : 0), table = h * row;  // entries of a row, of a matrix
    // LDS strides of an element's (c, b, a) array: P1 of b, P2 of c.  r lines are
    // read along a at a stride of P1 between lanes: an odd stride, or for even
    // N+1 an odd number of 16-byte units (lines are read 16 bytes at a time).
    static constexpr int P1 = odd ? n1 : (((n1 / 2) & 1) ? n1 : n1 + 2);
    static constexpr int P2 = P1 * n1 + (N == 7 ? 8 : 0);
    static constexpr int vol = P2 * n1;
};

// Elements and threads of a workgroup.  Variant 0: 256 threads (or one element,
// from N = 11); variant 1, where an element fits a wave (N <= 7): one wave.
template <int N, int V>
struct Shape {
    static constexpr int np2 = Line<N>::np2;
    static constexpr int target = V == 1 && np2 <= 64 ? 64 : 256;
    static constexpr int epb = target / np2 > 0 ? target / np2 : 1;
    static constexpr int threads = (epb * np2 + 63) / 64 * 64;
    static constexpr int lds = 2 * epb * Line<N>::vol;  // LDS entries of a tile: two arrays per element
};

// Materialise a value here; with step(), which memory operations and the
// scheduler do not cross, it keeps the phases of a tile apart (interleaved, their
// operands together would take twice the registers).
template <typename T>
__device__ inline void pin(T &v)
{
    asm volatile("" : "+v"(v));
}
__device__ inline void step()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// A pointer the compiler cannot identify with earlier ones, so that what is read
// through it is read again rather than kept in scalar registers across phases.
template <typename P>
__device__ inline P opaque(P p)
{
    asm volatile("" : "+s"(p));
    return p;
}
// Scalar values wanted here: their loads are issued before this point and waited
// for at it, and they are kept, not loaded again at each use.
template <typename T, int K>
__device__ inline void arrive(T (&v)[K])
{
#pragma unroll
    for (int i = 0; i < K; ++i) asm volatile("" : "+s"(v[i]));
}

// The half matrices of one product.  Up to N = 7 they fit the scalar registers and
// are read whole, ahead of the phase that uses them; above, row by row, each row
// while the one before it is used.
template <int N, typename T>
struct Rows {
    static constexpr bool whole = N <= 7;
    static constexpr int K = whole ? Line<N>::table : Line<N>::row;
    T v[K];
    cptr<T> from;
    __device__ __attribute__((always_inline)) inline void fetch(cptr<T> tab)
    {
        from = opaque(tab);
#pragma unroll
        for (int i = 0; i < K; ++i) v[i] = from[i];
    }
};

// u <- D u (or D^T u: the other table) on one line, by its even and odd parts.
template <int N, typename T>
__device__ __attribute__((always_inline)) inline void line_apply(Rows<N, T> &rows, T (&u)[N + 1])
{
    using L = Line<N>;
    constexpr int h = L::h;
    T s[h], d[h];
#pragma unroll
    for (int j = 0; j < h; ++j) {
        s[j] = u[j] + u[N - j];
        d[j] = u[j] - u[N - j];
    }
    const T um = u[h];
    T mid = 0;
    T next[Rows<N, T>::whole ? 1 : L::row];
#pragma unroll
    for (int i = 0; i < h; ++i) {
        const T *r = rows.v;
        if constexpr (Rows<N, T>::whole) {
            r += i * L::row;
        } else {
            if (i + 1 < h) {
                const auto from = opaque(rows.from);
#pragma unroll
                for (int k = 0; k < L::row; ++k) next[k] = from[(i + 1) * L::row + k];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        T even = 0, odd = 0;
#pragma unroll
        for (int j = 0; j < h; ++j) {
            even += r[j] * d[j];
            odd += r[h + j] * s[j];
        }
        if constexpr (L::odd) {
            odd += r[2 * h] * um;
            mid += r[2 * h + 1] * d[i];
        }
        u[i] = even + odd;
        u[N - i] = even - odd;
        if constexpr (!Rows<N, T>::whole) {
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < h) {
#pragma unroll
                for (int k = 0; k < L::row; ++k) rows.v[k] = next[k];
            }
        }
    }
    if constexpr (L::odd) u[h] = mid;
}

// lambda as the operator of type T applies it: rounded to FP32 in the FP32 one.
template <typename T>
__host__ __device__ inline double operator_lambda(double lambda)
{
    return static_cast<double>(static_cast<T>(lambda));
}

// 1/x for positive normal x: the hardware estimate and two Newton steps.
__device__ inline double reciprocal(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

__device__ inline void cross(const double *p, const double *q, double *o)
{
    o[0] = p[1] * q[2] - p[2] * q[1];
    o[1] = p[2] * q[0] - p[0] * q[2];
    o[2] = p[0] * q[1] - p[1] * q[0];
}

// Cofactor rows and determinant along the column at (r, s) of an element, as
// polynomials in t.  The element's map is x = sum C_ijk r^i s^j t^k over i, j, k
// in {0, 1}; C holds C_100, C_010, C_001, C_110, C_101, C_011, C_111.  Then
// x_r = R0 + R1 t, x_s = S0 + S1 t and x_t = Q is constant along the column, so
// c_r = x_s x x_t and c_s = x_t x x_r are linear in t, c_t = x_r x x_s and
// J = x_t . c_t quadratic.
struct Column {
    double A0[3], A1[3], B0[3], B1[3], T0[3], T1[3], T2[3], J0, J1, J2;
    __device__ __attribute__((always_inline)) inline Column(const double (&C)[21], double r, double s)
    {
        double R0[3], R1[3], S0[3], S1[3], Q[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            R0[i] = C[i] + s * C[9 + i];
            R1[i] = C[12 + i] + s * C[18 + i];
            S0[i] = C[3 + i] + r * C[9 + i];
            S1[i] = C[15 + i] + r * C[18 + i];
            Q[i] = C[6 + i] + s * C[15 + i] + r * R1[i];
        }
        cross(S0, Q, A0);
        cross(S1, Q, A1);
        cross(Q, R0, B0);
        cross(Q, R1, B1);
        cross(R0, S0, T0);
        cross(R1, S1, T2);
        cross(R0, S1, T1);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int j = (i + 1) % 3, k = (i + 2) % 3;
            T1[i] += R1[j] * S0[k] - R1[k] * S0[j];
        }
        J0 = Q[0] * T0[0] + Q[1] * T0[1] + Q[2] * T0[2];
        J1 = Q[0] * T1[0] + Q[1] * T1[1] + Q[2] * T1[2];
        J2 = Q[0] * T2[0] + Q[1] * T2[1] + Q[2] * T2[2];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            pin(A0[i]);
            pin(A1[i]);
            pin(B0[i]);
            pin(B1[i]);
            pin(T0[i]);
            pin(T1[i]);
            pin(T2[i]);
        }
        pin(J0);
        pin(J1);
        pin(J2);
    }
    // cofactor rows and determinant at t = z
    __device__ __attribute__((always_inline)) inline double at(double z, double *cr, double *cs, double *ct) const
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            cr[i] = A0[i] + z * A1[i];
            cs[i] = B0[i] + z * B1[i];
            ct[i] = T0[i] + z * (T1[i] + z * T2[i]);
        }
        return J0 + z * (J1 + z * J2);
    }
};

// A tile's place in the tile grid.
struct TilePlace {
    int32_t x, y, z;
};

__device__ inline TilePlace tile_place(const TilePlan &p, uint32_t tile)
{
    const uint32_t row = p.tx(tile), z = p.ty(row);
    return TilePlace{static_cast<int32_t>(tile - row * p.tx.d), static_cast<int32_t>(row - z * p.ty.d),
                     static_cast<int32_t>(z)};
}

// One tile: y = A x (ADD: y += A x) on the DOFs it owns, the sums of the others into
// the halo.  With DOT, returns (in thread 0) the tile's share of x . A x, summed
// at the nodes as q_r f_r + q_s f_s + q_t f_t + lambda c q^2.  Every thread of the
// workgroup must call it; t: its number among the tile's threads (several tiles may
// share a workgroup and its barriers; live: this one is real, the others compute
// on a valid place and store nothing).  plan: in constant memory, read again by each phase (held
// in scalar registers throughout, it would crowd out D's entries).
// lds: Shape::lds entries of LDS, 16-byte aligned; red: threads / 64 entries (DOT).
// st: null, or the state of a solve whose stop makes the call do nothing.
// (Always inlined: the single-problem, batched and persistent kernels call it.)
template <int N, int V, typename T, bool DOT, bool MASK, bool ADD>
__device__ __attribute__((always_inline)) inline double ax_tile(int t, bool live, T *lds, double *red,
                                                                cptr<TilePlan> plan, TilePlace at,
                                                                gptr<const double> coef, cptr<T> tab,
                                                                cptr<double> tab64, cptr<double> xw, double lambda,
                                                                gptr<const double> x, gptr<T> y, gptr<T> halo,
                                                                cptr<CgState> st)
{
    using L = Line<N>;
    using S = Shape<N, V>;
    constexpr int n1 = L::n1, np2 = L::np2, P1 = L::P1, P2 = L::P2, epb = S::epb;
    // elements that do not straddle waves need no workgroup barrier between phases
    constexpr bool wave_sync = 64 % np2 == 0;
    auto sync = [] {
        if constexpr (wave_sync) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else {
            __syncthreads();
        }
    };
    // spare lanes mirror a column and store nothing
    const bool used = live && (epb * np2 == S::threads || t < epb * np2);
    int el = used ? t / np2 : 0;
    if constexpr (np2 == 64) el = __builtin_amdgcn_readfirstlane(el);
    const int ab = used ? t - el * np2 : 0;
    const int a = ab % n1, b = ab / n1;
    // the element's place: in the tile (the last tile of a direction may be short)
    // and in the box
    int lx = 0, ly = 0, lz = 0, nlx, nly, nlz;
    bool active = used;
    int I, J, K0, e, sxy, invdeg;
    T q[n1];
    {
        const auto p = opaque(plan);
        nlx = min(p->kx, p->nx - at.x * p->kx);
        nly = min(p->ky, p->ny - at.y * p->ky);
        nlz = min(p->kz, p->nz - at.z * p->kz);
        if constexpr (epb > 1) {
            const FastDiv dx{p->ex.d, p->ex.m, p->ex.s}, dxy{p->exy.d, p->exy.m, p->exy.s};
            lz = dxy(el);
            const int lxy = el - lz * static_cast<int>(dxy.d);
            ly = dx(lxy);
            lx = lxy - ly * static_cast<int>(dx.d);
            const bool in = lx < nlx && ly < nly && lz < nlz;
            active = used && in;
            if (!in) lx = ly = lz = 0;  // a valid element, discarded
        }
        const int ex = at.x * p->kx + lx, ey = at.y * p->ky + ly, ez = at.z * p->kz + lz;
        e = ex + p->nx * (ey + p->ny * ez);
        I = ex * N + a;
        J = ey * N + b;
        K0 = ez * N;
        sxy = p->sxy;
        invdeg = p->invdeg;
        // gather through Z: the (a,b) column of the element
        const int base = p->off + I + p->sx * J + sxy * K0;
        if constexpr (MASK) {
            const bool col = I > 0 && I < p->gx - 1 && J > 0 && J < p->gy - 1;
            const bool on0 = col && K0 > 0, on1 = col && K0 + N < p->gz - 1;
#pragma unroll
            for (int c = 0; c < n1; ++c) {
                const bool on = c == 0 ? on0 : c == N ? on1 : col;
                const double v = x[on ? base + c * sxy : 0];
                q[c] = on ? static_cast<T>(v) : T(0);
            }
        } else {
#pragma unroll
            for (int c = 0; c < n1; ++c) q[c] = static_cast<T>(x[base + c * sxy]);
        }
    }
    // and what the metric terms need of the element, ahead of their use
    double C[21];
    const auto xv = (gptr<const double>)(const double *)xw;
    const double r_a = xv[2 * a], w_a = xv[2 * a + 1], s_b = xv[2 * b], w_b = xv[2 * b + 1];
    {
        const gptr<const double> Ce = coef + static_cast<uint32_t>(e) * 21u;
#pragma unroll
        for (int i = 0; i < 21; ++i) C[i] = Ce[i];
    }
    // CG: stopped, or stopping at the next alpha step (which reads no partials)
    if constexpr (DOT) {
        if (st && (st->done | st->pending)) return 0.0;
    }
    Rows<N, T> D;
    D.fetch(tab);
    T *const s0 = lds + el * L::vol, *const s1 = s0 + epb * L::vol;
    T *const col0 = s0 + b * P1 + a, *const col1 = s1 + b * P1 + a;    // the column (a,b): + c P2
    T *const rl0 = s0 + b * P2 + a * P1, *const rl1 = rl0 + epb * L::vol;  // the r line b' = a, c' = b: + m
    T *const sl0 = s0 + b * P2 + a;                                    // the s line a' = a, c' = b: + m P1
    if (used) {
#pragma unroll
        for (int c = 0; c < n1; ++c) col0[c * P2] = q[c];
    }
    sync();
    step();
    {
        T u[n1];
#pragma unroll
        for (int m = 0; m < n1; ++m) u[m] = rl0[m];
        if constexpr (D.whole) arrive(D.v);
        line_apply(D, u);
        if constexpr (!D.whole) D.fetch(tab);
        if (used) {
#pragma unroll
            for (int m = 0; m < n1; ++m) rl1[m] = u[m];
        }
    }
    step();
    {
        T u[n1];
#pragma unroll
        for (int m = 0; m < n1; ++m) u[m] = sl0[m * P1];
        sync();  // every r line has been read
        line_apply(D, u);
        if (used) {
#pragma unroll
            for (int m = 0; m < n1; ++m) sl0[m * P1] = u[m];
        }
    }
    step();
    // t direction: registers only, and FP64 in the FP32 operator too
    double f[n1];
#pragma unroll
    for (int c = 0; c < n1; ++c) f[c] = static_cast<double>(q[c]);
    if constexpr (sizeof(T) == 8) {
        if constexpr (!D.whole) D.fetch(tab);
        line_apply(D, f);
    } else {
        Rows<N, double> D64;
        D64.fetch(tab64);
        if constexpr (D64.whole) arrive(D64.v);
        line_apply(D64, f);
    }
#pragma unroll
    for (int c = 0; c < n1; ++c) pin(f[c]);
    step();
    double dot = 0.0;
    {
        double zw[2 * n1];  // node and weight of each layer
        const auto xs = opaque(xw);
#pragma unroll
        for (int i = 0; i < 2 * n1; ++i) zw[i] = xs[i];
        const double wab = w_a * w_b;
        const Column g(C, r_a, s_b);
        // identity mass: 1 / multiplicity of the node, a power of two
        double mab = 1.0, m0 = 1.0, m1 = 1.0;
        if (invdeg) {
            const auto p = opaque(plan);
            if ((a == 0 && I > 0) || (a == N && I < p->gx - 1)) mab *= 0.5;
            if ((b == 0 && J > 0) || (b == N && J < p->gy - 1)) mab *= 0.5;
            m0 = K0 > 0 ? 0.5 : 1.0;
            m1 = K0 + N < p->gz - 1 ? 0.5 : 1.0;
        }
        sync();
        T nr = col1[0], ns = col0[0];
        arrive(zw);
#pragma unroll
        for (int c = 0; c < n1; ++c) {
            step();
            const double qr = nr, qs = ns, qt = f[c];
            const double z = zw[2 * c], wc = wab * zw[2 * c + 1];
            if (c < N) {  // the next node's, while this one is worked on
                nr = col1[(c + 1) * P2];
                ns = col0[(c + 1) * P2];
            }
            double cr[3], cs[3], ct[3], v[3];
            const double J = g.at(z, cr, cs, ct);
            const double wj = wc * reciprocal(J);
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i] = wj * (cr[i] * qr + cs[i] * qs + ct[i] * qt);
            const double fr = cr[0] * v[0] + cr[1] * v[1] + cr[2] * v[2];
            const double fs = cs[0] * v[0] + cs[1] * v[1] + cs[2] * v[2];
            const double ft = ct[0] * v[0] + ct[1] * v[1] + ct[2] * v[2];
            const double mass = invdeg ? mab * (c == 0 ? m0 : c == N ? m1 : 1.0) : wc * J;
            const double mq = lambda * mass * static_cast<double>(q[c]);
            if constexpr (DOT) {
                dot += (fr * qr + fs * qs) + (ft * qt + mq * static_cast<double>(q[c]));
                pin(dot);
            }
            if (used) {
                col1[c * P2] = static_cast<T>(fr);
                col0[c * P2] = static_cast<T>(fs);
            }
            f[c] = ft;
            q[c] = static_cast<T>(mq);
            pin(f[c]);
            pin(q[c]);
        }
    }
    // DOT: the wave's sum, added up over the waves after the last barrier
    if constexpr (DOT) {
        const double ws = wave_sum(active ? dot : 0.0);
        if (live && (t & 63) == 0) red[t >> 6] = ws;
    }
    constexpr int T1 = L::table;  // the table of D^T
    if constexpr (sizeof(T) == 8) {
        D.fetch(tab + T1);
        step();
        if constexpr (D.whole) arrive(D.v);
        line_apply(D, f);
        if constexpr (!D.whole) D.fetch(tab + T1);
    } else {
        Rows<N, double> D64;
        D64.fetch(tab64 + T1);
        step();
        if constexpr (D64.whole) arrive(D64.v);
        line_apply(D64, f);
        D.fetch(tab + T1);
    }
#pragma unroll
    for (int c = 0; c < n1; ++c) {
        q[c] = static_cast<T>(static_cast<double>(q[c]) + f[c]);
        pin(q[c]);
    }
    sync();
    step();
    {
        T u[n1];
#pragma unroll
        for (int m = 0; m < n1; ++m) u[m] = rl1[m];
        if constexpr (D.whole && sizeof(T) == 4) arrive(D.v);
        line_apply(D, u);
        if constexpr (!D.whole) D.fetch(tab + T1);
        if (used) {
#pragma unroll
            for (int m = 0; m < n1; ++m) rl1[m] = u[m];
        }
    }
    step();
    {
        T u[n1];
#pragma unroll
        for (int m = 0; m < n1; ++m) u[m] = sl0[m * P1];
        line_apply(D, u);
        if (used) {
#pragma unroll
            for (int m = 0; m < n1; ++m) sl0[m * P1] = u[m];
        }
    }
    sync();
    step();
#pragma unroll
    for (int c = 0; c < n1; ++c) q[c] += col0[c * P2] + col1[c * P2];
    // assembly of the tile: a node shared by elements of the tile goes to the
    // element that has it on its first plane, whose column adds the others' copies
    // from LDS in a fixed order; each column then stores its nodes
    const bool upx = lx + 1 < nlx, upy = ly + 1 < nly, upz = lz + 1 < nlz;  // neighbours above in the tile
    if constexpr (epb > 1) {
        const auto p = opaque(plan);
        if (p->kx * p->ky * p->kz > 1) {
            const int ystep = p->kx * L::vol, zstep = p->kx * p->ky * L::vol;
            const bool edge = (a == N && upx) || (b == N && upy);
            if (active) {
#pragma unroll
                for (int c = 0; c < n1; ++c)
                    if (edge || (c == N && upz)) col0[c * P2] = q[c];
            }
            __syncthreads();
            const bool shx = a == 0 && lx > 0, shy = b == 0 && ly > 0, shz = lz > 0;
            if (active && shx) {
                const T *o = col0 + N - L::vol;
#pragma unroll
                for (int c = 0; c < n1; ++c) q[c] += o[c * P2];
            }
            if (active && shy) {
                const T *o = col0 + N * P1 - ystep;
#pragma unroll
                for (int c = 0; c < n1; ++c) q[c] += o[c * P2];
                if (shx) {
                    o += N - L::vol;
#pragma unroll
                    for (int c = 0; c < n1; ++c) q[c] += o[c * P2];
                }
            }
            if (active && shz) {
                const T *o = col0 + N * P2 - zstep;
                q[0] += o[0];
                if (shx) q[0] += o[N - L::vol];
                if (shy) {
                    q[0] += o[N * P1 - ystep];
                    if (shx) q[0] += o[N * P1 - ystep + N - L::vol];
                }
            }
        }
    }
    if (active && !(a == N && upx) && !(b == N && upy)) {
        const auto p = opaque(plan);
        const bool hx = a == N && at.x + 1 < p->ntx, hy = b == N && at.y + 1 < p->nty, hz = at.z + 1 < p->ntz;
        const int kn = lz * N, cz = p->kz * N + 1;
        gptr<T> out;
        int stride;
        bool on = true, on0 = true, on1 = !upz;
        if (hx) {
            out = halo + (p->hx + (((at.x * p->nty + at.y) * p->ntz + at.z) * cz + kn) * (p->ky * N + 1) + ly * N + b);
            stride = p->ky * N + 1;
        } else if (hy) {
            out = halo + (p->hy + ((at.y * p->ntz + at.z) * cz + kn) * p->gx + I);
            stride = p->gx;
        } else {
            out = y + (p->off + I + p->sx * J + sxy * K0);
            stride = sxy;
            if constexpr (MASK) {
                on = I > 0 && I < p->gx - 1 && J > 0 && J < p->gy - 1;
                on0 = K0 > 0;
                on1 = on1 && K0 + N < p->gz - 1;
            }
            if (hz && !upz) {  // the tile's last z plane
                on1 = false;
                halo[(at.z * p->gy + J) * p->gx + I] = q[N];
            }
        }
        if (!MASK || on) {
#pragma unroll
            for (int c = 0; c < n1; ++c) {
                if ((MASK && c == 0 && !on0) || (c == N && !on1)) continue;
                gptr<T> o = out + c * stride;
                if constexpr (ADD) {
                    if (!(hx | hy))
                        *o += q[c];
                    else
                        *o = q[c];
                } else {
                    *o = q[c];
                }
            }
        }
    }
    if constexpr (DOT) {
        if constexpr (S::threads > 64) __syncthreads();
        dot = 0.0;
        if (t == 0) {
#pragma unroll
            for (int i = 0; i < S::threads / 64; ++i) dot += red[i];
        }
    }
    return dot;
}

template <int N, int V, typename T, bool DOT, bool MASK, bool ADD>
__global__ __launch_bounds__((Shape<N, V>::threads)) void ax_kernel(TilePlan p, const double *__restrict__ coef,
                                                                   const T *__restrict__ tab,
                                                                   const double *__restrict__ tab64,
                                                                   const double *__restrict__ xw, double lambda,
                                                                   const double *__restrict__ x, T *__restrict__ y,
                                                                   T *__restrict__ halo, double *__restrict__ partial,
                                                                   const CgState *__restrict__ st)
{
    __shared__ __attribute__((aligned(16))) T lds[Shape<N, V>::lds];
    // p: the kernel's first argument, read from the argument segment
    const auto plan = (cptr<TilePlan>)__builtin_amdgcn_kernarg_segment_ptr();
    const TilePlace at = tile_place(p, walk_tile(p.walk, xcd_remap(blockIdx.x, gridDim.x)));
    __shared__ double red[Shape<N, V>::threads / 64];
    const double d = ax_tile<N, V, T, DOT, MASK, ADD>(threadIdx.x, true, lds, red, plan, at, to_global(coef), to_const(tab), to_const(tab64),
                                                      to_const(xw), lambda, to_global(x), to_global(y),
                                                      to_global(halo), to_const(st));
    if (DOT && threadIdx.x == 0) partial[blockIdx.x] = d;
}

// Values read from a work list or a problem table are the same for the whole
// block; saying so lets the compiler keep them (and everything derived from
// them) in scalar registers.
__device__ inline int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uniform(int64_t v)
{
    const uint64_t u = static_cast<uint64_t>(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}
template <typename P>
__device__ inline P *uniform(P *p)
{
    return reinterpret_cast<P *>(uniform(reinterpret_cast<int64_t>(p)));
}
__device__ inline double uniform(double v)
{
    return __builtin_bit_cast(double, uniform(__builtin_bit_cast(int64_t, v)));
}

// The batched operator: one block per (problem, tile) item of a class's work
// list, with p.Ap fused.  The tables depend only on the degree, so all problems of
// a class share them.
template <int N, int V, typename T, bool MASK>
__global__ __launch_bounds__((Shape<N, V>::threads)) void batch_ax_kernel(const WorkItem *__restrict__ items,
                                                                         const BatchProb *__restrict__ probs,
                                                                         const T *__restrict__ tab,
                                                                         const double *__restrict__ tab64,
                                                                         const double *__restrict__ xw)
{
    __shared__ __attribute__((aligned(16))) T lds[Shape<N, V>::lds];
    const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
    const int32_t prob = uniform(it.prob), tile = uniform(it.idx);
    const BatchProb &P = probs[prob];
    const auto x = to_global(uniform(P.p));
    T *y, *halo;
    if constexpr (sizeof(T) == 4) {
        y = P.Ap32;
        halo = P.halo32;
    } else {
        y = P.Ap;
        halo = P.halo;
    }
    const double lambda = operator_lambda<T>(uniform(P.lambda));
    __shared__ double red[Shape<N, V>::threads / 64];
    const double d = ax_tile<N, V, T, true, MASK, false>(threadIdx.x, true, lds, red, to_const(&P.plan), tile_place(P.plan, tile), to_global(uniform(P.coef)), to_const(tab),
                                                         to_const(tab64), to_const(xw), lambda, x,
                                                         to_global(uniform(y)), to_global(uniform(halo)),
                                                         to_const(uniform(P.st)));
    if (threadIdx.x == 0) to_global(uniform(P.part_ax))[tile] = d;
}

// Run-time variant -> compile-time instantiation.
template <int N, typename F>
decltype(auto) with_variant(int v, F &&f)
{
    if constexpr (Line<N>::np2 <= 64)
        if (v == 1) return f(std::integral_constant<int, 1>{});
    return f(std::integral_constant<int, 0>{});
}

template <int N, typename T, bool MASK>
hb_status launch_ax_n(const hb_mesh_s *m, const T *tab, double lambda, const double *x, T *y, T *halo, bool add,
                      double *partial, CgState *st, hipStream_t s)
{
    const int v = mesh_variant(m, sizeof(T) == 4);
    const TilePlan &p = m->plan[v];
    return with_variant<N>(v, [&](auto VV) -> hb_status {
        constexpr int V = decltype(VV)::value;
        const int grid = p.tiles(), threads = Shape<N, V>::threads;
        const double lam = operator_lambda<T>(lambda);
        if (st)
            ax_kernel<N, V, T, true, MASK, false><<<grid, threads, 0, s>>>(p, m->coef, tab, m->tab, m->xw, lam, x, y, halo,
                                                                           partial, st);
        else if (!add)
            ax_kernel<N, V, T, false, MASK, false><<<grid, threads, 0, s>>>(p, m->coef, tab, m->tab, m->xw, lam, x, y, halo,
                                                                            nullptr, nullptr);
        else if constexpr (sizeof(T) == 8)
            ax_kernel<N, V, T, false, MASK, true><<<grid, threads, 0, s>>>(p, m->coef, tab, m->tab, m->xw, lam, x, y, halo,
                                                                           nullptr, nullptr);
        HB_HIP(hipGetLastError());
        return HB_OK;
    });
}

template <int N, bool MASK>
hb_status launch_batch_ax_n(int v, const void *tab, const double *tab64, const double *xw, bool fp32, const WorkItem *items, int nitems,
                            const BatchProb *probs, hipStream_t s)
{
    if (nitems == 0) return HB_OK;
    return with_variant<N>(v, [&](auto VV) -> hb_status {
        constexpr int V = decltype(VV)::value;
        if (fp32)
            batch_ax_kernel<N, V, float, MASK><<<nitems, Shape<N, V>::threads, 0, s>>>(
                items, probs, static_cast<const float *>(tab), tab64, xw);
        else
            batch_ax_kernel<N, V, double, MASK><<<nitems, Shape<N, V>::threads, 0, s>>>(
                items, probs, static_cast<const double *>(tab), tab64, xw);
        HB_HIP(hipGetLastError());
        return HB_OK;
    });
}

}  // namespace hb

// One degree's entry points (FP64 and FP32 operator, batched operator), expanded
// in the per-range translation units so the instantiations compile in parallel;
// the masked (Dirichlet) variants in units of their own.
#define HB_AX_ENTRY(n, suffix, MASK)                                                                             \
    namespace hb {                                                                                               \
    hb_status launch_ax##suffix##n(const hb_mesh_s *m, double l, const double *x, double *y, bool add, double *p, \
                                   CgState *st, hipStream_t s)                                                   \
    {                                                                                                            \
        return launch_ax_n<n, double, MASK>(m, m->tab, l, x, y, m->halo, add, p, st, s);                         \
    }                                                                                                            \
    hb_status launch_ax32##suffix##n(const hb_mesh_s *m, double l, const double *x, float *y, double *p,          \
                                     CgState *st, hipStream_t s)                                                 \
    {                                                                                                            \
        return launch_ax_n<n, float, MASK>(m, m->tab32, l, x, y, m->halo32, false, p, st, s);                    \
    }                                                                                                            \
    hb_status launch_batch_ax##suffix##n(int v, const void *tab, const double *tab64, const double *xw, bool fp32,  \
                                         const WorkItem *it, int ni, const BatchProb *pr, hipStream_t s)         \
    {                                                                                                            \
        return launch_batch_ax_n<n, MASK>(v, tab, tab64, xw, fp32, it, ni, pr, s);                                      \
    }                                                                                                            \
    }
#define HB_AX_INSTANCE(n) HB_AX_ENTRY(n, _, false)
#define HB_AX_INSTANCE_DIRICHLET(n) HB_AX_ENTRY(n, _d_, true)
