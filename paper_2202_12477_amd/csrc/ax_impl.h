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
// 60 bytes per node; atomic assembly into a cleared vector): 32^3 N = 7 237 -> 110 us,
// 61x83x47 N = 2 masked 95 -> 50 us, 16^3 N = 15 328 -> 138 us; FP32 26^3 N = 9 188 ->
// 124 us.  Bounds at 32^3 N = 7 (81 us on x and y of the last call, 88 on others, and the
// halo's addition 24 to 30): 104 FP64 and 20
// other vector instructions per node keep the vector units two thirds busy at the 1.9
// GHz the card holds under this load (the FP64 rate alone would allow 45 us); of a
// wave's 14600 cycles its own arithmetic is 4000, the three waves of a SIMD share the
// rest with the latency of loads (3500), LDS exchanges and stores (1800).  Neither a
// fourth wave (without LDS padding, 109 us), nor persistent workgroups that load the
// next tile's x ahead (109 us), nor element maps through LDS (101 us) hide more of it.
// Measured on the way, same kernel: atomics
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
    // N = 7: of the lanes that an LDS access serves together, a plane of 8 P1 leaves the r
    // lines (16 bytes, 16 lanes: two planes) without conflicts and the s lines (8 bytes, 32
    // lanes: four planes) with two lanes to a bank; 8 entries more, the other way round.  CG
    // is faster with them (32^3 100 iterations 20.28 ms against 20.38, 50^3 Jacobi 95.4
    // against 95.6), y = A x alone without (109 us against 102; repeated on the same vectors
    // 97.6 against 96.8).  At every other degree 8 more are even or cost up to 7% (N = 3).
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
// An LDS address as one register, from which entries at constant offsets are read
// without further arithmetic.
template <typename T>
using lptr = const __attribute__((address_space(3))) T *;
template <typename T>
__device__ inline lptr<T> pinned(const T *p)
{
    lptr<T> l = (lptr<T>)p;
    asm volatile("" : "+v"(l));
    return l;
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
            // N = 12, 14: the middle row's products belong to their rows; gathered at the
            // end they keep every row's entries, through spilled registers (17^3 N = 14
            // 142 us against 132; no gain, or 1% lost, at the other degrees)
            if constexpr (L::odd && N > 11) {
                pin(u[i]);
                pin(u[N - i]);
                pin(mid);
            }
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

// 1/x for positive normal x: the hardware estimate r (good to 2^-23 or better) and
// one step of third order, r (1 + e + e^2) with e = 1 - x r: the same error as two
// Newton steps for one operation less.
__device__ inline double reciprocal(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    const double e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, __builtin_fma(e, e, e), r);
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

// The same from the Jacobian's columns at each node: 13 operations more per node, 50
// fewer per column and 18 registers fewer, which at N = 1 and 2 is a wave per SIMD more.
// 128^3 N = 1 146 us against 161 with the polynomials, 84^3 N = 2 105 against 113 (with
// p.Ap 117, 121); even at N = 3 to 6 and 8, 3% slower at N = 7 and above.
struct Direct {
    double R0[3], R1[3], S0[3], S1[3], Q[3];
    __device__ __attribute__((always_inline)) inline Direct(const double (&C)[21], double r, double s)
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            R0[i] = C[i] + s * C[9 + i];
            R1[i] = C[12 + i] + s * C[18 + i];
            S0[i] = C[3 + i] + r * C[9 + i];
            S1[i] = C[15 + i] + r * C[18 + i];
            Q[i] = C[6 + i] + s * C[15 + i] + r * R1[i];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            pin(R0[i]);
            pin(R1[i]);
            pin(S0[i]);
            pin(S1[i]);
            pin(Q[i]);
        }
    }
    __device__ __attribute__((always_inline)) inline double at(double z, double *cr, double *cs, double *ct) const
    {
        double xr[3], xs[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            xr[i] = R0[i] + z * R1[i];
            xs[i] = S0[i] + z * S1[i];
        }
        cross(xs, Q, cr);
        cross(Q, xr, cs);
        cross(xr, xs, ct);
        return Q[0] * ct[0] + Q[1] * ct[1] + Q[2] * ct[2];
    }
};

// What an operator kernel is launched with.  The tile routine reads these and the plan
// from constant memory, through pointers that the compiler cannot see through, in the
// phase that needs them: as plain kernel arguments all were loaded at the start, crowded
// D's entries out of the scalar registers and travelled through lanes of vector
// registers (64 of 1137 vector instructions of a wave at N = 7, 244 of 1770 at N = 11;
// with them gone 32^3 N = 7 104 -> 99 us, 21^3 N = 11 135 -> 129 us).
template <typename T>
struct AxArgs {
    TilePlan plan;
    const double *coef;          // the elements' trilinear maps
    const T *tab;                // the degree's tables (Line) in T and in FP64
    const double *tab64, *xw;    // xw: node and weight of each layer
    double lambda;
    const double *x;
    T *y, *halo;
    double *partial;             // DOT: one per workgroup
    const CgState *st;
};
template <typename T>
struct AxFromArgs {
    cptr<AxArgs<T>> k;
    __device__ cptr<TilePlan> plan() const { return &opaque(k)->plan; }
    __device__ gptr<const double> coef() const { return to_global(opaque(k)->coef); }
    __device__ cptr<T> tab() const { return to_const(opaque(k)->tab); }
    __device__ cptr<double> tab64() const { return to_const(opaque(k)->tab64); }
    __device__ cptr<double> xw() const { return to_const(opaque(k)->xw); }
    __device__ double lambda() const { return opaque(k)->lambda; }
    __device__ gptr<const double> x() const { return to_global(opaque(k)->x); }
    __device__ gptr<T> y() const { return to_global(opaque(k)->y); }
    __device__ gptr<T> halo() const { return to_global(opaque(k)->halo); }
    __device__ cptr<CgState> st() const { return to_const(opaque(k)->st); }
};
// The same from a problem of a batch.
template <typename T>
struct AxFromBatch {
    cptr<BatchProb> k;
    __device__ cptr<TilePlan> plan() const { return &opaque(k)->plan; }
    __device__ gptr<const double> coef() const { return to_global(opaque(k)->coef); }
    __device__ cptr<T> tab() const
    {
        if constexpr (sizeof(T) == 4)
            return to_const(opaque(k)->tab32);
        else
            return to_const(opaque(k)->tab);
    }
    __device__ cptr<double> tab64() const { return to_const(opaque(k)->tab); }
    __device__ cptr<double> xw() const { return to_const(opaque(k)->xw); }
    __device__ double lambda() const { return operator_lambda<T>(opaque(k)->lambda); }
    __device__ gptr<const double> x() const { return to_global(static_cast<const double *>(opaque(k)->p)); }
    __device__ gptr<T> y() const
    {
        if constexpr (sizeof(T) == 4)
            return to_global(opaque(k)->Ap32);
        else
            return to_global(opaque(k)->Ap);
    }
    __device__ gptr<T> halo() const
    {
        if constexpr (sizeof(T) == 4)
            return to_global(opaque(k)->halo32);
        else
            return to_global(opaque(k)->halo);
    }
    __device__ cptr<CgState> st() const { return to_const(static_cast<const CgState *>(opaque(k)->st)); }
};

// How a tile's sums reach y: y = A x, y += A x, or every one added atomically, those of
// neighbouring tiles too (a kernel of its own: with the choice made at run time the
// addition through the halo took 1 us, 2%, longer).
enum { kAssign = 0, kAdd = 1, kAddDirect = 2 };

// One tile: y = A x (kAdd: y += A x) on the DOFs it owns, the sums of the others into
// the halo (kAddDirect: added to y).  With DOT, returns (in thread 0) the tile's share of x . A x, summed
// at the nodes as q_r f_r + q_s f_s + q_t f_t + lambda c q^2.  Every thread of the
// workgroup must call it.  at: the tile's place (uniform); from: an AxFrom...
// lds: Shape::lds entries of LDS, 16-byte aligned; red: threads / 64 entries (DOT).
// With DOT, nothing is done once the solve's state says that it has stopped.
// (Always inlined: the single-problem, batched and persistent kernels call it.)
template <int N, int V, typename T, bool DOT, bool MASK, int ADD, typename From>
__device__ __attribute__((always_inline)) inline double ax_tile(T *lds, double *red, const From &from, TilePlace at)
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
    const int t = threadIdx.x;
    // spare lanes mirror a column and store nothing
    const bool used = epb * np2 == S::threads || t < epb * np2;
    int el = used ? t / np2 : 0;
    if constexpr (np2 == 64) el = __builtin_amdgcn_readfirstlane(el);
    const int ab = used ? t - el * np2 : 0;
    const int a = ab % n1, b = ab / n1;
    // the element's place: in the tile (the last tile of a direction may be short)
    // and in the box
    int lx = 0, ly = 0, lz = 0;
    bool active = used;
    T q[n1];
    int e;
    bool invdeg;
    {
        const auto p = from.plan();
        const auto x = from.x();
        invdeg = p->invdeg != 0;
        const int tx = at.x * p->kx, ty = at.y * p->ky, tz = at.z * p->kz, sxy = p->sxy;
        if constexpr (epb > 1) {
            const FastDiv dx{p->ex.d, p->ex.m, p->ex.s}, dxy{p->exy.d, p->exy.m, p->exy.s};
            lz = dxy(el);
            const int lxy = el - lz * static_cast<int>(dxy.d);
            ly = dx(lxy);
            lx = lxy - ly * static_cast<int>(dx.d);
            const bool in = lx < min(p->kx, p->nx - tx) && ly < min(p->ky, p->ny - ty) && lz < min(p->kz, p->nz - tz);
            active = used && in;
            if (!in) lx = ly = lz = 0;  // a valid element, discarded
        }
        e = tx + lx + p->nx * (ty + ly + p->ny * (tz + lz));
        int i = lx * N + a, j = ly * N + b;
        const int k = lz * N;
        const int I = tx * N + i, J = ty * N + j, K0 = tz * N + k;
        // gather through Z: the (a,b) column of the element, each node as the tile's
        // first node of its layer (uniform) plus one byte offset, of 32 bits where the
        // tile's reach allows: then an address takes no vector arithmetic
        const auto xt = x + (p->off + static_cast<int64_t>(tx) * N + static_cast<int64_t>(p->sx) * (ty * N) +
                             static_cast<int64_t>(sxy) * (tz * N));
        auto load = [&](int c, auto bytes) {
            return *(gptr<const double>)((gptr<const char>)(xt + static_cast<int64_t>(c) * sxy) + bytes);
        };
        if constexpr (MASK) {
            // a node without a DOF reads its neighbour inside the box, and is zero
            const bool col = I > 0 && I < p->gx - 1 && J > 0 && J < p->gy - 1;
            i += (I == 0) - (I == p->gx - 1);
            j += (J == 0) - (J == p->gy - 1);
            const bool low = K0 == 0, high = K0 + N == p->gz - 1;
            auto column = [&](auto o, auto layer) {
#pragma unroll
                for (int c = 0; c < n1; ++c) {
                    const double v = c == 0   ? load(0, low ? o + layer : o)
                                     : c == N ? load(N - 1, high ? o : o + layer)
                                              : load(c, o);
                    const bool on = c == 0 ? col && !low : c == N ? col && !high : col;
                    q[c] = on ? static_cast<T>(v) : T(0);
                }
            };
            const uint32_t o = static_cast<uint32_t>(i + p->sx * j + sxy * k), layer = static_cast<uint32_t>(sxy);
            if (p->wide)
                column(uint64_t{o} * 8, uint64_t{layer} * 8);
            else
                column(o * 8, layer * 8);
        } else {
            auto column = [&](auto o) {
#pragma unroll
                for (int c = 0; c < n1; ++c) q[c] = static_cast<T>(load(c, o));
            };
            const uint32_t o = static_cast<uint32_t>(i + p->sx * j + sxy * k);
            if (p->wide)
                column(uint64_t{o} * 8);
            else
                column(o * 8);
        }
    }
    // and what the metric terms need of the element, ahead of their use
    double C[21];
    const auto xv = (gptr<const double>)(const double *)from.xw();
    const double r_a = xv[2 * a], w_a = xv[2 * a + 1], s_b = xv[2 * b], w_b = xv[2 * b + 1];
    {
        const gptr<const double> Ce = from.coef() + static_cast<uint64_t>(static_cast<uint32_t>(e)) * 21u;
#pragma unroll
        for (int i = 0; i < 21; ++i) C[i] = Ce[i];
    }
    // CG: stopped, or stopping at the next alpha step (which reads no partials)
    if constexpr (DOT) {
        const auto st = from.st();
        if (st->done | st->pending) return 0.0;
    }
    const auto tab = from.tab();
    const double lambda = from.lambda();
    const auto y = from.y();
    const auto halo = from.halo();
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
        D64.fetch(from.tab64());
        if constexpr (D64.whole) arrive(D64.v);
        line_apply(D64, f);
    }
#pragma unroll
    for (int c = 0; c < n1; ++c) pin(f[c]);
    step();
    double dot = 0.0;
    {
        // node and weight of each layer up to the middle; above, x_{N-c} = -x_c and
        // w_{N-c} = w_c
        double zw[n1 + (L::odd ? 1 : 0)];
        const auto xs = from.xw();
#pragma unroll
        for (int i = 0; i < n1 + (L::odd ? 1 : 0); ++i) zw[i] = xs[i];
        const double wab = w_a * w_b;
        const std::conditional_t<(N <= 2), Direct, Column> g(C, r_a, s_b);
        // lambda times the mass of a node is (mass w_c) J + extra: the diagonal mass
        // w J, or the identity mass, 1 / multiplicity of the node (a power of two)
        double mass = lambda * wab, extra = 0.0;
        bool below = false, above = false;  // elements that share the column's end nodes
        {
            const auto p = from.plan();
            if (invdeg) {
                mass = 0.0;
                extra = lambda;
                const int ex = at.x * p->kx + lx, ey = at.y * p->ky + ly, ez = at.z * p->kz + lz;
                if ((a == 0 && ex > 0) || (a == N && ex < p->nx - 1)) extra *= 0.5;
                if ((b == 0 && ey > 0) || (b == N && ey < p->ny - 1)) extra *= 0.5;
                below = ez > 0;
                above = ez < p->nz - 1;
            }
        }
        sync();
        arrive(zw);
#pragma unroll
        for (int c = 0; c < n1; ++c) {
            step();
            // (read one node ahead, these cost registers that are worth a wave per SIMD
            // at N = 5: 42^3 111 us against 106; even at N = 7 and 15)
            const double qr = col1[c * P2], qs = col0[c * P2], qt = f[c];
            // opaque: products shared with layer N - c would be kept in registers
            const double z = opaque(2 * c <= N ? zw[2 * c] : -zw[2 * (N - c)]);
            const double w = opaque(zw[2 * (2 * c <= N ? c : N - c) + 1]);
            double cr[3], cs[3], ct[3], v[3];
            const double J = g.at(z, cr, cs, ct);
            const double wj = wab * w * reciprocal(J);
#pragma unroll
            for (int i = 0; i < 3; ++i) v[i] = wj * (cr[i] * qr + cs[i] * qs + ct[i] * qt);
            const double fr = cr[0] * v[0] + cr[1] * v[1] + cr[2] * v[2];
            const double fs = cs[0] * v[0] + cs[1] * v[1] + cs[2] * v[2];
            const double ft = ct[0] * v[0] + ct[1] * v[1] + ct[2] * v[2];
            const double mq = __builtin_fma(mass * w, J, (c == 0 && below) || (c == N && above) ? 0.5 * extra : extra) * static_cast<double>(q[c]);
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
        if ((t & 63) == 0) red[t >> 6] = ws;
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
        D64.fetch(from.tab64() + T1);
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
    // the tile's numbers for the assembly, on their way while the lines are written
    const auto p = from.plan();
    const int kx = p->kx, ky = p->ky, kz = p->kz, ntx = p->ntx, nty = p->nty, ntz = p->ntz, gx = p->gx, gy = p->gy;
    const int sx = p->sx, sxy = p->sxy, off = p->off;
    const uint32_t hx0 = p->hx, hy0 = p->hy;
    const bool upx = epb > 1 && lx + 1 < min(kx, p->nx - at.x * kx), upy = epb > 1 && ly + 1 < min(ky, p->ny - at.y * ky),
               upz = epb > 1 && lz + 1 < min(kz, p->nz - at.z * kz);  // neighbours above in the tile
    sync();
    step();
#pragma unroll
    for (int c = 0; c < n1; ++c) q[c] += col0[c * P2] + col1[c * P2];
    // assembly of the tile: a node shared by elements of the tile goes to the
    // element that has it on its first plane, whose column adds the others' copies
    // from LDS in a fixed order; each column then stores its nodes
    if constexpr (epb > 1) {
        if (kx * ky * kz > 1) {
            const int ystep = kx * L::vol, zstep = kx * ky * L::vol;
            const bool edge = (a == N && upx) || (b == N && upy);
            if (active) {
#pragma unroll
                for (int c = 0; c < n1; ++c)
                    if (edge || (c == N && upz)) col0[c * P2] = q[c];
            }
            __syncthreads();
            const bool shx = a == 0 && lx > 0, shy = b == 0 && ly > 0, shz = lz > 0;
            auto add = [&](const T *o) {
                const auto l = pinned(o);
#pragma unroll
                for (int c = 0; c < n1; ++c) q[c] += l[c * P2];
            };
            if (active && shx) add(col0 + N - L::vol);
            if (active && shy) {
                add(col0 + N * P1 - ystep);
                if (shx) add(col0 + N * P1 - ystep + N - L::vol);
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
        const bool hx = a == N && at.x + 1 < ntx, hy = b == N && at.y + 1 < nty, hz = at.z + 1 < ntz;
        const int kn = lz * N, cz = kz * N + 1;
        const int I = (at.x * kx + lx) * N + a, J = (at.y * ky + ly) * N + b, K0 = at.z * kz * N + kn;
        gptr<T> out;
        int stride;
        bool on = true, on0 = true, on1 = !upz;
        if (ADD == kAddDirect) {
            stride = sxy;
            out = y + (off + I + sx * J + stride * K0);
            if constexpr (MASK) {
                on = I > 0 && I < gx - 1 && J > 0 && J < gy - 1;
                on0 = K0 > 0;
                on1 = on1 && K0 + N < p->gz - 1;
            }
        } else if (hx) {
            out = halo + (hx0 + (((at.x * nty + at.y) * ntz + at.z) * cz + kn) * (ky * N + 1) + ly * N + b);
            stride = ky * N + 1;
        } else if (hy) {
            out = halo + (hy0 + ((at.y * ntz + at.z) * cz + kn) * gx + I);
            stride = gx;
        } else {
            stride = sxy;
            out = y + (off + I + sx * J + stride * K0);
            if constexpr (MASK) {
                on = I > 0 && I < gx - 1 && J > 0 && J < gy - 1;
                on0 = K0 > 0;
                on1 = on1 && K0 + N < p->gz - 1;
            }
            if (hz && !upz) {  // the tile's last z plane
                on1 = false;
                halo[(at.z * gy + J) * gx + I] = q[N];
            }
        }
        if (!MASK || on) {
#pragma unroll
            for (int c = 0; c < n1; ++c) {
                if ((MASK && c == 0 && !on0) || (c == N && !on1)) continue;
                gptr<T> o = out + c * stride;
                if constexpr (ADD == kAddDirect) {
                    atomicAdd((T *)o, q[c]);
                } else if constexpr (ADD == kAdd) {
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

template <int N, int V, typename T, bool DOT, bool MASK, int ADD>
__global__ __launch_bounds__((Shape<N, V>::threads)) void ax_kernel(AxArgs<T> args)
{
    __shared__ __attribute__((aligned(16))) T lds[Shape<N, V>::lds];
    __shared__ double red[Shape<N, V>::threads / 64];
    const AxFromArgs<T> from{(cptr<AxArgs<T>>)__builtin_amdgcn_kernarg_segment_ptr()};
    const TilePlace at = place_in_walk(args.plan, xcd_remap(blockIdx.x, gridDim.x));
    const double d = ax_tile<N, V, T, DOT, MASK, ADD>(lds, red, from, at);
    if (DOT && threadIdx.x == 0) to_global(opaque(from.k)->partial)[blockIdx.x] = d;
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

// One (problem, tile) item of a work list.
template <int N, int V, typename T, bool MASK>
__device__ __attribute__((always_inline)) inline void batch_item(T *lds, double *red, int32_t prob, int32_t tile,
                                                                 const BatchProb *__restrict__ probs)
{
    const AxFromBatch<T> from{to_const(probs + prob)};
    const double d = ax_tile<N, V, T, true, MASK, kAssign>(lds, red, from, tile_place(probs[prob].plan, tile));
    if (threadIdx.x == 0) to_global(opaque(from.k)->part_ax)[tile] = d;
}

// The batched operator: one block per item of a class's work list, with p.Ap fused.
template <int N, int V, typename T, bool MASK>
__global__ __launch_bounds__((Shape<N, V>::threads)) void batch_ax_kernel(const WorkItem *__restrict__ items,
                                                                         const BatchProb *__restrict__ probs)
{
    __shared__ __attribute__((aligned(16))) T lds[Shape<N, V>::lds];
    __shared__ double red[Shape<N, V>::threads / 64];
    const WorkItem it = items[xcd_remap(blockIdx.x, gridDim.x)];
    batch_item<N, V, T, MASK>(lds, red, uniform(it.prob), uniform(it.idx), probs);
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
hb_status launch_ax_n(const hb_mesh_s *m, int v, const T *tab, double lambda, const double *x, T *y, T *halo, bool add,
                      double *partial, CgState *st, hipStream_t s)
{
    const TilePlan &p = m->plan[v];
    return with_variant<N>(v, [&](auto VV) -> hb_status {
        constexpr int V = decltype(VV)::value;
        const int grid = p.tiles(), threads = Shape<N, V>::threads;
        const AxArgs<T> args{p, m->coef, tab, m->tab, m->xw, operator_lambda<T>(lambda), x, y, halo, partial, st};
        if (st)
            ax_kernel<N, V, T, true, MASK, kAssign><<<grid, threads, 0, s>>>(args);
        else if (!add)
            ax_kernel<N, V, T, false, MASK, kAssign><<<grid, threads, 0, s>>>(args);
        else if constexpr (sizeof(T) == 8) {
            if (halo)
                ax_kernel<N, V, T, false, MASK, kAdd><<<grid, threads, 0, s>>>(args);
            else
                ax_kernel<N, V, T, false, MASK, kAddDirect><<<grid, threads, 0, s>>>(args);
        }
        HB_HIP(hipGetLastError());
        return HB_OK;
    });
}

template <int N, bool MASK>
hb_status launch_batch_ax_n(int v, bool fp32, const WorkItem *items, int nitems, const BatchProb *probs, hipStream_t s)
{
    if (nitems == 0) return HB_OK;
    return with_variant<N>(v, [&](auto VV) -> hb_status {
        constexpr int V = decltype(VV)::value;
        if (fp32)
            batch_ax_kernel<N, V, float, MASK><<<nitems, Shape<N, V>::threads, 0, s>>>(items, probs);
        else
            batch_ax_kernel<N, V, double, MASK><<<nitems, Shape<N, V>::threads, 0, s>>>(items, probs);
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
    hb_status launch_ax##suffix##n(const hb_mesh_s *m, int v, double l, const double *x, double *y, double *halo, \
                                   bool add, double *p, CgState *st, hipStream_t s)                              \
    {                                                                                                            \
        return launch_ax_n<n, double, MASK>(m, v, m->tab, l, x, y, halo, add, p, st, s);                         \
    }                                                                                                            \
    hb_status launch_ax32##suffix##n(const hb_mesh_s *m, int v, double l, const double *x, float *y, float *halo, \
                                     double *p, CgState *st, hipStream_t s)                                      \
    {                                                                                                            \
        return launch_ax_n<n, float, MASK>(m, v, m->tab32, l, x, y, halo, false, p, st, s);                      \
    }                                                                                                            \
    hb_status launch_batch_ax##suffix##n(int v, bool fp32, const WorkItem *it, int ni, const BatchProb *pr,       \
                                         hipStream_t s)                                                          \
    {                                                                                                            \
        return launch_batch_ax_n<n, MASK>(v, fp32, it, ni, pr, s);                                               \
    }                                                                                                            \
    }
#define HB_AX_INSTANCE(n) HB_AX_ENTRY(n, _, false)
#define HB_AX_INSTANCE_DIRICHLET(n) HB_AX_ENTRY(n, _d_, true)
