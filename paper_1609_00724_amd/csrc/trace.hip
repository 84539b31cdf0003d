// Field-line + deviation tracer for gfx950 (QSL Squasher, Sect. 3.1-3.5).
//
// A trace call, after the seed pass and the work list (in spatial order):
//   stepping   each half-line (seed x direction) takes adaptive Cash-Karp 5(4)
//              steps of y = (x, dx1, dx2) under eq. (1) and eq. (5) in the
//              stepping precision T until a trial step leaves the box or a
//              stop condition holds.  k_trace: persistent wave64 lanes, one
//              half-line each, refilled from a device work counter (ballot +
//              prefix count).  k_trace_quad (quad.h): four lanes a half-line,
//              for lists whose longest line sets the time.  Where the list's
//              length decides, both are launched and one returns at once.
//              k_trace_geo (quad_geo.h): general geometry.
//   ends       FP64: the step that left the box re-solved for the step length
//              whose 5th-order end lies on the first face crossed (regula
//              falsi on the signed face distance, Anderson-Bjorck variant),
//              then snapped to it; per seed, the deviations perpendicular to
//              the renormalised field at both ends and Q by eq. (10)-(11), the
//              determinant form, the exit-face-plane Q and the length.
//              k_finish (finish.h) does both for calls of few seeds
//              (finish_seeds); k_land, k_land_final (k_land_euler) and
//              k_assemble for larger ones.  k_land_geo: general geometry.
// launch_rules.h holds the rules that choose.
//
// Field records are 4-vectors per node (x fastest): PAPER mode holds
// (Bhat, |B|) with Bhat = B/|B| formed on the nodes (footnote to Sect. 3.5);
// INTERP_NORMALIZE holds B.  One RHS evaluation gathers the 8 corner records of
// the containing cell (eq. 3-4) and forms the value and the analytic gradient
// of the trilinear interpolant with a lerp tree (Sect. 3.3).
#include <math.h>

#include <mutex>
#include <type_traits>

#include "launch_rules.h"
#include "qsq_internal.h"

namespace qsq {

// One line is computed by different kernels in different calls (one lane or
// four, any gather, landing apart or together with Q), and has to come out the
// same.  So the compiler fuses nothing here on its own: every fused
// multiply-add of this file and the headers it includes is written as one.
#pragma clang fp contract(off)

// ---------------------------------------------------------------------------
// Cash-Karp 5(4) coefficients (Cash & Karp 1990, the stepper of Sect. 3.4)
// ---------------------------------------------------------------------------
namespace ck {
constexpr double a21 = 1.0 / 5.0;
constexpr double a31 = 3.0 / 40.0, a32 = 9.0 / 40.0;
constexpr double a41 = 3.0 / 10.0, a42 = -9.0 / 10.0, a43 = 6.0 / 5.0;
constexpr double a51 = -11.0 / 54.0, a52 = 5.0 / 2.0, a53 = -70.0 / 27.0, a54 = 35.0 / 27.0;
constexpr double a61 = 1631.0 / 55296.0, a62 = 175.0 / 512.0, a63 = 575.0 / 13824.0,
                 a64 = 44275.0 / 110592.0, a65 = 253.0 / 4096.0;
constexpr double b1 = 37.0 / 378.0, b3 = 250.0 / 621.0, b4 = 125.0 / 594.0, b6 = 512.0 / 1771.0;
// difference between the 5th- and the embedded 4th-order weights
constexpr double e1 = b1 - 2825.0 / 27648.0, e3 = b3 - 18575.0 / 48384.0,
                 e4 = b4 - 13525.0 / 55296.0, e5 = -277.0 / 14336.0, e6 = b6 - 1.0 / 4.0;
}  // namespace ck

// ---------------------------------------------------------------------------
// node loads
// ---------------------------------------------------------------------------
// A pointer read from a table in memory, as one into global memory: the
// compiler cannot tell and would take flat loads, which also wait on LDS
template <typename P>
__device__ __forceinline__ const P *in_global(const void *p)
{
    return (const P *)(const __attribute__((address_space(1))) P *)reinterpret_cast<uintptr_t>(p);
}

template <typename T>
struct V4 {
    T x, y, z, w;
};

__device__ __forceinline__ V4<float> ld4(const float *__restrict__ p, int64_t i)
{
    float4 v = reinterpret_cast<const float4 *>(p)[i];
    return {v.x, v.y, v.z, v.w};
}

__device__ __forceinline__ V4<double> ld4(const double *__restrict__ p, int64_t i)
{
    const double2 *q = reinterpret_cast<const double2 *>(p) + 2 * i;
    double2 a = q[0], b = q[1];
    return {a.x, a.y, b.x, b.y};
}

// BF16 records: one 8-byte load, each value widened to FP32 exactly
__device__ __forceinline__ V4<float> ld4(const Bf16 *__restrict__ p, int64_t i)
{
    const uint2 v = reinterpret_cast<const uint2 *>(p)[i];
    return {__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
            __uint_as_float(v.y & 0xffff0000u)};
}

// value and grid-unit partial derivatives of one trilinear component
template <typename T>
__device__ __forceinline__ void lerp_tree(T v000, T v100, T v010, T v110, T v001, T v101, T v011,
                                          T v111, T tx, T ty, T tz, T &val, T &dx, T &dy, T &dz)
{
    const T d00 = v100 - v000, d10 = v110 - v010, d01 = v101 - v001, d11 = v111 - v011;
    const T a00 = fma(tx, d00, v000), a10 = fma(tx, d10, v010);
    const T a01 = fma(tx, d01, v001), a11 = fma(tx, d11, v011);
    const T e0 = a10 - a00, e1 = a11 - a01;
    const T b0 = fma(ty, e0, a00), b1 = fma(ty, e1, a01);
    const T g0 = fma(ty, d10 - d00, d00), g1 = fma(ty, d11 - d01, d01);
    dz = b1 - b0;
    val = fma(tz, dz, b0);
    dx = fma(tz, g1 - g0, g0);
    dy = fma(tz, e1 - e0, e0);
}

template <typename T>
__device__ __forceinline__ T lerp_val(T v000, T v100, T v010, T v110, T v001, T v101, T v011, T v111,
                                      T tx, T ty, T tz)
{
    const T a00 = fma(tx, v100 - v000, v000), a10 = fma(tx, v110 - v010, v010);
    const T a01 = fma(tx, v101 - v001, v001), a11 = fma(tx, v111 - v011, v011);
    const T b0 = fma(ty, a10 - a00, a00), b1 = fma(ty, a11 - a01, a01);
    return fma(tz, b1 - b0, b0);
}

// Cell of a point given in grid units as integer reference ib plus offset q:
// c = clamp(floor(ib + q), 0, n-2), fraction t = ib + q - c (not clamped, so
// points slightly outside the box extrapolate the boundary cell linearly).
template <typename T>
__device__ __forceinline__ void cell_of(int ib, T q, int n, int &c, T &t)
{
    const T fl = floor(q);
    int ci = ib + (int)fl;
    ci = ci < 0 ? 0 : ci;
    ci = ci > n - 2 ? n - 2 : ci;
    c = ci;
    t = q - (T)(ci - ib);
}

// ---------------------------------------------------------------------------
// Higher interpolation orders (Sect. 3.2): the 27-vertex triquadratic stencil
// (Dodgson 1997) and the 64-vertex tricubic stencil (Keys 1981).  The order
// rides in the MODE template value: bit 0 is the interpolation mode
// (QSQ_INTERP_*), the bits above hold order - 1.
// ---------------------------------------------------------------------------
template <int MODE>
constexpr int interp_order() { return ((MODE >> 1) & 3) + 1; }
template <int MODE>
constexpr bool normalize_first() { return (MODE & 1) == QSQ_INTERP_PAPER; }

// Per-axis stencil of K = order + 1 nodes starting at node s, with the
// weights w of the values and dw of the grid-unit derivative.  Cubic (Keys'
// kernel with a = -1/2): nodes c-1 .. c+2 of the cell c, fraction t.
// Quadratic (Dodgson's interpolating kernel, 1 - 2d^2 within half a spacing,
// d^2 - 5|d|/2 + 3/2 out to 3/2 spacings): the node m nearest the point and
// its two neighbours, offset u = t or t - 1 from m.  A stencil node beyond the
// grid stands for Keys' extrapolation f(-1) = 3 f(0) - 3 f(1) + f(2) (and the
// same at the top end); its weight is folded onto those three nodes and the
// stencil starts at the first node inside.  The last weight is then zero and
// its node index may lie past the grid (the caller clamps it).
template <int K, typename T>
__device__ __forceinline__ void axis_stencil(int c, T t, int n, int &s, T w[K], T dw[K])
{
    if constexpr (K == 4) {
        const T t2 = t * t, t3 = t2 * t;
        const T a2 = (T)3 * t2, b2 = (T)9 * t2, a3 = (T)3 * t3;
        w[0] = (T)0.5 * (fma((T)2, t2, -t3) - t);
        w[1] = (T)0.5 * (fma((T)-5, t2, a3) + (T)2);
        w[2] = (T)0.5 * (fma((T)4, t2, -a3) + t);
        w[3] = (T)0.5 * fma(t, t2, -t2);
        dw[0] = (T)0.5 * (fma((T)4, t, -a2) - (T)1);
        dw[1] = (T)0.5 * fma((T)-10, t, b2);
        dw[2] = (T)0.5 * (fma((T)8, t, -b2) + (T)1);
        dw[3] = (T)0.5 * fma((T)-2, t, a2);
        s = c - 1;
    } else {
        const bool low = t < (T)0.5;
        const T u = low ? t : t - (T)1;
        w[0] = u * (u - (T)0.5);
        w[1] = fma(-u, (T)2 * u, (T)1);
        w[2] = u * (u + (T)0.5);
        dw[0] = fma((T)2, u, (T)-0.5);
        dw[1] = (T)-4 * u;
        dw[2] = fma((T)2, u, (T)0.5);
        s = low ? c - 1 : c;
    }
    if (s < 0) {
        // node -1 folded onto nodes 0, 1, 2 (weights 3, -3, 1)
        const T a = w[0], da = dw[0];
#pragma unroll
        for (int k = 0; k < K - 1; ++k) {
            w[k] = w[k + 1];
            dw[k] = dw[k + 1];
        }
        w[K - 1] = (T)0;
        dw[K - 1] = (T)0;
        w[0] = fma((T)3, a, w[0]), w[1] = fma((T)-3, a, w[1]), w[2] += a;
        dw[0] = fma((T)3, da, dw[0]), dw[1] = fma((T)-3, da, dw[1]), dw[2] += da;
        s = 0;
    } else if (s + K - 1 > n - 1) {
        // node n folded onto nodes n-1, n-2, n-3 (weights 3, -3, 1); the
        // stencil then starts at n-3
        const T a = w[K - 1], da = dw[K - 1];
        const int shift = s - (n - 3);   // 0 for the cubic, 1 for the quadratic stencil
        T nw[K], ndw[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            nw[k] = (T)0;
            ndw[k] = (T)0;
        }
#pragma unroll
        for (int k = 0; k < K - 1; ++k) {
            nw[k + shift] += w[k];
            ndw[k + shift] += dw[k];
        }
        nw[0] += a, nw[1] = fma((T)-3, a, nw[1]), nw[2] = fma((T)3, a, nw[2]);
        ndw[0] += da, ndw[1] = fma((T)-3, da, ndw[1]), ndw[2] = fma((T)3, da, ndw[2]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            w[k] = nw[k];
            dw[k] = ndw[k];
        }
        s = n - 3;
    }
}

// Value and grid-unit gradient of the first NC record components by the
// separable stencil sum: along x per row, then y, then z.
template <int K, int NC, typename T, typename S>
__device__ __forceinline__ void stencil_sum(const S *__restrict__ nodes, const Geom &g, const int s[3],
                                            const T w[3][K], const T dw[3][K], T val[NC], T dx[NC], T dy[NC],
                                            T dz[NC])
{
#pragma unroll
    for (int k = 0; k < NC; ++k) val[k] = dx[k] = dy[k] = dz[k] = (T)0;
    const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
    // rows one at a time (only the K records of a row in flight): unrolling
    // the z and y loops lets the compiler hoist all K^3 loads and spill
#pragma unroll 1
    for (int kz = 0; kz < K; ++kz) {
        const int iz = s[2] + kz < g.n[2] - 1 ? s[2] + kz : g.n[2] - 1;
        T ay[NC], axy[NC], ayy[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) ay[k] = axy[k] = ayy[k] = (T)0;
#pragma unroll 1
        for (int ky = 0; ky < K; ++ky) {
            const int iy = s[1] + ky < g.n[1] - 1 ? s[1] + ky : g.n[1] - 1;
            const int64_t row = (int64_t)iz * sz + (int64_t)iy * sy;
            T rx[NC], drx[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) rx[k] = drx[k] = (T)0;
#pragma unroll
            for (int kx = 0; kx < K; ++kx) {
                const int ix = s[0] + kx < g.n[0] - 1 ? s[0] + kx : g.n[0] - 1;
                const auto v = ld4(nodes, row + ix);
                const T c4[4] = {(T)v.x, (T)v.y, (T)v.z, (T)v.w};
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    rx[k] = fma(w[0][kx], c4[k], rx[k]);
                    drx[k] = fma(dw[0][kx], c4[k], drx[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                ay[k] = fma(w[1][ky], rx[k], ay[k]);
                axy[k] = fma(w[1][ky], drx[k], axy[k]);
                ayy[k] = fma(dw[1][ky], rx[k], ayy[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            val[k] = fma(w[2][kz], ay[k], val[k]);
            dx[k] = fma(w[2][kz], axy[k], dx[k]);
            dy[k] = fma(w[2][kz], ayy[k], dy[k]);
            dz[k] = fma(dw[2][kz], ay[k], dz[k]);
        }
    }
}

// u . g, beginning with the second component
template <typename T>
__device__ __forceinline__ T along(T u0, T u1, T u2, T g0, T g1, T g2)
{
    return fma(u2, g2, fma(u0, g0, u1 * g1));
}

// |v|^2 of a field vector interpolated in T from records of type S.  Every
// evaluator of a call's types forms it here: the order of the sum shows in the
// results, and they depend neither on the gather nor on the size of the call.
// (Trilinear FP32 records stepped in FP32 begin with the first component, all
// others with the second: what the register cache and the direct loads gave
// when the order was the compiler's.)
template <typename T, typename S, int MODE>
__device__ __forceinline__ T norm2(T v0, T v1, T v2)
{
    constexpr bool first = std::is_same<T, float>::value && std::is_same<S, float>::value && MODE >> 1 == 0;
    return first ? fma(v2, v2, fma(v1, v1, v0 * v0)) : along(v0, v1, v2, v0, v1, v2);
}

// u, the physical gradient rows and |B| from the interpolated components
// (value and grid-unit derivatives; val[3] = interpolated |B| in PAPER mode)
template <typename T, typename S, int MODE, bool MAG>
__device__ __forceinline__ void field_finish(const double ih[3], const T val[4], const T dx[4], const T dy[4],
                                             const T dz[4], T u[3], T G[3][3], T &mag)
{
    const T ihx = (T)ih[0], ihy = (T)ih[1], ihz = (T)ih[2];
    if (normalize_first<MODE>()) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i];
            G[0][i] = dx[i] * ihx;
            G[1][i] = dy[i] * ihy;
            G[2][i] = dz[i] * ihz;
        }
        if (MAG) mag = val[3];
    } else {
        // u = B/|B|, grad u = (I - u u^T) grad B / |B|
        const T bn = sqrt(norm2<T, S, MODE>(val[0], val[1], val[2]));
        const T inv = bn > (T)1e-300 ? (T)1 / bn : (T)0;
        T Gb[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i] * inv;
            Gb[0][i] = dx[i] * ihx;
            Gb[1][i] = dy[i] * ihy;
            Gb[2][i] = dz[i] * ihz;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const T ug = along(u[0], u[1], u[2], Gb[j][0], Gb[j][1], Gb[j][2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) G[j][i] = fma(-u[i], ug, Gb[j][i]) * inv;
        }
        if (MAG) mag = bn;
    }
}

// Field value u (Bhat as interpolated) and physical gradient rows
// G[j][i] = d u_i / d x_j at a point; optionally |B| (PAPER: interpolated node
// magnitudes; INTERP_NORMALIZE: magnitude of the interpolated B).
// CELLS: `nodes` points at cell records (the 8 corner records of each cell,
// contiguous, corner a + 2b + 4c) instead of node records; the same values.
template <typename T, typename S, int MODE, bool MAG, bool CELLS = false>
__device__ __forceinline__ void field_at(const S *__restrict__ nodes, const Geom &g, const int ib[3],
                                         const T q[3], T u[3], T G[3][3], T &mag)
{
    int c[3];
    T t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) cell_of(ib[d], q[d], g.n[d], c[d], t[d]);
    T val[4], dx[4], dy[4], dz[4];
    if constexpr (interp_order<MODE>() > 1) {
        constexpr int K = interp_order<MODE>() + 1;
        int s0[3];
        T w[3][K], dw[3][K];
#pragma unroll
        for (int d = 0; d < 3; ++d) axis_stencil<K, T>(c[d], t[d], g.n[d], s0[d], w[d], dw[d]);
        // |B| is the 4th component in PAPER mode; INTERP_NORMALIZE takes |interpolated B|
        constexpr int NC = (MAG && normalize_first<MODE>()) ? 4 : 3;
        stencil_sum<K, NC, T, S>(nodes, g, s0, w, dw, val, dx, dy, dz);
        field_finish<T, S, MODE, MAG>(g.ih, val, dx, dy, dz, u, G, mag);
        return;
    }
    int64_t o[8];
    if constexpr (CELLS) {
        const int64_t b = 8 * (((int64_t)c[2] * (g.n[1] - 1) + c[1]) * (g.n[0] - 1) + c[0]);
#pragma unroll
        for (int v = 0; v < 8; ++v) o[v] = b + v;
    } else {
        const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
        const int64_t b = (int64_t)c[2] * sz + (int64_t)c[1] * sy + c[0];
        o[0] = b, o[1] = b + 1, o[2] = b + sy, o[3] = b + sy + 1;
        o[4] = b + sz, o[5] = b + sz + 1, o[6] = b + sz + sy, o[7] = b + sz + sy + 1;
    }
    const auto n000 = ld4(nodes, o[0]), n100 = ld4(nodes, o[1]);
    const auto n010 = ld4(nodes, o[2]), n110 = ld4(nodes, o[3]);
    const auto n001 = ld4(nodes, o[4]), n101 = ld4(nodes, o[5]);
    const auto n011 = ld4(nodes, o[6]), n111 = ld4(nodes, o[7]);
#define QSQ_COMP(F, k)                                                                              \
    lerp_tree<T>((T)n000.F, (T)n100.F, (T)n010.F, (T)n110.F, (T)n001.F, (T)n101.F, (T)n011.F,       \
                 (T)n111.F, t[0], t[1], t[2], val[k], dx[k], dy[k], dz[k])
    QSQ_COMP(x, 0);
    QSQ_COMP(y, 1);
    QSQ_COMP(z, 2);
#undef QSQ_COMP
    if (MAG && normalize_first<MODE>())
        val[3] = lerp_val<T>((T)n000.w, (T)n100.w, (T)n010.w, (T)n110.w, (T)n001.w, (T)n101.w, (T)n011.w,
                             (T)n111.w, t[0], t[1], t[2]);
    field_finish<T, S, MODE, MAG>(g.ih, val, dx, dy, dz, u, G, mag);
}

// The interpolated direction u alone (no gradient): the same operations as
// the value part of field_at, so both give the same u bit for bit.
template <typename T, typename S, int MODE>
__device__ __forceinline__ void field_u(const S *__restrict__ nodes, const Geom &g, const int ib[3], const T q[3],
                                        T u[3])
{
    int c[3];
    T t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) cell_of(ib[d], q[d], g.n[d], c[d], t[d]);
    T val[3];
    if constexpr (interp_order<MODE>() > 1) {
        // the same stencil sums as field_at (the derivative sums are not used)
        constexpr int K = interp_order<MODE>() + 1;
        int s0[3];
        T w[3][K], dw[3][K], dx[3], dy[3], dz[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) axis_stencil<K, T>(c[d], t[d], g.n[d], s0[d], w[d], dw[d]);
        stencil_sum<K, 3, T, S>(nodes, g, s0, w, dw, val, dx, dy, dz);
    } else {
        const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
        const int64_t b = (int64_t)c[2] * sz + (int64_t)c[1] * sy + c[0];
        const auto n000 = ld4(nodes, b), n100 = ld4(nodes, b + 1);
        const auto n010 = ld4(nodes, b + sy), n110 = ld4(nodes, b + sy + 1);
        const auto n001 = ld4(nodes, b + sz), n101 = ld4(nodes, b + sz + 1);
        const auto n011 = ld4(nodes, b + sz + sy), n111 = ld4(nodes, b + sz + sy + 1);
#define QSQ_COMPV(F, k)                                                                                  \
    val[k] = lerp_val<T>((T)n000.F, (T)n100.F, (T)n010.F, (T)n110.F, (T)n001.F, (T)n101.F, (T)n011.F,    \
                         (T)n111.F, t[0], t[1], t[2])
        QSQ_COMPV(x, 0);
        QSQ_COMPV(y, 1);
        QSQ_COMPV(z, 2);
#undef QSQ_COMPV
    }
    if (normalize_first<MODE>()) {
#pragma unroll
        for (int i = 0; i < 3; ++i) u[i] = val[i];
    } else {
        const T bn = sqrt(norm2<T, S, MODE>(val[0], val[1], val[2]));
        const T inv = bn > (T)1e-300 ? (T)1 / bn : (T)0;
#pragma unroll
        for (int i = 0; i < 3; ++i) u[i] = val[i] * inv;
    }
}

// a0 b0 + a1 b1 + a2 b2, beginning with the first component
template <typename T>
__device__ __forceinline__ T jdot(T a0, T a1, T a2, T b0, T b1, T b2)
{
    return fma(a2, b2, fma(a1, b1, a0 * b0));
}

// Right-hand side f(y) = sigma * (u, J dx1, J dx2), J_ij = d u_i / d x_j
// (eq. 1 and eq. 5).  Returns |u|^2 for the null test.
template <typename T>
__device__ __forceinline__ T rhs_from(T sigma, const T u[3], const T G[3][3], const T d1[3], const T d2[3],
                                      T kx[3], T k1[3], T k2[3])
{
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        kx[i] = sigma * u[i];
        k1[i] = sigma * jdot(G[0][i], G[1][i], G[2][i], d1[0], d1[1], d1[2]);
        k2[i] = sigma * jdot(G[0][i], G[1][i], G[2][i], d2[0], d2[1], d2[2]);
    }
    return jdot(u[0], u[1], u[2], u[0], u[1], u[2]);
}

template <typename T, typename S, int MODE, bool CELLS = false>
__device__ __forceinline__ T rhs(const S *__restrict__ nodes, const Geom &g, const int ib[3],
                                 const T q[3], T sigma, const T d1[3], const T d2[3], T kx[3],
                                 T k1[3], T k2[3])
{
    T u[3], G[3][3], mag;
    field_at<T, S, MODE, false, CELLS>(nodes, g, ib, q, u, G, mag);
    return rhs_from(sigma, u, G, d1, d2, kx, k1, k2);
}

// Raw buffer load of 16 bytes.  Lanes whose byte offset lies at or beyond the
// buffer's record count get zeros back without any memory access, which lets a
// wave gather only for the lanes that need new data, with no divergent branch.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ f32x4 qsq_buffer_load16(__amdgpu_buffer_rsrc_t rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.ptr.buffer.load.v4f32");

// Raw buffer load of 8 bytes (one BF16 node record), same out-of-range rule.
typedef int i32x2 __attribute__((ext_vector_type(2)));
__device__ i32x2 qsq_buffer_load8(__amdgpu_buffer_rsrc_t rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.ptr.buffer.load.v2i32");

// Buffer resource over the node records (gfx9 descriptor word 3).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t node_rsrc(const void *nodes, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(nodes), (short)0, bytes, 0x00020000);
}

// bytes of one node record: 4 x FP32 or 4 x BF16
template <typename S>
constexpr int node_bytes() { return std::is_same<S, float>::value ? 16 : 8; }

// direction part (3 values, widened to FP32 exactly) of the node record at a
// byte offset
template <typename S>
__device__ __forceinline__ void load_dir(__amdgpu_buffer_rsrc_t rsrc, int off, float &x, float &y, float &z)
{
    if constexpr (std::is_same<S, float>::value) {
        const f32x4 v = qsq_buffer_load16(rsrc, off, 0, 0);
        x = v.x;
        y = v.y;
        z = v.z;
    } else {
        const i32x2 v = qsq_buffer_load8(rsrc, off, 0, 0);
        x = __uint_as_float((uint32_t)v.x << 16);
        y = __uint_as_float((uint32_t)v.x & 0xffff0000u);
        z = __uint_as_float((uint32_t)v.y << 16);
    }
}

// Per-lane cache of the 8 corner records (direction part, 24 floats) of the
// cell a lane evaluated last, kept in LDS (6 float4 planes of one workgroup's
// lanes, lane-consecutive, conflict-free 16-byte accesses).  Consecutive Runge-Kutta
// stages mostly fall in the same cell: only lanes whose stage point moved to
// another cell fetch from memory (the others issue out-of-range offsets, see
// above) and store the new corners into their slot; every lane then reads its
// slot (a wave's LDS operations complete in order).  Keyed by cell index
// alone, so it stays valid across the lines a lane traces.
constexpr int kCachePlanes = 6;

template <typename T, typename S, int MODE>
__device__ __forceinline__ T rhs_cached(__amdgpu_buffer_rsrc_t rsrc, int bytes, const Geom &g, const int ib[3],
                                        const T q[3], T sigma, const T d1[3], const T d2[3], T kx[3], T k1[3],
                                        T k2[3], int cc[3], float4 *slot, int stride)
{
    int c[3];
    T t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) cell_of(ib[d], q[d], g.n[d], c[d], t[d]);
    const bool miss = c[0] != cc[0] || c[1] != cc[1] || c[2] != cc[2];
    const int sy = g.n[0], sz = g.n[0] * g.n[1];
    constexpr int NB = node_bytes<S>();
    const int base = miss ? NB * (c[2] * sz + c[1] * sy + c[0]) : bytes;
    float w[24];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int o = NB * (((k & 1) ? 1 : 0) + ((k & 2) ? sy : 0) + ((k & 4) ? sz : 0));
        load_dir<S>(rsrc, base + o, w[3 * k], w[3 * k + 1], w[3 * k + 2]);
    }
    if (miss) {
#pragma unroll
        for (int j = 0; j < kCachePlanes; ++j) slot[j * stride] = make_float4(w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]);
    }
    cc[0] = c[0];
    cc[1] = c[1];
    cc[2] = c[2];
    float v[24];
#pragma unroll
    for (int j = 0; j < kCachePlanes; ++j) {
        const float4 x = slot[j * stride];
        v[4 * j] = x.x;
        v[4 * j + 1] = x.y;
        v[4 * j + 2] = x.z;
        v[4 * j + 3] = x.w;
    }
    T val[3], dx[3], dy[3], dz[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        lerp_tree<T>((T)v[i], (T)v[3 + i], (T)v[6 + i], (T)v[9 + i], (T)v[12 + i], (T)v[15 + i],
                     (T)v[18 + i], (T)v[21 + i], t[0], t[1], t[2], val[i], dx[i], dy[i], dz[i]);
    const T ihx = (T)g.ih[0], ihy = (T)g.ih[1], ihz = (T)g.ih[2];
    T u[3], G[3][3];
    if (normalize_first<MODE>()) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i];
            G[0][i] = dx[i] * ihx;
            G[1][i] = dy[i] * ihy;
            G[2][i] = dz[i] * ihz;
        }
    } else {
        const T bn = sqrt(norm2<T, S, MODE>(val[0], val[1], val[2]));
        const T inv = bn > (T)1e-300 ? (T)1 / bn : (T)0;
        T Gb[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i] * inv;
            Gb[0][i] = dx[i] * ihx;
            Gb[1][i] = dy[i] * ihy;
            Gb[2][i] = dz[i] * ihz;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const T ug = along(u[0], u[1], u[2], Gb[j][0], Gb[j][1], Gb[j][2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) G[j][i] = fma(-u[i], ug, Gb[j][i]) * inv;
        }
    }
    return rhs_from(sigma, u, G, d1, d2, kx, k1, k2);
}

// Per-lane cache of the 8 corner records (direction part, 24 floats) of the
// cell a lane evaluated last, kept in registers; the cell before it is parked
// in the lane's LDS slot, and a lane that moves back into it takes its corners
// from there instead of memory.  Only the lanes that moved load (the memory
// pipeline returns data for active lanes alone); a wave whose lanes all stayed
// in their cells issues no load and waits for none.  The node values and the
// arithmetic are those of the direct gather: the results are the same bit for
// bit.  The key is the cell's node index within the field (below 2 GiB).
//
// The corners are vector variables that every load fills in place (`pin` keeps
// the compiler from splitting them into scalars); only the lanes that move back
// copy, from a second set, so that their LDS reads and the others' loads are
// under way together.  From scalars each stage copied 50 registers: 4.87e8
// vector instructions for the stepping of a 1024 x 1024 map, 4.19e8 so.  (Two
// slots and reads straight into the corners leave out those copies too, but
// wait for one after the other: 0.92 of the speed.)
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
}

// eight corners of 3 values (a + 2b + 4c), loaded with 12 bytes each
struct CellNodes {
    typedef float Part __attribute__((ext_vector_type(3)));
    Part v0, v1, v2, v3, v4, v5, v6, v7;
    static constexpr int kPlanes = 8;

    template <int C, int I>
    __device__ __forceinline__ float get() const
    {
        return (C == 0 ? v0 : C == 1 ? v1 : C == 2 ? v2 : C == 3 ? v3 : C == 4 ? v4 : C == 5 ? v5 : C == 6 ? v6 : v7)[I];
    }
    __device__ __forceinline__ void pin()
    {
        asm volatile("" : "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3), "+v"(v4), "+v"(v5), "+v"(v6), "+v"(v7));
    }
    // to the lane's slot, eight planes of a wave's 16-byte rows
    __device__ __forceinline__ void put(float4 *slot) const
    {
        asm volatile("ds_write_b96 %0, %1\n\t"
                     "ds_write_b96 %0, %2 offset:1024\n\t"
                     "ds_write_b96 %0, %3 offset:2048\n\t"
                     "ds_write_b96 %0, %4 offset:3072\n\t"
                     "ds_write_b96 %0, %5 offset:4096\n\t"
                     "ds_write_b96 %0, %6 offset:5120\n\t"
                     "ds_write_b96 %0, %7 offset:6144\n\t"
                     "ds_write_b96 %0, %8 offset:7168" ::"v"(lds_address(slot)),
                     "v"(v0), "v"(v1), "v"(v2), "v"(v3), "v"(v4), "v"(v5), "v"(v6), "v"(v7)
                     : "memory");
    }
    __device__ __forceinline__ void get(const float4 *slot)
    {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(slot);
        v0 = p[0].xyz;
        v1 = p[64].xyz;
        v2 = p[128].xyz;
        v3 = p[192].xyz;
        v4 = p[256].xyz;
        v5 = p[320].xyz;
        v6 = p[384].xyz;
        v7 = p[448].xyz;
    }
};

// the same 24 values as a direction record packs them, six 16-byte parts
struct CellDirs {
    typedef float Part __attribute__((ext_vector_type(4)));
    Part v0, v1, v2, v3, v4, v5;
    static constexpr int kPlanes = 6;

    template <int C, int I>
    __device__ __forceinline__ float get() const
    {
        constexpr int e = 3 * C + I, p = e / 4;
        return (p == 0 ? v0 : p == 1 ? v1 : p == 2 ? v2 : p == 3 ? v3 : p == 4 ? v4 : v5)[e % 4];
    }
    __device__ __forceinline__ void pin()
    {
        asm volatile("" : "+v"(v0), "+v"(v1), "+v"(v2), "+v"(v3), "+v"(v4), "+v"(v5));
    }
    __device__ __forceinline__ void put(float4 *slot) const
    {
        Part *p = reinterpret_cast<Part *>(slot);
        p[0] = v0;
        p[64] = v1;
        p[128] = v2;
        p[192] = v3;
        p[256] = v4;
        p[320] = v5;
    }
    __device__ __forceinline__ void get(const float4 *slot)
    {
        const Part *p = reinterpret_cast<const Part *>(slot);
        v0 = p[0];
        v1 = p[64];
        v2 = p[128];
        v3 = p[192];
        v4 = p[256];
        v5 = p[320];
    }
};

// a lane's cached cell: its corners, the keys of the present and the previous
// cell, the LDS address of the present cell's slot (flip - at: the other slot's)
template <typename Cell>
struct CellCache {
    Cell c = {};
    int key = -1, prev = -1;
    float4 *slot = nullptr;
};

// the direction part of a node record, loaded straight into a corner
template <typename S>
__device__ __forceinline__ CellNodes::Part load_corner(__amdgpu_buffer_rsrc_t rsrc, int off)
{
    if constexpr (std::is_same<S, float>::value) {
        return __builtin_bit_cast(CellNodes::Part, __builtin_amdgcn_raw_buffer_load_b96(rsrc, off, 0, 0));
    } else {
        float x, y, z;
        load_dir<S>(rsrc, off, x, y, z);
        return CellNodes::Part{x, y, z};
    }
}

// record layouts of the register cache
constexpr int kLayoutNodes = 0, kLayoutBricks = 1, kLayoutDirs = 2;

// BRICKS: the records are the field's brick records (2 x 2 x 2 node bricks,
// bricks x fastest): node (i, j, k) sits at ((k/2 nby + j/2) nbx + i/2) 8 +
// 4 (k & 1) + 2 (j & 1) + (i & 1), so the step from a corner to its neighbour
// along an axis is 1, 2, 4 records from an even index and 7, 8 nbx - 2,
// 8 nbx nby - 4 from an odd one.  DIRS: `dirs` holds the field's direction
// records, the cell's 24 values in six 16-byte loads (global addresses: the
// records may exceed 2 GiB), keyed by the cell's index.
template <typename T, typename S, int MODE, int LAYOUT, typename Cell, typename Late>
__device__ __forceinline__ T rhs_regs(__amdgpu_buffer_rsrc_t rsrc, const float4 *__restrict__ dirs,
                                      const Geom &g, const int ib[3], const T q[3], T sigma, const T d1[3],
                                      const T d2[3], T kx[3], T k1[3], T k2[3], CellCache<Cell> &cc, Late late)
{
    int c[3];
    T t[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) cell_of(ib[d], q[d], g.n[d], c[d], t[d]);
    int b, sx, sy, sz;
    if constexpr (LAYOUT == kLayoutDirs) {
        b = (c[2] * (g.n[1] - 1) + c[1]) * (g.n[0] - 1) + c[0];
        sx = sy = sz = 0;
    } else if constexpr (LAYOUT == kLayoutBricks) {
        const int nbx = (g.n[0] + 1) >> 1, nby = (g.n[1] + 1) >> 1;
        b = (((c[2] >> 1) * nby + (c[1] >> 1)) * nbx + (c[0] >> 1)) * 8 + ((c[2] & 1) << 2) + ((c[1] & 1) << 1) +
            (c[0] & 1);
        sx = (c[0] & 1) ? 7 : 1;
        sy = (c[1] & 1) ? 8 * nbx - 2 : 2;
        sz = (c[2] & 1) ? 8 * nbx * nby - 4 : 4;
    } else {
        sx = 1;
        sy = g.n[0];
        sz = g.n[0] * g.n[1];
        b = c[2] * sz + c[1] * sy + c[0];
    }
    Cell &v = cc.c;
    if (b != cc.key) {
        const bool back = b == cc.prev;
        cc.prev = cc.key;
        cc.key = b;
        Cell old;
        if (back) old.get(cc.slot);
        v.put(cc.slot);
        if (!back) {
            if constexpr (LAYOUT == kLayoutDirs) {
                const CellDirs::Part *p = reinterpret_cast<const CellDirs::Part *>(dirs + 6 * (int64_t)b);
                v = Cell{p[0], p[1], p[2], p[3], p[4], p[5]};
            } else {
                constexpr int NB = node_bytes<S>();
                const int o = NB * b;
                const int ox = NB * sx, oy = NB * sy, oz = NB * sz;
                v.v0 = load_corner<S>(rsrc, o);
                v.v1 = load_corner<S>(rsrc, o + ox);
                v.v2 = load_corner<S>(rsrc, o + oy);
                v.v3 = load_corner<S>(rsrc, o + oy + ox);
                v.v4 = load_corner<S>(rsrc, o + oz);
                v.v5 = load_corner<S>(rsrc, o + oz + ox);
                v.v6 = load_corner<S>(rsrc, o + oz + oy);
                v.v7 = load_corner<S>(rsrc, o + oz + oy + ox);
            }
        }
        if (back) {
            old.pin();
            v = old;
        }
    }
    late();
    v.pin();
    T val[3], dx[3], dy[3], dz[3];
#define QSQ_COMPB(I)                                                                                            \
    lerp_tree<T>((T)v.template get<0, I>(), (T)v.template get<1, I>(), (T)v.template get<2, I>(),               \
                 (T)v.template get<3, I>(), (T)v.template get<4, I>(), (T)v.template get<5, I>(),               \
                 (T)v.template get<6, I>(), (T)v.template get<7, I>(), t[0], t[1], t[2], val[I], dx[I], dy[I], dz[I])
    QSQ_COMPB(0);
    QSQ_COMPB(1);
    QSQ_COMPB(2);
#undef QSQ_COMPB
    const T ihx = (T)g.ih[0], ihy = (T)g.ih[1], ihz = (T)g.ih[2];
    T u[3], G[3][3];
    if (normalize_first<MODE>()) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i];
            G[0][i] = dx[i] * ihx;
            G[1][i] = dy[i] * ihy;
            G[2][i] = dz[i] * ihz;
        }
    } else {
        const T bn = sqrt(norm2<T, S, MODE>(val[0], val[1], val[2]));
        const T inv = bn > (T)1e-300 ? (T)1 / bn : (T)0;
        T Gb[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            u[i] = val[i] * inv;
            Gb[0][i] = dx[i] * ihx;
            Gb[1][i] = dy[i] * ihy;
            Gb[2][i] = dz[i] * ihz;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const T ug = along(u[0], u[1], u[2], Gb[j][0], Gb[j][1], Gb[j][2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) G[j][i] = fma(-u[i], ug, Gb[j][i]) * inv;
        }
    }
    return rhs_from(sigma, u, G, d1, d2, kx, k1, k2);
}

// 5th-order combination and the 5th-minus-4th error combination of the
// stage slopes, fused operations spelled out
template <typename T>
__device__ __forceinline__ T ck_b5(T k0, T k2, T k3, T k5)
{
    return fma((T)ck::b6, k5, fma((T)ck::b4, k3, fma((T)ck::b3, k2, (T)ck::b1 * k0)));
}

template <typename T>
__device__ __forceinline__ T ck_e(T k0, T k2, T k3, T k4, T k5)
{
    return fma((T)ck::e6, k5, fma((T)ck::e5, k4, fma((T)ck::e4, k3, fma((T)ck::e3, k2, (T)ck::e1 * k0))));
}

// position x moved by h k: FP64 stepping fuses, FP32 adds the rounded product
__device__ __forceinline__ double advance(double x, float h, float k) { return x + (double)(h * k); }
__device__ __forceinline__ double advance(double x, double h, double k) { return fma(h, k, x); }

// atol + rtol max(|old|, |new|)
template <typename T>
__device__ __forceinline__ T err_scale(T atol, T rtol, T a, T b)
{
    return fma(rtol, fmax(fabs(a), fabs(b)), atol);
}

// a / b of the error norm: FP32 stepping multiplies by the hardware
// reciprocal (within 1 ulp; the norm only steers accept/reject and the step
// factor), FP64 stepping divides exactly
__device__ __forceinline__ float err_ratio(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ double err_ratio(double a, double b) { return a / b; }

// gather variants of the stepping kernel: direct corner loads, the LDS cell
// cache and the register cell cache (the caches: FP32 or BF16 storage, FP32
// stepping, one field below 2 GiB)
constexpr int kGatherDirect = 0, kGatherLds = 1, kGatherRegs = 2, kGatherCells = 3, kGatherBricks = 4,
              kGatherDirs = 5;

// one RHS evaluation of the stepping kernel
template <typename T, typename S, int MODE, int GATHER, typename Cell, typename Late>
__device__ __forceinline__ T rhs_step(const S *__restrict__ nodes, __amdgpu_buffer_rsrc_t rsrc, int bytes,
                                      const Geom &g, const int ib[3], const T q[3], T sigma, const T d1[3],
                                      const T d2[3], T kx[3], T k1[3], T k2[3], int lc[3], float4 *slot,
                                      int stride, CellCache<Cell> &cc, Late late)
{
    if constexpr (GATHER == kGatherLds)
        return rhs_cached<T, S, MODE>(rsrc, bytes, g, ib, q, sigma, d1, d2, kx, k1, k2, lc, slot, stride);
    else if constexpr (GATHER == kGatherRegs || GATHER == kGatherBricks || GATHER == kGatherDirs)
        // (the direction records' variant gets them as `nodes`)
        return rhs_regs<T, S, MODE,
                        GATHER == kGatherBricks ? kLayoutBricks : GATHER == kGatherDirs ? kLayoutDirs : kLayoutNodes>(
            rsrc, reinterpret_cast<const float4 *>(nodes), g, ib, q, sigma, d1, d2, kx, k1, k2, cc, late);
    else
        return rhs<T, S, MODE, GATHER == kGatherCells>(nodes, g, ib, q, sigma, d1, d2, kx, k1, k2);
}

// ---------------------------------------------------------------------------
// General geometry (Sect. 3.1-3.2): spherical coordinates (longitude phi,
// latitude theta, radius r; field components in the local orthonormal basis)
// and rectilinear axes whose cells have spans of their own.  MODE bit 3.
// These fields are stepped in physical coordinates by k_trace_geo and landed
// by k_land_geo; the seed pass and the Q assembly are shared.
// ---------------------------------------------------------------------------
template <int MODE>
constexpr bool geo_mode() { return (MODE & 8) != 0; }

// cell, fraction of the cell and the cell's span per axis at a physical point;
// a rectilinear axis is searched by bisection for the last cell whose lower
// node lies at or below the point (clamped to the grid's cells)
__device__ __forceinline__ void geo_cell(const Geom &g, const double x[3], int c[3], double t[3], double h[3])
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double *X = g.coord[d];
        const int n = g.n[d];
        if (X) {
            const double xv = fmax(x[d], -1e300);   // NaN -> the lowest cell
            int lo = 0, hi = n - 2;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (X[mid] <= xv)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            c[d] = lo;
            h[d] = X[lo + 1] - X[lo];
            t[d] = (x[d] - X[lo]) / h[d];
        } else {
            const double sg = fmin(fmax((x[d] - g.o[d]) * g.ih[d], -1e9), 1e9);
            double fl = floor(sg);
            fl = fl < 0.0 ? 0.0 : (fl > (double)(n - 2) ? (double)(n - 2) : fl);
            c[d] = (int)fl;
            t[d] = sg - fl;
            h[d] = g.h[d];
        }
    }
}

// trilinear value and physical gradient at a physical point
template <typename T, typename S, int MODE, bool MAG>
__device__ __forceinline__ void field_at_geo(const S *__restrict__ nodes, const Geom &g, const double x[3], T u[3],
                                             T G[3][3], T &mag)
{
    int c[3];
    double t64[3], h[3];
    geo_cell(g, x, c, t64, h);
    const T t[3] = {(T)t64[0], (T)t64[1], (T)t64[2]};
    const double ih[3] = {1.0 / h[0], 1.0 / h[1], 1.0 / h[2]};
    const int64_t sy = g.n[0], sz = (int64_t)g.n[0] * g.n[1];
    const int64_t b = (int64_t)c[2] * sz + (int64_t)c[1] * sy + c[0];
    const auto n000 = ld4(nodes, b), n100 = ld4(nodes, b + 1);
    const auto n010 = ld4(nodes, b + sy), n110 = ld4(nodes, b + sy + 1);
    const auto n001 = ld4(nodes, b + sz), n101 = ld4(nodes, b + sz + 1);
    const auto n011 = ld4(nodes, b + sz + sy), n111 = ld4(nodes, b + sz + sy + 1);
    T val[4], dx[4], dy[4], dz[4];
#define QSQ_COMPG(F, k)                                                                             \
    lerp_tree<T>((T)n000.F, (T)n100.F, (T)n010.F, (T)n110.F, (T)n001.F, (T)n101.F, (T)n011.F,       \
                 (T)n111.F, t[0], t[1], t[2], val[k], dx[k], dy[k], dz[k])
    QSQ_COMPG(x, 0);
    QSQ_COMPG(y, 1);
    QSQ_COMPG(z, 2);
#undef QSQ_COMPG
    if (MAG && normalize_first<MODE>())
        val[3] = lerp_val<T>((T)n000.w, (T)n100.w, (T)n010.w, (T)n110.w, (T)n001.w, (T)n101.w, (T)n011.w,
                             (T)n111.w, t[0], t[1], t[2]);
    field_finish<T, S, MODE, MAG>(ih, val, dx, dy, dz, u, G, mag);
}

// metric factors of eq. (2) and (8) at a physical point: (r cos theta, r, 1)
// in spherical geometry, ones otherwise
__device__ __forceinline__ void geo_scale(const Geom &g, const double x[3], double sc[3])
{
    if (g.geometry == QSQ_GEOMETRY_SPHERICAL) {
        sc[0] = x[2] * cos(x[1]);
        sc[1] = x[2];
        sc[2] = 1.0;
    } else {
        sc[0] = sc[1] = sc[2] = 1.0;
    }
}

// FP64 evaluation at a physical point (landing, assembly, seed frame)
template <typename S, int MODE, bool MAG>
__device__ __forceinline__ void field_at_x(const S *__restrict__ nodes, const Geom &g, const double x[3],
                                           double u[3], double G[3][3], double &mag)
{
    if constexpr (geo_mode<MODE>()) {
        field_at_geo<double, S, MODE, MAG>(nodes, g, x, u, G, mag);
        return;
    }
    int ib[3];
    double q[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double s = (x[d] - g.o[d]) * g.ih[d];
        s = fmin(fmax(s, -1e9), 1e9);
        const double fl = floor(s);
        ib[d] = (int)fl;
        q[d] = s - fl;
    }
    field_at<double, S, MODE, MAG>(nodes, g, ib, q, u, G, mag);
}

// not a point of the closed box (a non-finite coordinate is outside)
__device__ __forceinline__ bool outside_box(const Geom &g, double x0, double x1, double x2)
{
    return !(x0 >= g.lo[0] && x0 <= g.hi[0] && x1 >= g.lo[1] && x1 <= g.hi[1] && x2 >= g.lo[2] && x2 <= g.hi[2]);
}

// orthonormal (a, b) completing the unit vector n, branch-free
// (Duff, Burgess, Christensen, Hery, Kensler, Liani, Villemin 2017, JCGT 6(1))
__device__ __forceinline__ void frame_of(const double n[3], double a[3], double b[3])
{
    const double sg = copysign(1.0, n[2]);
    const double p = -1.0 / (sg + n[2]);
    const double q = n[0] * n[1] * p;
    a[0] = fma(sg * n[0] * n[0], p, 1.0);
    a[1] = sg * q;
    a[2] = -sg * n[0];
    b[0] = q;
    b[1] = fma(n[1] * n[1], p, sg);
    b[2] = -n[1];
}

// ---------------------------------------------------------------------------
// end records
// ---------------------------------------------------------------------------
__device__ __forceinline__ void put_rec(const Records &r, int64_t i, const double y[9], double s,
                                        double h, int status, int attempts)
{
    const int64_t P = 2 * r.cap;
#pragma unroll
    for (int k = 0; k < 9; ++k) r.y[k * P + i] = y[k];
    r.s[i] = s;
    r.h[i] = h;
    r.status[i] = status;
    r.attempts[i] = attempts;
}

__device__ __forceinline__ void get_rec(const Records &r, int64_t i, double y[9], double &s, double &h)
{
    const int64_t P = 2 * r.cap;
#pragma unroll
    for (int k = 0; k < 9; ++k) y[k] = r.y[k * P + i];
    s = r.s[i];
    h = r.h[i];
}

__device__ __forceinline__ int64_t seed_count(const TraceJob &j)
{
    return j.n_dev ? *j.n_dev : j.n_host;
}

// ---------------------------------------------------------------------------
// seed pass (FP64, one thread per seed): frame of eq. (9), and the half-lines
// that end at once -- seed outside the box, a null at the seed, or a seed on a
// face with its (signed) field pointing out (zero length, lowest such face).
// The others are flagged for stepping.  Bound by its writes (200 B a seed).  The
// faces are taken in an unrolled loop from the last to the first, all indices
// known: a search that ends at the first hit put the seed's arrays in scratch
// memory (168 B a lane), and 1.3 M seeds took 134 us against 63 (4.1 TB/s).
// ---------------------------------------------------------------------------
// set holding global seed i: the last set whose first seed is <= i (empty
// sets share their offset with the next set and are skipped)
__device__ __forceinline__ int find_set(const SetDesc *sets, int nsets, int64_t i)
{
    int lo = 0, hi = nsets - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sets[mid].off <= i)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

template <typename S, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_seed_pass(TraceJob job)
{
    const int64_t n = seed_count(job);
    if (blockIdx.x == 0 && threadIdx.x == 0) *job.rec.n_items = 2 * n;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const S *__restrict__ nodes = static_cast<const S *>(job.nodes);
        Geom gl = job.g;
        const double *sp = job.seeds;
        int64_t ss = job.seed_stride, li = i;
        if constexpr (BATCH) {
            const int set = find_set(job.sets, job.nsets, i);
            job.set_of[i] = set;
            const SetDesc &sd = job.sets[set];
            gl = sd.g;
            nodes = in_global<S>(sd.nodes);
            sp = sd.seeds;
            ss = sd.n;
            li = i - sd.off;
        }
        const Geom &g = gl;
        const double x0[3] = {sp[li], sp[ss + li], sp[2 * ss + li]};
        double y0[9] = {x0[0], x0[1], x0[2], 0, 0, 0, 0, 0, 0};
        int st[2] = {-1, -1};
        if (outside_box(g, x0[0], x0[1], x0[2])) {
            st[0] = st[1] = QSQ_END_SEED_OUTSIDE;
        } else {
            double u[3], G[3][3], mag;
            field_at_x<S, MODE, false>(nodes, g, x0, u, G, mag);
            const double un = sqrt(along(u[0], u[1], u[2], u[0], u[1], u[2]));
            if (un < 1e-6) {
                st[0] = st[1] = QSQ_END_NULL;
            } else {
                const double nn[3] = {u[0] / un, u[1] / un, u[2] / un};
                double a[3], b[3];
                frame_of(nn, a, b);
                double sc[3] = {1.0, 1.0, 1.0};
                if constexpr (geo_mode<MODE>()) geo_scale(g, x0, sc);   // eq. (8) inverted
                for (int k = 0; k < 3; ++k) {
                    y0[3 + k] = a[k] / sc[k];
                    y0[6 + k] = b[k] / sc[k];
                }
#pragma unroll
                for (int dir = 0; dir < 2; ++dir) {
                    const double sg = dir ? -1.0 : 1.0;
                    st[dir] = kPendingStep;
#pragma unroll
                    for (int f = 5; f >= 0; --f) {   // the lowest face wins
                        const int d = f >> 1;
                        const bool on = (f & 1) ? x0[d] == g.hi[d] : x0[d] == g.lo[d];
                        const double out = (f & 1) ? sg * nn[d] : -sg * nn[d];
                        if (on && out > 0.0) st[dir] = f;
                    }
                }
            }
        }
#pragma unroll
        for (int dir = 0; dir < 2; ++dir) {
            put_rec(job.rec, dir * job.rec.cap + i, y0, 0.0, 0.0, st[dir], 0);
            job.rec.flag[dir * n + i] = st[dir] == kPendingStep ? 1 : 0;
        }
    }
}

// work list: record indices of the flagged half-lines, forward ones first,
// each in seed order
static __global__ void k_compact(TraceJob job)
{
    const int64_t n2 = *job.rec.n_items, n = n2 / 2;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < n2; it += (int64_t)gridDim.x * blockDim.x)
        if (job.rec.flag[it]) job.rec.work[job.rec.wpos[it]] = (int32_t)(it >= n ? job.rec.cap + (it - n) : it);
}

// ---------------------------------------------------------------------------
// spatial order of the work list: sort keys (set, Morton index of the seed's
// cell at `bits` bits per axis of the set's box) for the compacted list; the
// sort itself is a stable radix sort.  No line's arithmetic depends on where
// it runs, so results do not change.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t spread3(uint32_t v)   // bit k of v -> bit 3k
{
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < 10; ++k) r |= ((v >> k) & 1u) << (3 * k);
    return r;
}

template <bool BATCH>
__global__ void k_sort_keys(TraceJob job, int bits)
{
    const int64_t nw = *job.rec.n_work;
    const int64_t P = 2 * job.rec.cap;
    const int side = 1 << bits;
    uint32_t *keys = reinterpret_cast<uint32_t *>(job.rec.flag);
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < nw; w += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = job.rec.work[w];
        const int64_t i = r >= job.rec.cap ? r - job.rec.cap : r;
        const Geom &g = BATCH ? job.sets[job.set_of[i]].g : job.g;
        uint32_t c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double u = (job.rec.y[d * P + r] - g.lo[d]) / (g.hi[d] - g.lo[d]);
            int k = (int)(u * side);
            k = k < 0 ? 0 : (k > side - 1 ? side - 1 : k);
            c[d] = (uint32_t)k;
        }
        const uint32_t set = BATCH ? (uint32_t)job.set_of[i] : 0u;
        keys[w] = (set << (3 * bits)) | spread3(c[0]) | (spread3(c[1]) << 1) | (spread3(c[2]) << 2);
    }
}

// The landing list: the half-lines that the stepping pass left outside the
// box, in record order (forward halves, then backward ones, each in seed
// order), so that the landing kernels read and write the record planes in
// runs rather than in the work list's (spatial) order.  Flags over the half-
// line records, then a compaction into work2.
__device__ __forceinline__ int64_t half_record(const TraceJob &job, int64_t it, int64_t n)
{
    return it >= n ? job.rec.cap + (it - n) : it;
}

static __global__ void k_land_flags(TraceJob job)
{
    const int64_t n2 = *job.rec.n_items, n = n2 / 2;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < n2; it += (int64_t)gridDim.x * blockDim.x)
        job.rec.flag[it] = job.rec.status[half_record(job, it, n)] == kPendingLand ? 1 : 0;
}

static __global__ void k_land_compact(TraceJob job)
{
    const int64_t n2 = *job.rec.n_items, n = n2 / 2;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < n2; it += (int64_t)gridDim.x * blockDim.x)
        if (job.rec.flag[it]) job.rec.work2[job.rec.wpos[it]] = (int32_t)half_record(job, it, n);
}

#include "quad.h"

// ---------------------------------------------------------------------------
// k_trace: persistent stepping kernel
// ---------------------------------------------------------------------------
// Waves per SIMD, least and most.  Left alone, the compiler moves the deviation
// slopes of every stage to the end of the step (the positions do not need
// them) and holds 9 corner differences a stage for them: 210 .. 250 registers,
// two waves.  With each stage's slopes formed while the next stage's corners
// are on their way (`late` in rhs_regs) 168 do: three waves, stepping of a 1024
// x 1024 map 1.64 -> 1.36 ms (together with the corners above), the first
// pass over a 384 x 384 x 256 rope from brick records 89.4 -> 82.6 ms, the L1 taking
// a lane's record per cycle 81 % of the time.  The other gathers are bound by
// the caches behind it, which three waves' cells overflow: direction records
// 43.8 ms with two waves, 46.2 with three; batched fields 3.1 against 3.6; direct
// loads of one field, 500 000 half-lines of 224 x 224 x 112 cells at a 1-cell cap,
// FP32 records 9.4 against 10.9, FP64 15.8 against 20.7, BF16 6.6 against 9.6.  Cell
// records (contiguous, no line shared with the next cell's) take all three that
// fit: FP32 5.7 with two and 6.0 with three there, but over 128 x 128 x 64 cells
// 200 000 half-lines 1.78 against 1.52, BF16 1.43 against 1.32.
// BF16 node records have the widening of each value on top, and 168 registers
// spill (500 000 lines of 224 x 224 x 112 cells, 4-cell cap: 3.27 ms with three
// waves, 2.64 with two).  FP64 stepping of a batch over FP32 or FP64 records holds
// more than 256 registers, one wave, and is told so: scheduled for two it missed
// them by 10 and took 85.8 ms for 15.9 M lines of 64 fields, 79.7 so; forced to two
// it spills 16, 76.4 there but 2.9 against 2.3 for 186 000 lines of two fields.
template <typename T, typename S, int GATHER, bool BATCH, bool EULER>
constexpr int trace_waves(int most)
{
    const bool three =
        EULER || (GATHER == kGatherRegs && !std::is_same<S, Bf16>::value) || GATHER == kGatherBricks;
    const bool any = sizeof(T) == 8 || three || GATHER == kGatherCells;
    const bool one = sizeof(T) == 8 && BATCH && !EULER && !std::is_same<S, Bf16>::value;
    return most ? (one ? 1 : any ? 8 : 2) : three ? 3 : 1;
}

// a list that the first job.few workgroups step (TraceJob)
__device__ __forceinline__ bool keeps_to_few(const TraceJob &job, int64_t total)
{
    return total > job.few_from || total <= job.few_upto;
}

// values formed here, not where they are used last
template <typename T>
__device__ __forceinline__ void hold(T v[3])
{
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
}

// a value that all lanes hold, in scalar registers
__device__ __forceinline__ float uniform(float v)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ __forceinline__ double uniform(double v) { return v; }

// (the Euler variants fit 3 waves per SIMD: one evaluation's state per step)
template <typename T, typename S, int MODE, int GATHER, bool BATCH, bool EULER = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(trace_waves<T, S, GATHER, BATCH, EULER>(0), trace_waves<T, S, GATHER, BATCH, EULER>(1)))) k_trace(TraceJob job)
{
    static_assert(GATHER == kGatherDirect || (!BATCH && sizeof(T) == 4),
                  "cell caches: one field per launch, FP32 corner values");
    static_assert(GATHER != kGatherDirs || std::is_same<S, float>::value, "direction records: FP32 storage");
    constexpr bool REGS = GATHER == kGatherRegs || GATHER == kGatherBricks || GATHER == kGatherDirs;
    constexpr bool CACHED =
        GATHER == kGatherLds || GATHER == kGatherRegs || GATHER == kGatherBricks || GATHER == kGatherDirs;
    // field and step limits of the lane's line: launch constants for one
    // field, reloaded from the set table at each refill in a batch (the cell
    // records' variant reads them in place of the node records)
    const S *__restrict__ nodes = static_cast<const S *>(
        GATHER == kGatherCells ? job.cells : GATHER == kGatherDirs ? static_cast<const void *>(job.dirs) : job.nodes);
    Geom gl = job.g;
    const Geom &g = gl;
    const StepOpts &o = job.o;
    double h_init = o.h_init, hmin = o.hmin;
    const int lane = (int)(threadIdx.x & 63);
    const int64_t total = *job.rec.n_work;
    if (total <= job.quad_max) return;   // the four-lane kernel's call, or nothing to do
    if (keeps_to_few(job, total) && (int)blockIdx.x >= job.few) return;

    // lane state
    double X[3] = {0, 0, 0}, s = 0.0;
    T D1[3] = {0, 0, 0}, D2[3] = {0, 0, 0};
    T h = 0, sigma = 1;
    int attempts = 0;
    int rec = 0;
    bool active = false, done = false, have_k1 = false;
    T Kx[6][3], K1[6][3], K2[6][3];

    const T rtol = uniform((T)o.rtol), atol = uniform((T)o.atol);
    T hmax = uniform((T)o.h_max);
    T ih[3] = {uniform((T)g.ih[0]), uniform((T)g.ih[1]), uniform((T)g.ih[2])};
    // work counters: attempts, first evaluations of a step, lines begun, lines
    // handed to the landing.  Each lane counts its own; the register caches'
    // adaptive steps, which have no registers to spare, count the wave's from
    // lane masks instead (the scalar work of that shows in short loops: 300 000
    // BF16 Euler lines by direct loads 1.39 ms with masks, 1.15 without)
    constexpr bool MASKS = REGS && !EULER;
    unsigned long long c_att = 0, c_first = 0, c_act = 0, c_land = 0;
    bool tried = false, first = false, landed = false;   // of the lane's last attempt
    // cached-gather state
    const uint64_t nrec = GATHER == kGatherBricks
                              ? 8 * (uint64_t)((g.n[0] + 1) / 2) * ((g.n[1] + 1) / 2) * ((g.n[2] + 1) / 2)
                              : (uint64_t)g.n[0] * g.n[1] * g.n[2];
    const int cbytes = CACHED ? (int)(node_bytes<S>() * nrec) : 0;
    const __amdgpu_buffer_rsrc_t rsrc = node_rsrc(GATHER == kGatherBricks ? job.bricks : job.nodes, cbytes);
    // LDS cell cache: kCachePlanes planes of blockDim.x float4 (dynamic size)
    extern __shared__ float4 lds_cache[];
    int lds_cell[3] = {-1, -1, -1};
    const int stride = (int)blockDim.x;
    float4 *slot = lds_cache + threadIdx.x;
    // register cell cache: a wave's slots together
    using Cell = std::conditional_t<GATHER == kGatherDirs, CellDirs, CellNodes>;
    CellCache<Cell> cell;
    cell.slot = lds_cache + (int)(threadIdx.x >> 6) * 64 * Cell::kPlanes + lane;
    // the brick variant's address registers make 168 too few: position and
    // length wait in LDS while the stages run (two planes of a wave's 16-byte
    // rows behind the slots)
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    constexpr bool PARK = GATHER == kGatherBricks && !EULER;   // (the launcher adds the planes)
    f64x2 *park = reinterpret_cast<f64x2 *>(lds_cache + Cell::kPlanes * blockDim.x) + (int)(threadIdx.x >> 6) * 128 + lane;
    auto leave = [&] {
        if constexpr (PARK) {
            park[0] = f64x2{X[0], X[1]};
            park[64] = f64x2{X[2], s};
        }
    };
    auto fetch = [&] {
        if constexpr (PARK) {
            asm volatile("" ::: "memory");
            const f64x2 u = park[0], v = park[64];
            X[0] = u.x;
            X[1] = u.y;
            X[2] = v.x;
            s = v.y;
        }
    };

    // Work distribution.  The work list is split into nparts contiguous parts
    // (one, or kParts with the partition bit of the launch word), each with
    // its own counter.  Workgroup b starts in part b mod nparts -- the XCD
    // the hardware dispatches it to, so that the lanes of one XCD trace lines
    // whose seeds lie together along the curve and share that XCD's L2 -- and
    // the first item of each of its lanes is the lane's index within the
    // part's workgroups (the launcher starts each counter past those).  After
    // that each wave takes chunks of kChunk items of its part with one atomic
    // and hands them to its idle lanes itself; a wave whose part is used up
    // moves on to the following parts, and its lanes are done when every
    // part is.  Which lane traces which line never changes a result.
    constexpr int64_t kChunk = 64;
    const int nparts = (o.launch >> 9) & 1 ? kParts : 1;
    const int home = (int)(blockIdx.x % (unsigned)nparts);
    unsigned long long *pcount = job.counter + kPartCounter;
    auto pbeg = [&](int p) { return total * p / nparts; };
    int part = home, spent = 0;    // the wave's part; parts found used up
    int64_t cnext = 0, cend = 0;   // the wave's unassigned items [cnext, cend)
    bool first_fill = true;
    for (;;) {
        // ---- refill idle lanes
        if constexpr (MASKS) {
            c_att += __popcll(__ballot(tried));
            c_first += __popcll(__ballot(first));
            c_land += __popcll(__ballot(landed));
            tried = first = landed = false;
        }
        const uint64_t need = __ballot(!active && !done);
        if (need) {
            const int j = __popcll(need & ((1ull << lane) - 1ull));   // rank among idle lanes
            int64_t item = -1;
            if (first_fill) {
                item = pbeg(home) + (int64_t)(blockIdx.x / (unsigned)nparts) * blockDim.x + (threadIdx.x & ~63u) + j;
                if (item >= pbeg(home + 1)) item = -1;
            } else {
                const int k = __popcll(need);
                const int64_t avail = cend - cnext;
                if (avail < k && spent < nparts) {
                    // one more chunk: from the wave's part, or the next part not used up
                    unsigned long long b = 0;
                    int p = part, t = spent;
                    const int leader = __ffsll((unsigned long long)need) - 1;
                    if (lane == leader) {
                        for (;;) {
                            b = atomicAdd(pcount + p, (unsigned long long)kChunk);
                            if ((int64_t)b < pbeg(p + 1)) break;
                            if (++t >= nparts) break;
                            p = p + 1 < nparts ? p + 1 : 0;
                        }
                    }
                    part = __builtin_amdgcn_readlane(p, leader);
                    spent = __builtin_amdgcn_readlane(t, leader);
                    const int64_t fresh = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), leader) << 32) |
                                                    (uint32_t)__builtin_amdgcn_readlane((int)b, leader));
                    const int64_t fend = spent < nparts ? min(fresh + kChunk, pbeg(part + 1)) : fresh;
                    const int64_t got = fend - fresh;
                    if (j < avail)
                        item = cnext + j;
                    else if (j - avail < got)
                        item = fresh + (j - avail);
                    const int64_t used = k - avail < got ? k - avail : got;
                    cnext = fresh + used;
                    cend = fend;
                } else {
                    if (j < avail) item = cnext + j;
                    cnext += k < avail ? k : avail;
                }
            }
            first_fill = false;
            if constexpr (MASKS) c_act += __popcll(__ballot(!active && !done && item >= 0));
            if (!active && !done) {
                if (item < 0) {
                    // no item this round; done once every part is used up
                    done = spent >= nparts;
                } else {
                    // the seed pass left x0 and the frame (eq. 9) in the record
                    rec = job.rec.work[item];
                    const int dir = rec >= job.rec.cap ? 1 : 0;
                    if constexpr (BATCH) {
                        const SetDesc &sd = job.sets[job.set_of[dir ? rec - job.rec.cap : rec]];
                        gl = sd.g;
                        nodes = in_global<S>(sd.nodes);
                        h_init = sd.h_init;
                        hmin = sd.hmin;
                        hmax = (T)sd.h_max;
#pragma unroll
                        for (int d = 0; d < 3; ++d) ih[d] = (T)gl.ih[d];
                    }
                    sigma = dir ? (T)-1 : (T)1;
                    const int64_t P = 2 * job.rec.cap;
                    X[0] = job.rec.y[rec];
                    X[1] = job.rec.y[P + rec];
                    X[2] = job.rec.y[2 * P + rec];
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        D1[k] = (T)job.rec.y[(3 + k) * P + rec];
                        D2[k] = (T)job.rec.y[(6 + k) * P + rec];
                    }
                    s = 0.0;
                    leave();
                    h = (T)h_init;
                    attempts = 0;
                    have_k1 = false;
                    active = true;
                    if constexpr (!MASKS) ++c_act;
                }
            }
        }
        if (__ballot(!done) == 0) break;
        // issue priority among the waves of a SIMD: waves holding a line that
        // has run many attempts go first, so the long lines that end a launch
        // are slowed less by the short ones beside them (scheduling only)
        if (__ballot(active && attempts >= 512)) __builtin_amdgcn_s_setprio(3);
        else if (__ballot(active && attempts >= 256)) __builtin_amdgcn_s_setprio(2);
        else if (__ballot(active && attempts >= 128)) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        if (!active) continue;

        // ---- one step attempt (oracle order: step cap, null, trial, accept/reject, exit)
        fetch();
        int stop = -1;
        if (attempts >= o.max_steps) stop = QSQ_END_MAX_STEPS;

        int ib[3];
        T fb[3];
        if (stop < 0) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double xg = (X[d] - g.o[d]) * g.ih[d];
                const double fl = floor(xg);
                ib[d] = (int)fl;
                fb[d] = (T)fma(X[d] - g.o[d], g.ih[d], -fl);
            }
            if (!EULER && !have_k1) {
                const T un2 = rhs_step<T, S, MODE, GATHER>(nodes, rsrc, cbytes, g, ib, fb, (T)1, D1, D2, Kx[0], K1[0],
                                                           K2[0], lds_cell, slot, stride, cell, [] {});
                if constexpr (MASKS)
                    first = true;
                else
                    ++c_first;
                if (un2 < (T)1e-12) stop = QSQ_END_NULL;   // NaN: not a null (the step reports it)
                have_k1 = true;
            }
        }
        if constexpr (EULER) {
            // explicit Euler (Sect. 3.4): one evaluation at the current point
            // per fixed step h, the whole state advanced along it
            if (stop < 0) {
                const T un2 = rhs_step<T, S, MODE, GATHER>(nodes, rsrc, cbytes, g, ib, fb, (T)1, D1, D2, Kx[0],
                                                           K1[0], K2[0], lds_cell, slot, stride, cell, [] {});
                if constexpr (MASKS)
                    first = true;
                else
                    ++c_first;
                if (un2 < (T)1e-12) stop = QSQ_END_NULL;   // NaN: not a null (the step reports it)
            }
            if (stop < 0) {
                T hs = h;
                bool last = false;
                if (o.max_length > 0.0 && (double)hs >= o.max_length - s) {
                    hs = (T)(o.max_length - s);
                    last = true;
                }
                const T hsig = sigma * hs;
                double Xn[3];
                T D1n[3], D2n[3], fsum = 0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    Xn[i] = advance(X[i], hsig, Kx[0][i]);
                    D1n[i] = fma(hsig, K1[0][i], D1[i]);
                    D2n[i] = fma(hsig, K2[0][i], D2[i]);
                    fsum += ((T)Xn[i] + D1n[i]) + D2n[i];
                }
                ++attempts;
                if constexpr (MASKS)
                    tried = true;
                else
                    ++c_att;
                if (!isfinite(fsum)) {
                    stop = QSQ_END_NONFINITE;
                } else if (outside_box(g, Xn[0], Xn[1], Xn[2])) {
                    // the step that leaves the box: cut at the face in FP64
                    const double y[9] = {X[0], X[1], X[2], (double)D1[0], (double)D1[1], (double)D1[2],
                                         (double)D2[0], (double)D2[1], (double)D2[2]};
                    put_rec(job.rec, rec, y, s, (double)hs, kPendingLand, attempts);
                    active = false;
                    if constexpr (MASKS)
                        landed = true;
                    else
                        ++c_land;
                } else {
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        X[i] = Xn[i];
                        D1[i] = D1n[i];
                        D2[i] = D2n[i];
                    }
                    if (last) {
                        s = o.max_length;
                        stop = QSQ_END_MAX_LENGTH;
                    } else {
                        s += (double)hs;
                    }
                }
            }
        }
        if (!EULER && stop < 0) {
            T hs = h < hmax ? h : hmax;
            bool last = false;
            if (o.max_length > 0.0 && (double)hs >= o.max_length - s) {
                hs = (T)(o.max_length - s);
                last = true;
            }
            // The stage slopes K hold the unsigned right-hand side F; the
            // direction sign rides on the step: sigma F h = F (sigma h), and
            // both products are exact sign flips, so the arithmetic is that of
            // f = sigma F bit for bit.
            const T hsig = sigma * hs;
            // stages 2..6
#define QSQ_STAGE(ST, ...)                                                                          \
    {                                                                                               \
        const T c_[] = {__VA_ARGS__};                                                               \
        T q[3], d1[3], d2[3];                                                                       \
        _Pragma("unroll") for (int i = 0; i < 3; ++i)                                               \
        {                                                                                           \
            T ax = 0, a1 = 0, a2 = 0;                                                               \
            _Pragma("unroll") for (int j = 0; j < ST; ++j)                                          \
            {                                                                                       \
                ax = fma(c_[j], Kx[j][i], ax);                                                      \
                a1 = fma(c_[j], K1[j][i], a1);                                                      \
                a2 = fma(c_[j], K2[j][i], a2);                                                      \
            }                                                                                       \
            q[i] = fma(hsig * ax, ih[i], fb[i]);                                                    \
            d1[i] = fma(hsig, a1, D1[i]);                                                           \
            d2[i] = fma(hsig, a2, D2[i]);                                                           \
        }                                                                                           \
        rhs_step<T, S, MODE, GATHER>(nodes, rsrc, cbytes, g, ib, q, (T)1, d1, d2, Kx[ST], K1[ST], K2[ST], \
                                     lds_cell, slot, stride, cell, [&] {          \
            if constexpr (ST > 1) {                                                                 \
                hold(K1[ST - 1]);                                                                   \
                hold(K2[ST - 1]);                                                                   \
            }                                                                                       \
        });                                                                                         \
    }
            QSQ_STAGE(1, (T)ck::a21)
            QSQ_STAGE(2, (T)ck::a31, (T)ck::a32)
            QSQ_STAGE(3, (T)ck::a41, (T)ck::a42, (T)ck::a43)
            QSQ_STAGE(4, (T)ck::a51, (T)ck::a52, (T)ck::a53, (T)ck::a54)
            QSQ_STAGE(5, (T)ck::a61, (T)ck::a62, (T)ck::a63, (T)ck::a64, (T)ck::a65)
#undef QSQ_STAGE
            // 5th-order solution (propagated) and the error estimate y5 - y4
            fetch();
            double Xn[3];
            T D1n[3], D2n[3];
            T err = 0, fsum = 0;
            bool finite;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const T bx = ck_b5(Kx[0][i], Kx[2][i], Kx[3][i], Kx[5][i]);
                const T b1 = ck_b5(K1[0][i], K1[2][i], K1[3][i], K1[5][i]);
                const T b2 = ck_b5(K2[0][i], K2[2][i], K2[3][i], K2[5][i]);
                const T ex = ck_e(Kx[0][i], Kx[2][i], Kx[3][i], Kx[4][i], Kx[5][i]);
                const T e1 = ck_e(K1[0][i], K1[2][i], K1[3][i], K1[4][i], K1[5][i]);
                const T e2 = ck_e(K2[0][i], K2[2][i], K2[3][i], K2[4][i], K2[5][i]);
                Xn[i] = advance(X[i], hsig, bx);
                D1n[i] = fma(hsig, b1, D1[i]);
                D2n[i] = fma(hsig, b2, D2[i]);
                const T xo = (T)X[i], xn = (T)Xn[i];
                err = fmax(err, err_ratio(fabs(hs * ex), err_scale(atol, rtol, xo, xn)));
                err = fmax(err, err_ratio(fabs(hs * e1), err_scale(atol, rtol, D1[i], D1n[i])));
                err = fmax(err, err_ratio(fabs(hs * e2), err_scale(atol, rtol, D2[i], D2n[i])));
                // one test for the whole state: an infinity or NaN anywhere
                // makes the sum non-finite
                fsum += (xn + D1n[i]) + (D2n[i] + ex) + (e1 + e2);
            }
            finite = isfinite(fsum);
            ++attempts;
            if constexpr (MASKS)
                tried = true;
            else
                ++c_att;
            if (!finite) {
                stop = QSQ_END_NONFINITE;
            } else if (err > (T)1) {
                // reject: shrink, keep k1 (y is unchanged)
                const T f = (T)0.9 * (T)exp2((T)-0.25 * (T)log2(err));
                h = hs * (f > (T)0.2 ? f : (T)0.2);
                if ((double)h < hmin) stop = QSQ_END_UNDERFLOW;
            } else if (outside_box(g, Xn[0], Xn[1], Xn[2])) {
                // accepted trial step leaves the box: hand over to FP64 landing
                const double y[9] = {X[0], X[1], X[2], (double)D1[0], (double)D1[1], (double)D1[2],
                                     (double)D2[0], (double)D2[1], (double)D2[2]};
                put_rec(job.rec, rec, y, s, (double)hs, kPendingLand, attempts);
                active = false;
                if constexpr (MASKS)
                    landed = true;
                else
                    ++c_land;
            } else {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    X[i] = Xn[i];
                    D1[i] = D1n[i];
                    D2[i] = D2n[i];
                }
                have_k1 = false;
                if (last) {
                    s = o.max_length;
                    stop = QSQ_END_MAX_LENGTH;
                } else {
                    s += (double)hs;
                    const T f = err > (T)0 ? (T)0.9 * (T)exp2((T)-0.2 * (T)log2(err)) : (T)5;
                    h = hs * (f < (T)5 ? f : (T)5);
                }
                leave();
            }
        }
        if (stop >= 0) {
            fetch();
            const double y[9] = {X[0], X[1], X[2], (double)D1[0], (double)D1[1], (double)D1[2],
                                 (double)D2[0], (double)D2[1], (double)D2[2]};
            put_rec(job.rec, rec, y, s, 0.0, stop, attempts);
            active = false;
        }
    }
    if (job.work) {
        // one atomic per counter per wave (an adaptive step evaluates 5 more slopes)
        if constexpr (!MASKS) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                c_att += __shfl_xor(c_att, d);
                c_first += __shfl_xor(c_first, d);
                c_act += __shfl_xor(c_act, d);
                c_land += __shfl_xor(c_land, d);
            }
        }
        const unsigned long long sum[4] = {c_att, c_first + (EULER ? 0 : 5 * c_att), c_act, c_land};
        if (lane == 0 && (sum[0] | sum[1] | sum[2] | sum[3])) {   // waves that stepped nothing add nothing
#pragma unroll
            for (int k = 0; k < 4; ++k) atomicAdd(&job.work[k], sum[k]);
        }
    }
}

// ---------------------------------------------------------------------------
// FP64 Cash-Karp step used by the landing pass (5th-order end only)
// ---------------------------------------------------------------------------
template <typename S, int MODE>
__device__ void ck54_fp64(const S *__restrict__ nodes, const Geom &g, double sigma, const double y[9],
                          double hs, double yo[9])
{
    double K[6][9];
    const double A[6][5] = {{0, 0, 0, 0, 0},
                            {ck::a21, 0, 0, 0, 0},
                            {ck::a31, ck::a32, 0, 0, 0},
                            {ck::a41, ck::a42, ck::a43, 0, 0},
                            {ck::a51, ck::a52, ck::a53, ck::a54, 0},
                            {ck::a61, ck::a62, ck::a63, ck::a64, ck::a65}};
    int ib[3];
    double fb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double xg = (y[d] - g.o[d]) * g.ih[d];
        const double fl = floor(fmin(fmax(xg, -1e9), 1e9));
        ib[d] = (int)fl;
        fb[d] = fma(y[d] - g.o[d], g.ih[d], -fl);
    }
#pragma unroll
    for (int st = 0; st < 6; ++st) {
        double q[3], d1[3], d2[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double ax = 0, a1 = 0, a2 = 0;
#pragma unroll
            for (int j = 0; j < st; ++j) {
                ax = fma(A[st][j], K[j][i], ax);
                a1 = fma(A[st][j], K[j][3 + i], a1);
                a2 = fma(A[st][j], K[j][6 + i], a2);
            }
            q[i] = fma(hs * ax, g.ih[i], fb[i]);
            d1[i] = fma(hs, a1, y[3 + i]);
            d2[i] = fma(hs, a2, y[6 + i]);
        }
        double kx[3], k1[3], k2[3];
        rhs<double, S, MODE>(nodes, g, ib, q, sigma, d1, d2, kx, k1, k2);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            K[st][i] = kx[i];
            K[st][3 + i] = k1[i];
            K[st][6 + i] = k2[i];
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
        yo[i] = fma(hs, ck_b5(K[0][i], K[2][i], K[3][i], K[5][i]), y[i]);
}

// The position part of one FP64 Cash-Karp step (eq. (1) alone: the position
// does not depend on the deviation vectors), the same operations as the
// position components of ck54_fp64.
template <typename S, int MODE>
__device__ void ck54_pos(const S *__restrict__ nodes, const Geom &g, double sigma, const double y[3], double hs,
                         double yo[3], double *slope0 = nullptr, const double *k1 = nullptr)
{
    double K[6][3];
    const double A[6][5] = {{0, 0, 0, 0, 0},
                            {ck::a21, 0, 0, 0, 0},
                            {ck::a31, ck::a32, 0, 0, 0},
                            {ck::a41, ck::a42, ck::a43, 0, 0},
                            {ck::a51, ck::a52, ck::a53, ck::a54, 0},
                            {ck::a61, ck::a62, ck::a63, ck::a64, ck::a65}};
    int ib[3];
    double fb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double xg = (y[d] - g.o[d]) * g.ih[d];
        const double fl = floor(fmin(fmax(xg, -1e9), 1e9));
        ib[d] = (int)fl;
        fb[d] = fma(y[d] - g.o[d], g.ih[d], -fl);
    }
#pragma unroll
    for (int st = 0; st < 6; ++st) {
        if (st == 0 && k1) {
            // the first stage sits at y whatever the step length: a caller
            // that took a step from y already has it
#pragma unroll
            for (int i = 0; i < 3; ++i) K[0][i] = k1[i];
            continue;
        }
        double q[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            double ax = 0;
#pragma unroll
            for (int j = 0; j < st; ++j) ax = fma(A[st][j], K[j][i], ax);
            q[i] = fma(hs * ax, g.ih[i], fb[i]);
        }
        double u[3];
        field_u<double, S, MODE>(nodes, g, ib, q, u);
#pragma unroll
        for (int i = 0; i < 3; ++i) K[st][i] = sigma * u[i];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
        yo[i] = fma(hs, ck_b5(K[0][i], K[2][i], K[3][i], K[5][i]), y[i]);
    if (slope0) {
        // dx/dlambda at the start of the step (the first stage)
#pragma unroll
        for (int i = 0; i < 3; ++i) slope0[i] = K[0][i];
    }
}

// First trial step length of the landing: the root in (0, hs) of the
// quadratic with gap g0 < 0 and slope s0 at 0 and gap g1 > 0 at hs, or the
// secant point if that root is not strictly inside.
__device__ __forceinline__ double landing_guess(double g0, double s0, double g1, double hs)
{
    const double sec = -g0 * hs / (g1 - g0);
    const double cq = fma(-s0, hs, g1 - g0) / (hs * hs);
    const double disc = fma(s0, s0, -(4.0 * cq * g0));
    const double den = s0 + sqrt(fmax(disc, 0.0));
    const double h = den > 0.0 ? -2.0 * g0 / den : -1.0;
    return (h > 0.0 && h < hs) ? h : sec;
}

// next trial length of the regula falsi between (a, ga < 0) and (b, gb > 0)
__device__ __forceinline__ double landing_secant(double a, double ga, double b, double gb)
{
    return fma(a, gb, -(b * ga)) / (gb - ga);
}

// v[d] for a run-time d in 0..2 as selects (a dynamic index would put the
// array in scratch memory)
__device__ __forceinline__ double pick3(const double *v, int d)
{
    return d == 0 ? v[0] : (d == 1 ? v[1] : v[2]);
}

// signed distance of x beyond face f (0..5 = x lo, x hi, y lo, ...): > 0 outside
__device__ __forceinline__ double beyond_face(const Geom &g, const double *x, int f)
{
    const int d = f >> 1;
    return (f & 1) ? pick3(x, d) - pick3(g.hi, d) : pick3(g.lo, d) - pick3(x, d);
}

template <typename S, int MODE>
__device__ double face_gap(const S *nodes, const Geom &g, double sigma, const double y[3], double hs,
                           int f, double yo[3], const double k1[3])
{
    if (hs == 0.0) {
#pragma unroll
        for (int i = 0; i < 3; ++i) yo[i] = y[i];
    } else {
        ck54_pos<S, MODE>(nodes, g, sigma, y, hs, yo, nullptr, k1);
    }
    return beyond_face(g, yo, f);
}

// ---------------------------------------------------------------------------
// k_land: FP64 landing of pending half-lines on the first face crossed, in
// two passes.  The step length that ends on the face needs the position only
// (eq. (1) does not involve the deviation vectors), so the root find steps
// three components (few registers, many waves); k_land_final then takes the
// one full nine-component step to the root and snaps onto the face.
// ---------------------------------------------------------------------------
template <typename S, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_land(TraceJob job)
{
    // the list of half-lines to land (compacted after the stepping pass), so
    // that every lane of a wave has one
    const int64_t total = *job.rec.n_land;
    const int64_t P = 2 * job.rec.cap;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < total;
         it += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = job.rec.work2[it];
        if (job.rec.status[r] != kPendingLand) continue;
        const int dir = r >= job.rec.cap ? 1 : 0;
        const int64_t i = dir ? r - job.rec.cap : r;
        const S *__restrict__ nodes = static_cast<const S *>(job.nodes);
        Geom gl = job.g;
        double gtol = job.o.gtol;
        if constexpr (BATCH) {
            const SetDesc &sd = job.sets[job.set_of[i]];
            gl = sd.g;
            nodes = in_global<S>(sd.nodes);
            gtol = sd.gtol;
        }
        const Geom &g = gl;
        const double sigma = dir ? -1.0 : 1.0;
        const double y[3] = {job.rec.y[r], job.rec.y[P + r], job.rec.y[2 * P + r]};
        const double hs = job.rec.h[r];
        double y5[3], v0[3];
        ck54_pos<S, MODE>(nodes, g, sigma, y, hs, y5, v0);
        double best = INFINITY;
        int face = -1;
        double gmax = -INFINITY;
        int fmax_ = 0;
        for (int f = 0; f < 6; ++f) {
            const double gend = beyond_face(g, y5, f);
            if (gend > gmax) {
                gmax = gend;
                fmax_ = f;
            }
            if (!(gend > 0.0)) continue;
            // regula falsi (Anderson-Bjorck) for the step length ending on face f
            double yo[3];
            double a = 0.0, b = hs;
            double ga = face_gap<S, MODE>(nodes, g, sigma, y, a, f, yo, v0);
            double hf;
            if (ga >= 0.0) {
                hf = 0.0;
            } else {
                double gb = gend;
                int side = 0;
                hf = -1.0;
                // the first trial uses the gap's slope at the start of the step
                // (a quadratic model); regula falsi from there on
                const int dd = f >> 1;
                const double s0 = (f & 1) ? pick3(v0, dd) : -pick3(v0, dd);
                const double c0 = landing_guess(ga, s0, gb, hs);
                for (int k = 0; k < 200; ++k) {
                    const double c = k == 0 ? c0 : landing_secant(a, ga, b, gb);
                    const double gc = face_gap<S, MODE>(nodes, g, sigma, y, c, f, yo, v0);
                    if (fabs(gc) <= gtol) {
                        hf = c;
                        break;
                    }
                    // the same end replaced twice in a row: scale the kept
                    // end's gap (Anderson-Bjorck factor 1 - gc/g_old, 1/2
                    // when that is not positive, which is Illinois)
                    if (gc > 0.0) {
                        if (side == 1) {
                            const double m = 1.0 - gc / gb;
                            ga *= m > 0.0 ? m : 0.5;
                        }
                        b = c;
                        gb = gc;
                        side = 1;
                    } else {
                        if (side == -1) {
                            const double m = 1.0 - gc / ga;
                            gb *= m > 0.0 ? m : 0.5;
                        }
                        a = c;
                        ga = gc;
                        side = -1;
                    }
                    if (b - a <= 1e-15 * hs) break;
                }
                if (hf < 0.0) hf = ga > -gb ? a : b;
            }
            if (hf < best) {
                best = hf;
                face = f;
            }
        }
        if (face < 0) {
            // the FP64 re-solve ends inside (the trial end was within rounding
            // of a face): land on the nearest face at the full step
            face = fmax_;
            best = hs;
        }
        job.rec.h[r] = best;
        job.rec.status[r] = kLandFace + face;
    }
}

template <typename S, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_land_final(TraceJob job)
{
    const int64_t total = *job.rec.n_land;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < total;
         it += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = job.rec.work2[it];
        const int face = job.rec.status[r] - kLandFace;
        if (face < 0 || face > 5) continue;   // not landed by k_land
        const int dir = r >= job.rec.cap ? 1 : 0;
        const int64_t i = dir ? r - job.rec.cap : r;
        const S *__restrict__ nodes = static_cast<const S *>(job.nodes);
        Geom gl = job.g;
        if constexpr (BATCH) {
            const SetDesc &sd = job.sets[job.set_of[i]];
            gl = sd.g;
            nodes = in_global<S>(sd.nodes);
        }
        const Geom &g = gl;
        const double sigma = dir ? -1.0 : 1.0;
        double y[9], s, best, yl[9];
        get_rec(job.rec, r, y, s, best);
        if (best > 0.0) {
            ck54_fp64<S, MODE>(nodes, g, sigma, y, best, yl);
        } else {
#pragma unroll
            for (int k = 0; k < 9; ++k) yl[k] = y[k];
        }
        const int d = face >> 1;
        const double snap = (face & 1) ? pick3(g.hi, d) : pick3(g.lo, d);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == d) yl[k] = snap;
        const int att = job.rec.attempts[r];
        put_rec(job.rec, r, yl, s + best, 0.0, face, att);
    }
}

// ---------------------------------------------------------------------------
// k_land_euler: FP64 landing of an explicit Euler step.  The end of an Euler
// step moves linearly with its length, so the length that ends on face f is
// the distance to the face over the step's rate towards it; the first face
// crossed (the shortest such length; exact ties keep the lower face) takes
// the line, the whole state is advanced by that length and the position
// snapped to the face.
// ---------------------------------------------------------------------------
template <typename S, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_land_euler(TraceJob job)
{
    const int64_t total = *job.rec.n_land;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < total;
         it += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = job.rec.work2[it];
        if (job.rec.status[r] != kPendingLand) continue;
        const int dir = r >= job.rec.cap ? 1 : 0;
        const int64_t i = dir ? r - job.rec.cap : r;
        const S *__restrict__ nodes = static_cast<const S *>(job.nodes);
        Geom gl = job.g;
        if constexpr (BATCH) {
            const SetDesc &sd = job.sets[job.set_of[i]];
            gl = sd.g;
            nodes = in_global<S>(sd.nodes);
        }
        const Geom &g = gl;
        const double sigma = dir ? -1.0 : 1.0;
        double y[9], s, hs;
        get_rec(job.rec, r, y, s, hs);
        double u[3], G[3][3], mag;
        field_at_x<S, MODE, false>(nodes, g, y, u, G, mag);
        double dy[9];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            dy[k] = sigma * u[k];
            dy[3 + k] = sigma * jdot(G[0][k], G[1][k], G[2][k], y[3], y[4], y[5]);
            dy[6 + k] = sigma * jdot(G[0][k], G[1][k], G[2][k], y[6], y[7], y[8]);
        }
        double best = INFINITY;
        int face = -1;
        for (int f = 0; f < 6; ++f) {
            const int d = f >> 1;
            const double wall = (f & 1) ? pick3(g.hi, d) : pick3(g.lo, d);
            const double yd = pick3(y, d), vd = pick3(dy, d);
            const double end = fma(hs, vd, yd);
            const double gap = (f & 1) ? end - wall : wall - end;
            if (!(gap > 0.0)) continue;
            double hf = (wall - yd) / vd;
            hf = hf < 0.0 ? 0.0 : (hf > hs ? hs : hf);
            if (hf < best) {
                best = hf;
                face = f;
            }
        }
        double yl[9];
        if (face < 0) {
            // the FP32 step left the box but the FP64 one does not: end on
            // the face nearest the FP64 end point of the full step
            best = hs;
            double gmax = -INFINITY;
            for (int f = 0; f < 6; ++f) {
                const int d = f >> 1;
                const double end = fma(hs, pick3(dy, d), pick3(y, d));
                const double gap = (f & 1) ? end - pick3(g.hi, d) : pick3(g.lo, d) - end;
                if (gap > gmax) {
                    gmax = gap;
                    face = f;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) yl[k] = fma(best, dy[k], y[k]);
        const int d = face >> 1;
        const double snap = (face & 1) ? pick3(g.hi, d) : pick3(g.lo, d);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == d) yl[k] = snap;
        put_rec(job.rec, r, yl, s + best, 0.0, face, job.rec.attempts[r]);
    }
}

// ---------------------------------------------------------------------------
// k_assemble: FP64 Q and length per seed (eq. 10-11)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double dot3(const double *a, const double *b)
{
    return fma(a[2], b[2], fma(a[0], b[0], a[1] * b[1]));
}

__device__ __forceinline__ double cross_len(const double *a, const double *b)
{
    const double c[3] = {fma(a[1], b[2], -(a[2] * b[1])), fma(a[2], b[0], -(a[0] * b[2])), fma(a[0], b[1], -(a[1] * b[0]))};
    return sqrt(dot3(c, c));
}

// a - u s
__device__ __forceinline__ double less_along(double a, double u, double s) { return fma(-u, s, a); }

// a_F^2 b_B^2 + a_B^2 b_F^2 - 2 (a_B . b_B)(a_F . b_F)
__device__ __forceinline__ double q_bracket(const double *aF, const double *bF, const double *aB,
                                            const double *bB)
{
    return fma(-2.0 * dot3(aB, bB), dot3(aF, bF), fma(dot3(aF, aF), dot3(bB, bB), dot3(aB, aB) * dot3(bF, bF)));
}

template <typename S, int MODE, bool BATCH>
__global__ void __launch_bounds__(256) k_assemble(TraceJob job)
{
    const int64_t n = seed_count(job);
    const int64_t P = 2 * job.rec.cap;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t rF = i, rB = job.rec.cap + i;
        // field, seeds and outputs of the seed (its set's in a batch)
        const S *__restrict__ nodes = static_cast<const S *>(job.nodes);
        Geom gl = job.g;
        const double *seeds = job.seeds;
        int64_t ss = job.seed_stride, os = job.out_stride, li = i;
        double *o_fpf = job.fp_fwd, *o_fpb = job.fp_bwd, *o_fll = job.fll;
        double *o_qp = job.q_perp, *o_qd = job.q_det, *o_qf = job.q_fp;
        int32_t *o_st = job.status, *o_steps = job.steps;
        if constexpr (BATCH) {
            const SetDesc &sd = job.sets[job.set_of[i]];
            gl = sd.g;
            nodes = in_global<S>(sd.nodes);
            seeds = sd.seeds;
            ss = os = sd.n;
            li = i - sd.off;
            o_fpf = sd.fp_fwd;
            o_fpb = sd.fp_bwd;
            o_fll = sd.fll;
            o_qp = sd.q_perp;
            o_qd = sd.q_det;
            o_qf = sd.q_fp;
            o_st = sd.status;
            o_steps = sd.steps;
        }
        const Geom &g = gl;
        const int stF = job.rec.status[rF], stB = job.rec.status[rB];
        double yF[9], yB[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            yF[k] = job.rec.y[k * P + rF];
            yB[k] = job.rec.y[k * P + rB];
        }
        const double sF = job.rec.s[rF], sB = job.rec.s[rB];
        const bool open = !(stF == QSQ_END_ZLO && stB == QSQ_END_ZLO);
        const int word = (stF & 0xff) | ((stB & 0xff) << 8) | (open ? QSQ_STATUS_OPEN : 0);
        o_st[li] = word;
        if (o_fll) o_fll[li] = sF + sB;
        if (o_fpf)
            for (int k = 0; k < 3; ++k) o_fpf[k * os + li] = yF[k];
        if (o_fpb)
            for (int k = 0; k < 3; ++k) o_fpb[k * os + li] = yB[k];
        if (o_steps) {
            if (job.steps_sum) {
                o_steps[li] = job.rec.attempts[rF] + job.rec.attempts[rB];
            } else {
                o_steps[li] = job.rec.attempts[rF];
                o_steps[os + li] = job.rec.attempts[rB];
            }
        }
        double qp = NAN, qd = NAN, qf = NAN;
        const bool defF = stF >= QSQ_END_XLO && stF <= QSQ_END_MAX_STEPS;
        const bool defB = stB >= QSQ_END_XLO && stB <= QSQ_END_MAX_STEPS;
        const bool skip = (job.o.flags & QSQ_FLAG_SKIP_OPEN) && open;
        if (defF && defB && !skip) {
            const double x0[3] = {seeds[li], seeds[ss + li], seeds[2 * ss + li]};
            double G[3][3], uF[3], uB[3], u0[3], BF, BB, B0;
            field_at_x<S, MODE, true>(nodes, g, yF, uF, G, BF);
            field_at_x<S, MODE, true>(nodes, g, yB, uB, G, BB);
            field_at_x<S, MODE, true>(nodes, g, x0, u0, G, B0);
            const double vF[3] = {uF[0], uF[1], uF[2]}, vB[3] = {uB[0], uB[1], uB[2]};
            const double nF = sqrt(dot3(uF, uF)), nB = sqrt(dot3(uB, uB));
            for (int k = 0; k < 3; ++k) {
                uF[k] /= nF;
                uB[k] /= nB;
            }
            if constexpr (geo_mode<MODE>()) {
                // the deviations as lengths at each end, eq. (8)
                double scF[3], scB[3];
                geo_scale(g, yF, scF);
                geo_scale(g, yB, scB);
                for (int k = 0; k < 3; ++k) {
                    yF[3 + k] *= scF[k];
                    yF[6 + k] *= scF[k];
                    yB[3 + k] *= scB[k];
                    yB[6 + k] *= scB[k];
                }
            }
            // perpendicular parts of the deviations at both ends (Sect. 3.5)
            double aF[3], bF[3], aB[3], bB[3];
            const double pa = dot3(uF, yF + 3), pb = dot3(uF, yF + 6);
            const double qa = dot3(uB, yB + 3), qb = dot3(uB, yB + 6);
            for (int k = 0; k < 3; ++k) {
                aF[k] = less_along(yF[3 + k], uF[k], pa);
                bF[k] = less_along(yF[6 + k], uF[k], pb);
                aB[k] = less_along(yB[3 + k], uB[k], qa);
                bB[k] = less_along(yB[6 + k], uB[k], qb);
            }
            const double br = q_bracket(aF, bF, aB, bB);
            qp = BF * BB / (B0 * B0) * br;                                  // eq. (11)
            qd = br / (cross_len(aF, bF) * cross_len(aB, bB));
            if (stF <= QSQ_END_ZHI && stB <= QSQ_END_ZHI) {
                // slide the deviations along the line into the exit-face planes
                const int dF = stF >> 1, dB = stB >> 1;
                const double rF1 = yF[3 + dF] / vF[dF], rF2 = yF[6 + dF] / vF[dF];
                const double rB1 = yB[3 + dB] / vB[dB], rB2 = yB[6 + dB] / vB[dB];
                double pF1[3], pF2[3], pB1[3], pB2[3];
                for (int k = 0; k < 3; ++k) {
                    pF1[k] = less_along(yF[3 + k], vF[k], rF1);
                    pF2[k] = less_along(yF[6 + k], vF[k], rF2);
                    pB1[k] = less_along(yB[3 + k], vB[k], rB1);
                    pB2[k] = less_along(yB[6 + k], vB[k], rB2);
                }
                qf = q_bracket(pF1, pF2, pB1, pB2) / (cross_len(pF1, pF2) * cross_len(pB1, pB2));
            }
        }
        if (o_qp) o_qp[li] = qp;
        if (o_qd) o_qd[li] = qd;
        if (o_qf) o_qf[li] = qf;
    }
}

#include "finish.h"

// ---------------------------------------------------------------------------
// General geometry: stepping and landing in physical coordinates
// ---------------------------------------------------------------------------
#include "quad_geo.h"

// counters of the stepping launch's work-list parts: part p starts past the
// first items of its workgroups (blocks b with b mod nparts = p, wg lanes each);
// of the four-lane kernel's qblocks waves where the call is its own
static __global__ void k_part_counters(TraceJob job, int blocks, int wg, int nparts, int qblocks)
{
    const int p = (int)threadIdx.x;
    if (p >= nparts) return;
    const int64_t total = *job.rec.n_work;
    if (total <= job.quad_max) {
        // the four-lane kernel's only counter, past the first 16 items of each wave
        if (p == 0) job.counter[kPartCounter] = (unsigned long long)qblocks * (kQuadWg / 64) * 16;
        return;
    }
    if (keeps_to_few(job, total)) blocks = job.few;
    const int64_t nb = p < blocks ? (blocks - p + nparts - 1) / nparts : 0;
    job.counter[kPartCounter + p] = (unsigned long long)(total * p / nparts + nb * wg);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
#ifndef QSQ_TRACE_HIGH_TU
int set_bits_for(int nsets)
{
    int b = 0;
    while (b < 16 && ((int64_t)1 << b) < (int64_t)nsets) ++b;
    return b;
}

int spatial_bits_for(int nsets)
{
    const int b = (32 - set_bits_for(nsets)) / 3;
    return b < 8 ? b : 8;
}

uint64_t records_bytes(int64_t cap)
{
    const uint64_t P = 2 * (uint64_t)cap, NC = (uint64_t)sort_count_words((int64_t)P);
    const uint64_t scan_n = P > NC ? P : NC;
    return P * (11 * sizeof(double) + 6 * sizeof(int32_t)) + NC * sizeof(int32_t) + 8 +
           (uint64_t)scan_tmp_words((int64_t)scan_n) * 8;
}

void carve_records(void *scratch, int64_t cap, Records *rec, unsigned long long **counter)
{
    char *p = static_cast<char *>(scratch);
    *counter = reinterpret_cast<unsigned long long *>(p);
    p += 256;
    const uint64_t P = 2 * (uint64_t)cap;
    // the scan's block sums need 8-byte alignment; planes below keep it
    rec->y = reinterpret_cast<double *>(p);
    p += 9 * P * sizeof(double);
    rec->s = reinterpret_cast<double *>(p);
    p += P * sizeof(double);
    rec->h = reinterpret_cast<double *>(p);
    p += P * sizeof(double);
    rec->status = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    rec->attempts = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    rec->flag = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    rec->wpos = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    rec->work = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    rec->work2 = reinterpret_cast<int32_t *>(p);
    p += P * sizeof(int32_t);
    const uint64_t NC = (uint64_t)sort_count_words((int64_t)P);
    rec->scnt = reinterpret_cast<int32_t *>(p);
    p += NC * sizeof(int32_t);
    p += (8 - ((uintptr_t)p & 7)) & 7;
    rec->scan_tmp = reinterpret_cast<int64_t *>(p);
    rec->cap = cap;
    // device scalars share the 256-byte block with the work counter
    rec->n_work = reinterpret_cast<int64_t *>(static_cast<char *>(scratch) + 8);
    rec->n_items = reinterpret_cast<int64_t *>(static_cast<char *>(scratch) + 16);
    rec->n_land = reinterpret_cast<int64_t *>(static_cast<char *>(scratch) + 24);
    rec->n_sort = reinterpret_cast<int64_t *>(static_cast<char *>(scratch) + 32);
}

int device_cu_count()
{
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
            v = 256;
        cus[dev] = v;
    }
    return cus[dev];
}

// Workgroups of `kern` (wg lanes, lds bytes of dynamic LDS) that stay resident
// on one CU together, from the runtime's occupancy calculator (cached).
#endif  // QSQ_TRACE_HIGH_TU

static int resident_blocks(const void *kern, int wg, size_t lds)
{
    struct Entry {
        const void *k;
        int wg;
        size_t lds;
        int n;
    };
    static Entry cache[64];
    static int used = 0;
    static std::mutex mu;
    std::lock_guard<std::mutex> lk(mu);
    for (int i = 0; i < used; ++i)
        if (cache[i].k == kern && cache[i].wg == wg && cache[i].lds == lds) return cache[i].n;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, wg, lds) != hipSuccess || n < 1) n = 1;
    if (used < 64) cache[used++] = Entry{kern, wg, lds, n};
    return n;
}

// record bytes that 32-bit offsets reach, with room for the neighbours' offsets
constexpr uint64_t kCacheLimit = ((uint64_t)1 << 31) - ((uint64_t)1 << 26);

// what the launch rules look at
static StepCall step_call(const TraceJob &job, bool step64, bool batch, int64_t n_max)
{
    const Geom &g = job.g;
    StepCall c{};
    c.step64 = step64;
    c.euler = job.o.stepper == QSQ_STEPPER_EULER;
    c.batch = batch;
    c.slice = job.slice;
    c.volume = job.volume;
    c.lattice = job.lattice;
    c.record = job.storage == QSQ_F64 ? 32 : job.storage == QSQ_F32 ? 16 : 8;
    c.field = (uint64_t)g.n[0] * (uint64_t)g.n[1] * (uint64_t)g.n[2] * (uint64_t)c.record;
    c.halves = 2 * n_max;
    c.cap = (c.euler ? job.o.h_init : job.o.h_max) * fmax(fmax(g.ih[0], g.ih[1]), g.ih[2]);
    return c;
}

// the stepping kernel of a gather variant for the job's stepper
template <typename T, typename S, int MODE, int GATHER, bool BATCH>
static const void *trace_kernel(bool euler)
{
    return euler ? reinterpret_cast<const void *>(&k_trace<T, S, MODE, GATHER, BATCH, true>)
                 : reinterpret_cast<const void *>(&k_trace<T, S, MODE, GATHER, BATCH, false>);
}

template <typename T, typename S, int MODE, bool BATCH>
static hipError_t launch_typed(const TraceJob &job, hipStream_t st)
{
    const bool euler = job.o.stepper == QSQ_STEPPER_EULER;
    const int cus = device_cu_count();
    const int64_t n_max = job.n_dev ? job.rec.cap : job.n_host;
    if (n_max <= 0) return hipSuccess;
    int64_t sb = (n_max + 255) / 256;
    const int sblocks = (int)(sb < (int64_t)cus * 16 ? sb : (int64_t)cus * 16);
    hipLaunchKernelGGL((k_seed_pass<S, MODE, BATCH>), dim3(sblocks), dim3(256), 0, st, job);
    int64_t cb = (2 * n_max + 255) / 256;
    const int cblocks = (int)(cb < (int64_t)cus * 16 ? cb : (int64_t)cus * 16);
    launch_scan_i32(job.rec.flag, job.rec.n_items, 2 * n_max, job.rec.scan_tmp, job.rec.wpos, job.rec.n_work, st);
    hipLaunchKernelGGL(k_compact, dim3(cblocks), dim3(256), 0, st, job);
    if (job.spatial_bits > 0) {
        // work list in spatial order: keys (in the flag array, free now),
        // then the stable sort with the work list as values
        const int bits = job.spatial_bits;
        hipLaunchKernelGGL((k_sort_keys<BATCH>), dim3(cblocks), dim3(256), 0, st, job, bits);
        const int key_bits = 3 * bits + (BATCH ? set_bits_for(job.nsets) : 0);
        launch_sort_pairs(reinterpret_cast<uint32_t *>(job.rec.flag), job.rec.work,
                          reinterpret_cast<uint32_t *>(job.rec.wpos), job.rec.work2, job.rec.scnt, job.rec.scan_tmp,
                          job.rec.n_sort, job.rec.n_work, 2 * n_max, key_bits, st);
    }
    // launch shape (QSQ_LAUNCH word): workgroup size and a resident-lane
    // target per CU, capped by what the kernel's registers and LDS let stay
    // resident, so that every workgroup of the persistent launch runs from the
    // start (the first item of each lane is its global index)
    int lanes = job.o.launch & 15;
    const int wg_code = (job.o.launch >> 4) & 3, gather = (job.o.launch >> 6) & 7;
    const int wg = wg_code == 1 ? 64 : wg_code == 2 ? 128 : 256;
    const void *kern;
    size_t lds = 0;
    StepLoads loads = kLoadsDirect;
    constexpr bool cacheable = sizeof(T) == 4 && interp_order<MODE>() == 1 &&
                               (std::is_same<S, float>::value || std::is_same<S, Bf16>::value);
    if constexpr (cacheable && !BATCH) {
        // the cell caches address the node records with 32-bit byte offsets
        const uint64_t field_bytes = (uint64_t)node_bytes<S>() * job.g.n[0] * job.g.n[1] * job.g.n[2];
        const uint64_t brick_bytes = (uint64_t)node_bytes<S>() * 8 * ((job.g.n[0] + 1) / 2) *
                                     ((job.g.n[1] + 1) / 2) * ((job.g.n[2] + 1) / 2);
        const uint64_t limit = kCacheLimit;
        const bool fits = field_bytes < limit;
        // the direction records' variant keys cells by a 32-bit cell index
        const uint64_t ncells =
            (uint64_t)(job.g.n[0] - 1) * (uint64_t)(job.g.n[1] - 1) * (uint64_t)(job.g.n[2] - 1);
        const void *dirs_kern = nullptr;
        if constexpr (std::is_same<S, float>::value)
            if (gather == 6 && job.dirs && ncells < ((uint64_t)1 << 31))
                dirs_kern = trace_kernel<T, S, MODE, kGatherDirs, false>(euler);
        if (dirs_kern) {
            kern = dirs_kern;
            loads = kLoadsDirs;
            lds = CellDirs::kPlanes * wg * sizeof(float4);
        } else if (gather == 5 && job.bricks && brick_bytes < limit) {
            kern = trace_kernel<T, S, MODE, kGatherBricks, false>(euler);
            lds = (CellNodes::kPlanes + 2) * wg * sizeof(float4);
            loads = kLoadsBricks;
        } else if (gather == 4 && job.cells) {
            kern = trace_kernel<T, S, MODE, kGatherCells, false>(euler);
            loads = kLoadsCells;
        } else if ((gather == 3 || gather == 5 || gather == 6 || gather == 0) && fits) {
            kern = trace_kernel<T, S, MODE, kGatherRegs, false>(euler);
            lds = CellNodes::kPlanes * wg * sizeof(float4);
            loads = kLoadsRegs;
        } else if (gather == 2 && fits) {
            kern = trace_kernel<T, S, MODE, kGatherLds, false>(euler);
            loads = kLoadsLds;
            lds = kCachePlanes * wg * sizeof(float4);
        } else {
            kern = trace_kernel<T, S, MODE, kGatherDirect, false>(euler);
        }
    } else {
        (void)gather;
        kern = trace_kernel<T, S, MODE, kGatherDirect, BATCH>(euler);
    }
    // workgroups that stay resident; of a list that turns out to be spread (of
    // a trace) or short (of a volume), which only the device knows, the first `few`
    const int64_t resident = (int64_t)cus * resident_blocks(kern, wg, lds);
    auto cap_blocks = [&](bool spread, int64_t halves) {
        int units = lanes;   // (256 lanes a compute unit: one wave per SIMD)
        if (units == 0 && interp_order<MODE>() == 1) {
            StepCall c = step_call(job, sizeof(T) == 8, BATCH, n_max);
            c.spread = spread;
            c.halves = halves;
            units = auto_waves(c, loads);
        }
        const int64_t b = (int64_t)cus * (units ? units : 8) * (256 / wg);
        return b < resident ? b : resident;
    };
    const int64_t want = (2 * n_max + wg - 1) / wg;
    const int blocks = (int)(want < cap_blocks(false, 2 * n_max) ? want : cap_blocks(false, 2 * n_max));
    TraceJob js = job;
    const int64_t few = job.spatial_bits > 0 ? cap_blocks(true, 2 * n_max) : job.volume ? cap_blocks(false, kShortList) : blocks;
    js.few = few < blocks ? (int)few : blocks;
    js.few_from = job.spatial_bits > 0 ? spread_halves(n_max) : 2 * n_max;
    js.few_upto = job.volume ? kShortList : 0;
    const int nparts = (job.o.launch >> 9) & 1 ? kParts : 1;
    // few half-lines: four lanes each.  The count is known on the device
    // only, so where it may fall on either side both kernels are launched and
    // the one whose call it is not returns at once.
    const void *quad = nullptr;
    int qblocks = 0;
    {
        if (job.quad_max > 0) {
            quad = euler ? reinterpret_cast<const void *>(&k_trace_quad<T, S, MODE, BATCH, true>)
                         : reinterpret_cast<const void *>(&k_trace_quad<T, S, MODE, BATCH, false>);
            // at least the workgroups of one wave per SIMD, so that a short list can spread
            const int64_t full = (int64_t)cus * resident_blocks(quad, kQuadWg, 0);
            const int64_t need = (2 * n_max * 4 + kQuadWg - 1) / kQuadWg;
            qblocks = (int)(need < cus ? cus : need < full ? need : full);
        }
    }
    hipLaunchKernelGGL(k_part_counters, dim3(1), dim3(64), 0, st, js, blocks, wg, nparts, qblocks);
    const bool prof = profiling();
    void *tok = nullptr;
    if (prof) prof_begin(kProfStep, st, &tok);
    void *args[] = {&js};
    hipError_t le = hipSuccess;
    if (quad) le = hipLaunchKernel(quad, dim3(qblocks), dim3(kQuadWg), args, 0, st);
    if (le == hipSuccess && (!quad || 2 * n_max > job.quad_max))
        le = hipLaunchKernel(kern, dim3(blocks), dim3(wg), args, lds, st);
    if (prof) prof_end(tok, st);
    if (le != hipSuccess) return le;
    {
        // (the higher orders' stencils take 32-bit byte offsets; the launch
        // word has no say, so that it never changes a result)
        if ((interp_order<MODE>() == 1 || job.quad_ok) && n_max <= finish_seeds(step_call(job, sizeof(T) == 8, BATCH, n_max), interp_order<MODE>())) {
            const int64_t fb = (4 * n_max + 255) / 256;
            const int fblocks = (int)(fb < (int64_t)cus * 32 ? fb : (int64_t)cus * 32);
            if (prof) prof_begin(kProfLand, st, &tok);
            if (euler)
                hipLaunchKernelGGL((k_finish<S, MODE, BATCH, true>), dim3(fblocks), dim3(256), 0, st, job);
            else
                hipLaunchKernelGGL((k_finish<S, MODE, BATCH, false>), dim3(fblocks), dim3(256), 0, st, job);
            if (prof) prof_end(tok, st);
            return hipGetLastError();
        }
    }
    int64_t lb = (2 * n_max + 255) / 256;
    int lblocks = (int)(lb < (int64_t)cus * 16 ? lb : (int64_t)cus * 16);
    if (prof) prof_begin(kProfLand, st, &tok);
    TraceJob jl = job;
    if (job.spatial_bits > 0) {
        // list of the half-lines to land, in record order
        hipLaunchKernelGGL(k_land_flags, dim3(cblocks), dim3(256), 0, st, job);
        launch_scan_i32(job.rec.flag, job.rec.n_items, 2 * n_max, job.rec.scan_tmp, job.rec.wpos, job.rec.n_land, st);
        hipLaunchKernelGGL(k_land_compact, dim3(cblocks), dim3(256), 0, st, job);
    } else {
        // the unsorted work list is in record order already, and nearly all
        // of its lines leave the box
        jl.rec.work2 = job.rec.work;
        jl.rec.n_land = job.rec.n_work;
    }
    if (euler) {
        hipLaunchKernelGGL((k_land_euler<S, MODE, BATCH>), dim3(lblocks), dim3(256), 0, st, jl);
    } else {
        hipLaunchKernelGGL((k_land<S, MODE, BATCH>), dim3(lblocks), dim3(256), 0, st, jl);
        hipLaunchKernelGGL((k_land_final<S, MODE, BATCH>), dim3(lblocks), dim3(256), 0, st, jl);
    }
    if (prof) prof_end(tok, st);
    int64_t ab = (n_max + 255) / 256;
    int ablocks = (int)(ab < (int64_t)cus * 16 ? ab : (int64_t)cus * 16);
    if (prof) prof_begin(kProfAssemble, st, &tok);
    hipLaunchKernelGGL((k_assemble<S, MODE, BATCH>), dim3(ablocks), dim3(256), 0, st, job);
    if (prof) prof_end(tok, st);
    return hipGetLastError();
}

#ifdef QSQ_TRACE_HIGH_TU
// higher interpolation orders: one field per call, FP32 or FP64 node records;
// each (order, mode) pair is instantiated in a translation unit of its own,
// so that the build compiles them side by side
// general geometry: seed pass, stepping in physical coordinates, FP64
// landing, the shared Q assembly
template <typename T, typename S, int MODE>
static hipError_t launch_geo(const TraceJob &job, hipStream_t st)
{
    const int cus = device_cu_count();
    const int64_t n_max = job.n_dev ? job.rec.cap : job.n_host;
    if (n_max <= 0) return hipSuccess;
    auto blocks_of = [&](int64_t items) {
        const int64_t b = (items + 255) / 256;
        return (int)(b < (int64_t)cus * 16 ? b : (int64_t)cus * 16);
    };
    hipLaunchKernelGGL((k_seed_pass<S, MODE, false>), dim3(blocks_of(n_max)), dim3(256), 0, st, job);
    launch_scan_i32(job.rec.flag, job.rec.n_items, 2 * n_max, job.rec.scan_tmp, job.rec.wpos, job.rec.n_work, st);
    hipLaunchKernelGGL(k_compact, dim3(blocks_of(2 * n_max)), dim3(256), 0, st, job);
    TraceJob jq = job;
    jq.quad_max = INT64_MAX;
    jq.simds = 4 * cus;
    const void *kern = reinterpret_cast<const void *>(&k_trace_geo<T, S, MODE>);
    const int64_t full = (int64_t)cus * resident_blocks(kern, kQuadWg, 0);
    const int64_t need = (2 * n_max * 4 + kQuadWg - 1) / kQuadWg;
    const int qblocks = (int)(need < cus ? cus : need < full ? need : full);
    hipLaunchKernelGGL(k_part_counters, dim3(1), dim3(64), 0, st, jq, 0, 0, 1, qblocks);
    const bool prof = profiling();
    void *tok = nullptr;
    if (prof) prof_begin(kProfStep, st, &tok);
    hipLaunchKernelGGL((k_trace_geo<T, S, MODE>), dim3(qblocks), dim3(kQuadWg), 0, st, jq);
    if (prof) prof_end(tok, st);
    if (prof) prof_begin(kProfLand, st, &tok);
    hipLaunchKernelGGL(k_land_flags, dim3(blocks_of(2 * n_max)), dim3(256), 0, st, job);
    launch_scan_i32(job.rec.flag, job.rec.n_items, 2 * n_max, job.rec.scan_tmp, job.rec.wpos, job.rec.n_land, st);
    hipLaunchKernelGGL(k_land_compact, dim3(blocks_of(2 * n_max)), dim3(256), 0, st, job);
    hipLaunchKernelGGL((k_land_geo<S, MODE>), dim3(blocks_of(4 * 2 * n_max)), dim3(kQuadWg), 0, st, job);
    if (prof) prof_end(tok, st);
    if (prof) prof_begin(kProfAssemble, st, &tok);
    hipLaunchKernelGGL((k_assemble<S, MODE, false>), dim3(blocks_of(n_max)), dim3(256), 0, st, job);
    if (prof) prof_end(tok, st);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_trace_mode(const TraceJob &job, int step_dtype, hipStream_t st)
{
    const bool f32 = step_dtype == QSQ_F32;
    if constexpr (geo_mode<MODE>()) {
        if (job.storage == QSQ_F32)
            return f32 ? launch_geo<float, float, MODE>(job, st) : launch_geo<double, float, MODE>(job, st);
        if (job.storage == QSQ_F64)
            return f32 ? launch_geo<float, double, MODE>(job, st) : launch_geo<double, double, MODE>(job, st);
        return hipErrorNotSupported;
    } else {
        if (job.storage == QSQ_F32)
            return f32 ? launch_typed<float, float, MODE, false>(job, st)
                       : launch_typed<double, float, MODE, false>(job, st);
        if (job.storage == QSQ_F64)
            return f32 ? launch_typed<float, double, MODE, false>(job, st)
                       : launch_typed<double, double, MODE, false>(job, st);
        return hipErrorNotSupported;
    }
}

template hipError_t launch_trace_mode<QSQ_TRACE_HIGH_MODE>(const TraceJob &job, int step_dtype, hipStream_t st);
#else

template <bool BATCH>
static hipError_t dispatch(const TraceJob &job, int step_dtype, hipStream_t st)
{
    const bool f32 = step_dtype == QSQ_F32;
    const bool paper = (job.mode & 1) == QSQ_INTERP_PAPER;
    constexpr int P = QSQ_INTERP_PAPER, N = QSQ_INTERP_NORMALIZE;
    if (job.mode > 1) {
        // higher interpolation orders: one field per call
        if constexpr (BATCH) {
            return hipErrorNotSupported;
        } else {
            // job.mode = interpolation mode | (order - 1) << 1
            switch (job.mode) {
            case 2: return launch_trace_mode<2>(job, step_dtype, st);
            case 3: return launch_trace_mode<3>(job, step_dtype, st);
            case 4: return launch_trace_mode<4>(job, step_dtype, st);
            case 5: return launch_trace_mode<5>(job, step_dtype, st);
            case 8: return launch_trace_mode<8>(job, step_dtype, st);
            case 9: return launch_trace_mode<9>(job, step_dtype, st);
            default: return hipErrorNotSupported;
            }
        }
    }
    if (job.storage == QSQ_BF16) {
        if (f32) return paper ? launch_typed<float, Bf16, P, BATCH>(job, st) : launch_typed<float, Bf16, N, BATCH>(job, st);
        return paper ? launch_typed<double, Bf16, P, BATCH>(job, st) : launch_typed<double, Bf16, N, BATCH>(job, st);
    }
    if (job.storage == QSQ_F32) {
        if (f32) return paper ? launch_typed<float, float, P, BATCH>(job, st) : launch_typed<float, float, N, BATCH>(job, st);
        return paper ? launch_typed<double, float, P, BATCH>(job, st) : launch_typed<double, float, N, BATCH>(job, st);
    }
    if (f32) return paper ? launch_typed<float, double, P, BATCH>(job, st) : launch_typed<float, double, N, BATCH>(job, st);
    return paper ? launch_typed<double, double, P, BATCH>(job, st) : launch_typed<double, double, N, BATCH>(job, st);
}

// four-lane kernels: records addressed with 32-bit byte offsets, their keys
// formed by 24-bit products
static bool quad_addressable(const Geom &g, int storage)
{
    const uint64_t rec = storage == QSQ_F64 ? 32 : storage == QSQ_F32 ? 16 : 8;
    const uint64_t xy = (uint64_t)g.n[0] * (uint64_t)g.n[1];
    return xy < ((uint64_t)1 << 23) && (uint64_t)g.n[2] < ((uint64_t)1 << 23) && xy * (uint64_t)g.n[2] * rec < kCacheLimit;
}

// largest work list that the four-lane kernel takes under an automatic gather
// (0: none; a named gather always gets the one-lane kernel)
static int64_t quad_limit(const TraceJob &job, const Geom &g, double h_init, double h_max, bool step64, bool batch, int order)
{
    if (!quad_addressable(g, job.storage)) return 0;
    TraceJob j = job;
    j.g = g;
    const StepCall c = step_call(j, step64, batch, 0);
    const double edge = fmax(fmax(g.hi[0] - g.lo[0], g.hi[1] - g.lo[1]), g.hi[2] - g.lo[2]);
    return quad_list(c, edge / (c.euler ? h_init : h_max), order);
}

hipError_t launch_trace(const TraceJob &job, int step_dtype, hipStream_t st)
{
    TraceJob j = job;
    j.simds = 4 * device_cu_count();
    j.quad_ok = quad_addressable(job.g, job.storage);
    j.quad_max = 0;
    if (((job.o.launch >> 6) & 7) == 0 && job.mode < 8)
        j.quad_max = quad_limit(job, job.g, job.o.h_init, job.o.h_max, step_dtype == QSQ_F64, false, ((job.mode >> 1) & 3) + 1);
    return dispatch<false>(j, step_dtype, st);
}

// The set table travels in kernel arguments, a few entries per launch, so
// that the whole batched call is plain kernel launches (capturable in a graph,
// no host buffer that must outlive the call).
constexpr int kSetsPerPut = 6;
struct SetChunk {
    SetDesc d[kSetsPerPut];
    int first, count;
};

__global__ void k_put_sets(SetDesc *table, SetChunk c)
{
    const int k = (int)threadIdx.x;
    if (k < c.count) table[c.first + k] = c.d[k];
}

hipError_t launch_trace_batch(const TraceJob &job, const SetDesc *host_sets, int nsets, int step_dtype,
                              hipStream_t st)
{
    SetDesc *table = const_cast<SetDesc *>(job.sets);
    for (int first = 0; first < nsets; first += kSetsPerPut) {
        SetChunk c{};
        c.first = first;
        c.count = nsets - first < kSetsPerPut ? nsets - first : kSetsPerPut;
        for (int k = 0; k < c.count; ++k) c.d[k] = host_sets[first + k];
        hipLaunchKernelGGL(k_put_sets, dim3(1), dim3(64), 0, st, table, c);
    }
    TraceJob j = job;
    j.simds = 4 * device_cu_count();
    j.quad_max = 0;
    if (((job.o.launch >> 6) & 7) == 0) {
        j.quad_max = (int64_t)1 << 30;
        for (int k = 0; k < nsets; ++k) {
            const SetDesc &d = host_sets[k];
            const int64_t q = quad_limit(job, d.g, d.h_init, d.h_max, step_dtype == QSQ_F64, true, 1);
            if (q < j.quad_max) j.quad_max = q;
        }
    }
    return dispatch<true>(j, step_dtype, st);
}

#endif  // QSQ_TRACE_HIGH_TU

}  // namespace qsq
