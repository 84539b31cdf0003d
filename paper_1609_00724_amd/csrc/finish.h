// End of a trace: FP64 landing of both half-lines of a seed and Q (eq. 10-11)
// in one kernel, eight lanes per seed.  A quad (four adjacent lanes) takes one
// half-line, lane c of it component c of the position and the deviations; the
// two quads of a seed then exchange the few scalars that eq. (11) combines.
// A half-line that left the box is landed by a root find on the position alone
// (eq. (1) does not involve the deviations), one full step to the root, and
// the snap onto the face.  Included by trace.hip after quad.h.
#pragma once

// the lane's axis of a grid, FP64
struct FinAxis {
    int n, nx, ny;
    double o, ih, lo, hi;
    double ihx, ihy, ihz;
};

__device__ __forceinline__ FinAxis fin_axis(const Geom &g, int c)
{
    FinAxis a;
    a.n = c == 0 ? g.n[0] : c == 1 ? g.n[1] : g.n[2];
    a.nx = g.n[0];
    a.ny = g.n[1];
    a.o = c == 0 ? g.o[0] : c == 1 ? g.o[1] : g.o[2];
    a.ih = c == 0 ? g.ih[0] : c == 1 ? g.ih[1] : g.ih[2];
    a.lo = c == 0 ? g.lo[0] : c == 1 ? g.lo[1] : g.lo[2];
    a.hi = c == 0 ? g.hi[0] : c == 1 ? g.hi[1] : g.hi[2];
    a.ihx = g.ih[0];
    a.ihy = g.ih[1];
    a.ihz = g.ih[2];
    return a;
}

// corner values (one component of the records) of the cell the quad evaluated last
struct FinCell {
    int64_t key;
    double v[8];
};

// fractions of every axis at grid-unit reference ib plus offset q (the lane's
// axis), corner values of the cell in `cell`
template <typename S>
__device__ __forceinline__ void fin_corners(const char *comp, const FinAxis &a, int ib, double q, double t[3],
                                            FinCell &cell)
{
    constexpr int RB = 4 * value_bytes<S>();
    int ci;
    double tl;
    cell_of(ib, q, a.n, ci, tl);
    t[0] = quad_get<0>(tl);
    t[1] = quad_get<1>(tl);
    t[2] = quad_get<2>(tl);
    const int64_t key = ((int64_t)quad_get<2>(ci) * a.ny + quad_get<1>(ci)) * a.nx + quad_get<0>(ci);
    if (key != cell.key) {
        cell.key = key;
        const int64_t dy = (int64_t)a.nx * RB, dz = dy * a.ny;
        const char *p = comp + key * RB;
        cell.v[0] = quad_load<double, S>(p);
        cell.v[1] = quad_load<double, S>(p + RB);
        cell.v[2] = quad_load<double, S>(p + dy);
        cell.v[3] = quad_load<double, S>(p + dy + RB);
        cell.v[4] = quad_load<double, S>(p + dz);
        cell.v[5] = quad_load<double, S>(p + dz + RB);
        cell.v[6] = quad_load<double, S>(p + dz + dy);
        cell.v[7] = quad_load<double, S>(p + dz + dy + RB);
    }
}

__device__ __forceinline__ double fin_lerp(const FinCell &c, const double t[3])
{
    return lerp_val<double>(c.v[0], c.v[1], c.v[2], c.v[3], c.v[4], c.v[5], c.v[6], c.v[7], t[0], t[1], t[2]);
}

// value and gradient of record component comp by a higher order's stencil (a
// call: inlined at its twenty-odd places the cubic's 64 nodes outgrow the
// instruction cache)
struct FinStencil {
    double val, dx, dy, dz;
};
template <typename S, int MODE>
__device__ __attribute__((noinline)) double fin_stencil_value(const char *recs, int n, int nx, int ny, int c3, int comp,
                                                              int ib, double q)
{
    constexpr uint32_t RB = 4 * value_bytes<S>();
    int ci;
    double t, val, dx, dy, dz;
    cell_of(ib, q, n, ci, t);
    const uint32_t sy = RB * (uint32_t)nx;
    quad_stencil<double, S, interp_order<MODE>() + 1>(recs, n, sy, sy * (uint32_t)ny, c3, comp, ci, t, val, dx, dy, dz);
    return val;
}
template <typename S, int MODE>
__device__ __attribute__((noinline)) FinStencil fin_stencil_of(const char *recs, int n, int nx, int ny, int c3, int comp,
                                                               int ib, double q)
{
    constexpr uint32_t RB = 4 * value_bytes<S>();
    int ci;
    double t;
    cell_of(ib, q, n, ci, t);
    const uint32_t sy = RB * (uint32_t)nx;
    FinStencil r;
    quad_stencil<double, S, interp_order<MODE>() + 1>(recs, n, sy, sy * (uint32_t)ny, c3, comp, ci, t, r.val, r.dx, r.dy,
                                                      r.dz);
    return r;
}
template <typename S, int MODE>
__device__ __forceinline__ void fin_stencil(const char *recs, const FinAxis &a, int c3, int comp, int ib, double q,
                                            double &val, double &dx, double &dy, double &dz)
{
    const FinStencil r = fin_stencil_of<S, MODE>(recs, a.n, a.nx, a.ny, c3, comp, ib, q);
    val = r.val;
    dx = r.dx;
    dy = r.dy;
    dz = r.dz;
}

// 1 / |v| over the quad's three components (0 for |v| <= 1e-300); bn = |v|
template <typename S, int MODE>
__device__ __forceinline__ double fin_inverse(double val, double &bn)
{
    const double v0 = quad_get<0>(val), v1 = quad_get<1>(val), v2 = quad_get<2>(val);
    bn = sqrt(norm2<double, S, MODE>(v0, v1, v2));
    return bn > 1e-300 ? 1.0 / bn : 0.0;
}

// the lane's component of the direction u
template <typename S, int MODE>
__device__ __forceinline__ double fin_u(const char *recs, const FinAxis &a, int c3, int ib, double q, FinCell &cell)
{
    double bn, val;
    if constexpr (interp_order<MODE>() > 1) {
        val = fin_stencil_value<S, MODE>(recs, a.n, a.nx, a.ny, c3, c3 == 3 ? 2 : c3, ib, q);
    } else {
        double t[3];
        fin_corners<S>(recs + (c3 == 3 ? 2 : c3) * value_bytes<S>(), a, ib, q, t, cell);
        val = fin_lerp(cell, t);
    }
    return normalize_first<MODE>() ? val : val * fin_inverse<S, MODE>(val, bn);
}

// right-hand side for the lane's components: sigma (u, J d1, J d2)
template <typename S, int MODE>
__device__ __forceinline__ void fin_rhs(const char *recs, const FinAxis &a, int c3, int ib, double q, double sigma,
                                        double d1, double d2, double k[3], FinCell &cell)
{
    double val, dx, dy, dz, G[3], u;
    if constexpr (interp_order<MODE>() > 1) {
        fin_stencil<S, MODE>(recs, a, c3, c3 == 3 ? 2 : c3, ib, q, val, dx, dy, dz);
    } else {
        double t[3];
        fin_corners<S>(recs + (c3 == 3 ? 2 : c3) * value_bytes<S>(), a, ib, q, t, cell);
        lerp_tree<double>(cell.v[0], cell.v[1], cell.v[2], cell.v[3], cell.v[4], cell.v[5], cell.v[6], cell.v[7], t[0],
                          t[1], t[2], val, dx, dy, dz);
    }
    const double Gb[3] = {dx * a.ihx, dy * a.ihy, dz * a.ihz};
    if (normalize_first<MODE>()) {
        u = val;
#pragma unroll
        for (int j = 0; j < 3; ++j) G[j] = Gb[j];
    } else {
        double bn;
        const double inv = fin_inverse<S, MODE>(val, bn);
        u = val * inv;
        const double u0 = quad_get<0>(u), u1 = quad_get<1>(u), u2 = quad_get<2>(u);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const double ug = along(u0, u1, u2, quad_get<0>(Gb[j]), quad_get<1>(Gb[j]), quad_get<2>(Gb[j]));
            G[j] = fma(-u, ug, Gb[j]) * inv;
        }
    }
    k[0] = sigma * u;
    k[1] = sigma * jdot(G[0], G[1], G[2], quad_get<0>(d1), quad_get<1>(d1), quad_get<2>(d1));
    k[2] = sigma * jdot(G[0], G[1], G[2], quad_get<0>(d2), quad_get<1>(d2), quad_get<2>(d2));
}

// grid-unit reference of coordinate x along the lane's axis
__device__ __forceinline__ void fin_ref(const FinAxis &a, double x, int &ib, double &fb)
{
    const double xg = (x - a.o) * a.ih, fl = floor(fmin(fmax(xg, -1e9), 1e9));
    ib = (int)fl;
    fb = fma(x - a.o, a.ih, -fl);
}

// the same as field_at_x forms it (the product rounded before the subtraction)
__device__ __forceinline__ void fin_point(const FinAxis &a, double x, int &ib, double &q)
{
    const double s = fmin(fmax((x - a.o) * a.ih, -1e9), 1e9), fl = floor(s);
    ib = (int)fl;
    q = s - fl;
}

#define QSQ_FIN_STAGES(STAGE)                                \
    STAGE(1, ck::a21)                                        \
    STAGE(2, ck::a31, ck::a32)                               \
    STAGE(3, ck::a41, ck::a42, ck::a43)                      \
    STAGE(4, ck::a51, ck::a52, ck::a53, ck::a54)             \
    STAGE(5, ck::a61, ck::a62, ck::a63, ck::a64, ck::a65)

// the lane's position component at the end of a Cash-Karp step of length h
// from x, whose first-stage slope is k0
template <typename S, int MODE>
__device__ __forceinline__ double fin_step_x(const char *recs, const FinAxis &a, int c3, int ib, double fb, double sigma, double x,
                                             double h, double k0, FinCell &cell)
{
    double K[6];
    K[0] = k0;
#define QSQ_FSTAGE(ST, ...)                                                                         \
    {                                                                                               \
        const double c_[] = {__VA_ARGS__};                                                          \
        double ax = 0;                                                                              \
        _Pragma("unroll") for (int j = 0; j < ST; ++j) ax = fma(c_[j], K[j], ax);                   \
        K[ST] = sigma * fin_u<S, MODE>(recs, a, c3, ib, fma(h * ax, a.ih, fb), cell);               \
    }
    QSQ_FIN_STAGES(QSQ_FSTAGE)
#undef QSQ_FSTAGE
    return fma(h, ck_b5(K[0], K[2], K[3], K[5]), x);
}

// signed distance beyond face f of the quad's point, from every lane's
// distances beyond its axis' two faces
__device__ __forceinline__ double fin_gap(double glo, double ghi, int f)
{
    const double v = (f & 1) ? ghi : glo;
    const double g0 = quad_get<0>(v), g1 = quad_get<1>(v), g2 = quad_get<2>(v);
    return f < 2 ? g0 : f < 4 ? g1 : g2;
}

// Landing of one half-line: the step from (x, d1, d2) over hs, whose end lies
// outside the box, is cut to the length whose 5th-order end lies on the first
// face crossed (the smallest such length; exact ties keep the lower face).
// Regula falsi with the Anderson-Bjorck factor from a quadratic model's root.
// Returns the length and the face; x, d1, d2 become the landed state.
template <typename S, int MODE, bool EULER>
__device__ __forceinline__ double fin_land(const char *recs, const FinAxis &a, int c3, double gtol, double sigma, double hs,
                                           double &x, double &d1, double &d2, int &face, FinCell &cell)
{
    const int c = c3 == 3 ? 2 : c3;
    int ib;
    double fb;
    if (EULER)
        fin_point(a, x, ib, fb);
    else
        fin_ref(a, x, ib, fb);
    double Kx[6], K1[6], K2[6], k[3];
    fin_rhs<S, MODE>(recs, a, c3, ib, fb, sigma, d1, d2, k, cell);
    Kx[0] = k[0];
    K1[0] = k[1];
    K2[0] = k[2];
    double best = INFINITY, gmax = -INFINITY;
    int fnear = 0;
    unsigned crossed = 0;
    face = -1;
    const double xe = EULER ? fma(hs, Kx[0], x) : fin_step_x<S, MODE>(recs, a, c3, ib, fb, sigma, x, hs, Kx[0], cell);
    const double elo = a.lo - xe, ehi = xe - a.hi;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const double ge = fin_gap(elo, ehi, f);
        if (ge > gmax) {
            gmax = ge;
            fnear = f;
        }
        if (ge > 0.0) crossed |= 1u << f;
    }
    // the faces crossed, lowest first
    while (crossed) {
        const int f = __ffs(crossed) - 1;
        crossed &= crossed - 1;
        double hf;
        if constexpr (EULER) {
            // the end of an Euler step moves linearly with its length
            const double wall = (f & 1) ? a.hi : a.lo, h = (wall - x) / Kx[0];
            const double h0 = quad_get<0>(h), h1 = quad_get<1>(h), h2 = quad_get<2>(h);
            hf = f < 2 ? h0 : f < 4 ? h1 : h2;
            hf = hf < 0.0 ? 0.0 : (hf > hs ? hs : hf);
        } else {
            double lo = 0.0, hi = hs, ga = fin_gap(a.lo - x, x - a.hi, f), gb = fin_gap(elo, ehi, f);
            if (ga >= 0.0) {
                hf = 0.0;
            } else {
                const double v0 = quad_get<0>(Kx[0]), v1 = quad_get<1>(Kx[0]), v2 = quad_get<2>(Kx[0]);
                const double v = f < 2 ? v0 : f < 4 ? v1 : v2;
                const double c0 = landing_guess(ga, (f & 1) ? v : -v, gb, hs);
                int side = 0;
                hf = -1.0;
                for (int it = 0; it < 200; ++it) {
                    const double h = it == 0 ? c0 : landing_secant(lo, ga, hi, gb);
                    double xh = x;
                    if (h != 0.0) xh = fin_step_x<S, MODE>(recs, a, c3, ib, fb, sigma, x, h, Kx[0], cell);
                    const double gc = fin_gap(a.lo - xh, xh - a.hi, f);
                    if (fabs(gc) <= gtol) {
                        hf = h;
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
                        hi = h;
                        gb = gc;
                        side = 1;
                    } else {
                        if (side == -1) {
                            const double m = 1.0 - gc / ga;
                            gb *= m > 0.0 ? m : 0.5;
                        }
                        lo = h;
                        ga = gc;
                        side = -1;
                    }
                    if (hi - lo <= 1e-15 * hs) break;
                }
                if (hf < 0.0) hf = ga > -gb ? lo : hi;
            }
        }
        if (hf < best) {
            best = hf;
            face = f;
        }
    }
    if (face < 0) {
        // the FP64 re-solve ends inside (the trial end was within rounding
        // of a face): land on the nearest face at the full step
        face = fnear;
        best = hs;
    }
    if constexpr (EULER) {
        x = fma(best, Kx[0], x);
        d1 = fma(best, K1[0], d1);
        d2 = fma(best, K2[0], d2);
    } else if (best > 0.0) {
#define QSQ_FSTAGE(ST, ...)                                                                                        \
    {                                                                                                              \
        const double c_[] = {__VA_ARGS__};                                                                         \
        double ax = 0, a1 = 0, a2 = 0;                                                                             \
        _Pragma("unroll") for (int j = 0; j < ST; ++j)                                                             \
        {                                                                                                          \
            ax = fma(c_[j], Kx[j], ax);                                                                            \
            a1 = fma(c_[j], K1[j], a1);                                                                            \
            a2 = fma(c_[j], K2[j], a2);                                                                            \
        }                                                                                                          \
        fin_rhs<S, MODE>(recs, a, c3, ib, fma(best * ax, a.ih, fb), sigma, fma(best, a1, d1), fma(best, a2, d2), k, \
                         cell);                                                                                    \
        Kx[ST] = k[0];                                                                                             \
        K1[ST] = k[1];                                                                                             \
        K2[ST] = k[2];                                                                                             \
    }
        QSQ_FIN_STAGES(QSQ_FSTAGE)
#undef QSQ_FSTAGE
        x = fma(best, ck_b5(Kx[0], Kx[2], Kx[3], Kx[5]), x);
        d1 = fma(best, ck_b5(K1[0], K1[2], K1[3], K1[5]), d1);
        d2 = fma(best, ck_b5(K2[0], K2[2], K2[3], K2[5]), d2);
    }
    if (c == (face >> 1)) x = (face & 1) ? a.hi : a.lo;
    return best;
}
#undef QSQ_FIN_STAGES

// u (not renormalised; the lane's component) and |B| at coordinate x: the
// fourth record component, which lane 3 takes (PAPER), or |interpolated B|
template <typename S, int MODE>
__device__ __forceinline__ double fin_value(const char *recs, const FinAxis &a, int c3, double x, double &mag)
{
    int ib;
    double fb, val;
    fin_point(a, x, ib, fb);
    if constexpr (interp_order<MODE>() > 1) {
        val = fin_stencil_value<S, MODE>(recs, a.n, a.nx, a.ny, c3, c3, ib, fb);
    } else {
        FinCell cell;
        double t[3];
        cell.key = -1;
        fin_corners<S>(recs + c3 * value_bytes<S>(), a, ib, fb, t, cell);
        val = fin_lerp(cell, t);
    }
    if (normalize_first<MODE>()) {
        mag = quad_get<3>(val);
        return val;
    }
    const double inv = fin_inverse<S, MODE>(val, mag);
    return val * inv;
}

// a0 b0 + a1 b1 + a2 b2 over the quad's components
__device__ __forceinline__ double quad_dot(double a, double b)
{
    return fma(quad_get<2>(a), quad_get<2>(b), fma(quad_get<0>(a), quad_get<0>(b), quad_get<1>(a * b)));
}

__device__ __forceinline__ int quad_perm_i(int v, bool next)
{
    return next ? __builtin_amdgcn_mov_dpp(v, 0xc9, 0xf, 0xf, true) : __builtin_amdgcn_mov_dpp(v, 0xd2, 0xf, 0xf, true);
}
// component c + 1 (next) or c + 2 (cyclic) of the quad's vector
__device__ __forceinline__ double quad_turn(double v, bool next)
{
    return __hiloint2double(quad_perm_i(__double2hiint(v), next), quad_perm_i(__double2loint(v), next));
}

__device__ __forceinline__ double quad_cross_len(double a, double b)
{
    const double x = fma(quad_turn(a, true), quad_turn(b, false), -(quad_turn(a, false) * quad_turn(b, true)));
    return sqrt(quad_dot(x, x));
}

// |a|^2, |b|^2, a . b and |a x b| of a half-line's end vectors, and eq. (11)'s
// bracket with the other half's (shared by lanes 4 apart)
struct EndDots {
    double aa, bb, ab, area;
};
__device__ __forceinline__ EndDots end_dots(double a, double b)
{
    return {quad_dot(a, a), quad_dot(b, b), quad_dot(a, b), quad_cross_len(a, b)};
}
__device__ __forceinline__ double end_bracket(const EndDots &e, double &areas)
{
    const double aa = __shfl_xor(e.aa, 4), bb = __shfl_xor(e.bb, 4), ab = __shfl_xor(e.ab, 4);
    areas = e.area * __shfl_xor(e.area, 4);
    return fma(-2.0 * ab, e.ab, fma(e.aa, bb, aa * e.bb));
}

// A wave takes 16 seeds.  First its quads land the half-lines that left the
// box, 16 at a time in record order (seeds on the bottom face have one such
// half each, and no quad idles for the other), then eight lanes per seed form
// Q from the records, which the wave itself has just written.  Bound by FP64
// issue and by the latency of its gathers (about 24 evaluations of 8 corners
// per landed half-line; a quad's lanes read one record together).
template <typename S, int MODE, bool BATCH, bool EULER>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(interp_order<MODE>() > 1 ? 2 : 1))) k_finish(TraceJob job)
{
    const int64_t n = seed_count(job), P = 2 * job.rec.cap;
    const int lane = (int)(threadIdx.x & 63), c3 = lane & 3, c = c3 == 3 ? 2 : c3;
    FinAxis a = fin_axis(job.g, c);
    const char *recs = static_cast<const char *>(job.nodes);
    double gtol = job.o.gtol;
    for (int64_t i0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 16; i0 < n;
         i0 += (((int64_t)gridDim.x * blockDim.x) >> 6) * 16) {
        // lane k < 32: half k / 16 of seed i0 + k % 16
        const bool mine = lane < 32 && i0 + (lane & 15) < n;
        uint64_t left = __ballot(mine && job.rec.status[(lane >> 4) * job.rec.cap + i0 + (lane & 15)] == kPendingLand);
        while (left) {
            // the quad's pending half-line: the (lane / 4)-th of the wave's
            uint64_t m = left;
            for (int k = 0; k < (lane >> 2); ++k) m &= m - 1;
            if (m) {
                const int h = __ffsll((unsigned long long)m) - 1;
                const int64_t i = i0 + (h & 15), r = (h >> 4) * job.rec.cap + i;
                if constexpr (BATCH) {
                    const SetDesc &sd = job.sets[job.set_of[i]];
                    a = fin_axis(sd.g, c);
                    recs = in_global<char>(sd.nodes);
                    gtol = sd.gtol;
                }
                double x = job.rec.y[c * P + r], d1 = job.rec.y[(3 + c) * P + r], d2 = job.rec.y[(6 + c) * P + r];
                const double s = job.rec.s[r];
                int face;
                FinCell cell;
                cell.key = -1;
                const double cut = fin_land<S, MODE, EULER>(recs, a, c3, gtol, h >> 4 ? -1.0 : 1.0, job.rec.h[r], x,
                                                            d1, d2, face, cell);
                if (c3 < 3) {
                    job.rec.y[c * P + r] = x;
                    job.rec.y[(3 + c) * P + r] = d1;
                    job.rec.y[(6 + c) * P + r] = d2;
                } else {
                    job.rec.s[r] = s + cut;
                    job.rec.status[r] = face;
                }
            }
            for (int k = 0; k < 16; ++k) left &= left - 1;
        }
        // what the quads wrote is read below by other lanes of the wave
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const int half = (lane >> 2) & 1;
        for (int64_t i = i0 + (lane >> 3); i < i0 + 16 && i < n; i += 8) {
            const int64_t r = half * job.rec.cap + i;
            const double *seeds = job.seeds;
            int64_t ss = job.seed_stride, os = job.out_stride, li = i;
            double *o_fp = half ? job.fp_bwd : job.fp_fwd, *o_fll = job.fll;
            double *o_qp = job.q_perp, *o_qd = job.q_det, *o_qf = job.q_fp;
            int32_t *o_st = job.status, *o_steps = job.steps;
            if constexpr (BATCH) {
                const SetDesc &sd = job.sets[job.set_of[i]];
                a = fin_axis(sd.g, c);
                recs = in_global<char>(sd.nodes);
                seeds = sd.seeds;
                ss = os = sd.n;
                li = i - sd.off;
                o_fp = half ? sd.fp_bwd : sd.fp_fwd;
                o_fll = sd.fll;
                o_qp = sd.q_perp;
                o_qd = sd.q_det;
                o_qf = sd.q_fp;
                o_st = sd.status;
                o_steps = sd.steps;
            }
            const int st = job.rec.status[r];
            const double x = job.rec.y[c * P + r], d1 = job.rec.y[(3 + c) * P + r], d2 = job.rec.y[(6 + c) * P + r];
            const double s = job.rec.s[r];
            const int att = job.rec.attempts[r];
            const int st2 = __shfl_xor(st, 4), att2 = __shfl_xor(att, 4);
            const double s2 = __shfl_xor(s, 4);
            const int stF = half ? st2 : st, stB = half ? st : st2;
            const bool open = !(stF == QSQ_END_ZLO && stB == QSQ_END_ZLO);
            const bool first = (lane & 7) == 0;
            if (first) {
                o_st[li] = (stF & 0xff) | ((stB & 0xff) << 8) | (open ? QSQ_STATUS_OPEN : 0);
                if (o_fll) o_fll[li] = s + s2;
                if (o_steps) {
                    if (job.steps_sum) {
                        o_steps[li] = att + att2;
                    } else {
                        o_steps[li] = att;
                        o_steps[os + li] = att2;
                    }
                }
            }
            if (o_fp && c3 < 3) o_fp[c * os + li] = x;
            double qp = NAN, qd = NAN, qf = NAN;
            const bool defF = stF >= QSQ_END_XLO && stF <= QSQ_END_MAX_STEPS;
            const bool defB = stB >= QSQ_END_XLO && stB <= QSQ_END_MAX_STEPS;
            const bool skip = (job.o.flags & QSQ_FLAG_SKIP_OPEN) && open;
            if (defF && defB && !skip) {
                double mag, mag0;
                const double v = fin_value<S, MODE>(recs, a, c3, x, mag);
                fin_value<S, MODE>(recs, a, c3, seeds[c * ss + li], mag0);
                const double u = v / sqrt(quad_dot(v, v));
                // perpendicular parts of the deviations (Sect. 3.5)
                const EndDots ep = end_dots(less_along(d1, u, quad_dot(u, d1)), less_along(d2, u, quad_dot(u, d2)));
                double areas;
                const double br = end_bracket(ep, areas);
                qp = mag * __shfl_xor(mag, 4) / (mag0 * mag0) * br;   // eq. (11)
                qd = br / areas;
                if (stF <= QSQ_END_ZHI && stB <= QSQ_END_ZHI) {
                    // slide the deviations along the line into the exit-face planes
                    const int d = st >> 1;
                    auto pick = [&](double w) {
                        const double w0 = quad_get<0>(w), w1 = quad_get<1>(w), w2 = quad_get<2>(w);
                        return d == 0 ? w0 : d == 1 ? w1 : w2;
                    };
                    const double vd = pick(v), r1 = pick(d1) / vd, r2 = pick(d2) / vd;
                    const EndDots ef = end_dots(less_along(d1, v, r1), less_along(d2, v, r2));
                    const double bf = end_bracket(ef, areas);
                    qf = bf / areas;
                }
            }
            if (first) {
                if (o_qp) o_qp[li] = qp;
                if (o_qd) o_qd[li] = qd;
                if (o_qf) o_qf[li] = qf;
            }
        }
    }
}
