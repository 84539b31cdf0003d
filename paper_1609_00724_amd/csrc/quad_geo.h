// General geometry (spherical coordinates, rectilinear axes) with four lanes per
// half-line: lane c of a quad holds axis c of the position and component c of
// the deviations, searches its own axis for the cell, evaluates its own field
// component and carries its own metric factor (lane 3 repeats lane 2).  The
// work of a step is FP64 along each axis (cell, latitude cosine, metric
// division), which one lane per line did three times over with its stage
// slopes in scratch memory: 40 000 half-lines of a 97 x 97 x 65 wedge at a
// 1-cell cap (279 attempts the longest) step in 1.58 ms against 5.2, and land
// in 0.125 ms against 0.92.  Bound by the serial chain of the longest line
// (5.7 us an attempt: six cosines, a power and six dependent gathers).
// Included by trace.hip after quad.h.
#pragma once

// the lane's axis of a general-geometry grid
struct GeoAxis {
    int n, nx, ny;        // nodes along the axis; of the record rows
    const double *X;      // node coordinates (null: uniform)
    double o, h, ih, rh;  // origin, spacing, the grid's 1 / spacing and 1.0 / spacing
    double lo, hi;
    bool sphere;
};

__device__ __forceinline__ GeoAxis geo_axis(const Geom &g, int c)
{
    GeoAxis a;
    a.n = c == 0 ? g.n[0] : c == 1 ? g.n[1] : g.n[2];
    a.nx = g.n[0];
    a.ny = g.n[1];
    a.X = c == 0 ? g.coord[0] : c == 1 ? g.coord[1] : g.coord[2];
    a.o = c == 0 ? g.o[0] : c == 1 ? g.o[1] : g.o[2];
    a.h = c == 0 ? g.h[0] : c == 1 ? g.h[1] : g.h[2];
    a.ih = c == 0 ? g.ih[0] : c == 1 ? g.ih[1] : g.ih[2];
    a.rh = 1.0 / a.h;
    a.lo = c == 0 ? g.lo[0] : c == 1 ? g.lo[1] : g.lo[2];
    a.hi = c == 0 ? g.hi[0] : c == 1 ? g.hi[1] : g.hi[2];
    a.sphere = g.geometry == QSQ_GEOMETRY_SPHERICAL;
    return a;
}

// cell, fraction and 1 / span along the lane's axis at coordinate x (as geo_cell)
__device__ __forceinline__ void geo_locate(const GeoAxis &a, double x, int &c, double &t, double &rh)
{
    if (a.X) {
        const double xv = fmax(x, -1e300);   // NaN -> the lowest cell
        int lo = 0, hi = a.n - 2;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.X[mid] <= xv)
                lo = mid;
            else
                hi = mid - 1;
        }
        const double x0 = a.X[lo], h = a.X[lo + 1] - x0;
        c = lo;
        t = (x - x0) / h;
        rh = 1.0 / h;
    } else {
        const double sg = fmin(fmax((x - a.o) * a.ih, -1e9), 1e9);
        double fl = floor(sg);
        fl = fl < 0.0 ? 0.0 : (fl > (double)(a.n - 2) ? (double)(a.n - 2) : fl);
        c = (int)fl;
        t = sg - fl;
        rh = a.rh;
    }
}

// the 8 corner values (the lane's component) of the cell the quad evaluated last
template <typename S>
struct GeoCell {
    int64_t key;
    S v[8];
};

// cell of the quad's point: fractions t of every axis, corner values (the
// lane's component) in `cell`; rh: the lane's 1 / span
template <typename T, typename S>
__device__ __forceinline__ void geo_corners(const S *nodes, const GeoAxis &a, double x, T t[3], double &rh,
                                            GeoCell<S> &cell)
{
    int c;
    double tf;
    geo_locate(a, x, c, tf, rh);
    const T tt = (T)tf;
    t[0] = quad_get<0>(tt);
    t[1] = quad_get<1>(tt);
    t[2] = quad_get<2>(tt);
    const int64_t sy = a.nx, sz = (int64_t)a.nx * a.ny;
    const int64_t key = (int64_t)quad_get<2>(c) * sz + (int64_t)quad_get<1>(c) * sy + quad_get<0>(c);
    if (key != cell.key) {
        cell.key = key;
        const S *p = nodes + 4 * key;
        cell.v[0] = p[0];
        cell.v[1] = p[4];
        cell.v[2] = p[4 * sy];
        cell.v[3] = p[4 * sy + 4];
        cell.v[4] = p[4 * sz];
        cell.v[5] = p[4 * sz + 4];
        cell.v[6] = p[4 * (sz + sy)];
        cell.v[7] = p[4 * (sz + sy) + 4];
    }
}

// 1 / (metric factor of the lane's axis) at the quad's point, eq. (2)
__device__ __forceinline__ double geo_inverse_scale(const GeoAxis &a, int c, double x)
{
    const double r = quad_get<2>(x), lat = quad_get<1>(x);
    const double sc = c == 0 ? r * cos(lat) : c == 1 ? r : 1.0;
    return 1.0 / sc;
}

// Right-hand side at the quad's point for the lane's components (rhs_from on
// field_at_geo, metric factors divided out); returns |u|^2 if NORM2.
template <typename T, typename S, int MODE, bool NORM2>
__device__ __forceinline__ T geo_rhs(const S *nodes, const GeoAxis &a, int c, double x, T sigma, T d1, T d2, T &kx,
                                     T &k1, T &k2, GeoCell<S> &cell)
{
    T t[3], val, dx, dy, dz, n2 = 0;
    double rh;
    geo_corners<T, S>(nodes, a, x, t, rh, cell);
    lerp_tree<T>((T)cell.v[0], (T)cell.v[1], (T)cell.v[2], (T)cell.v[3], (T)cell.v[4], (T)cell.v[5], (T)cell.v[6],
                 (T)cell.v[7], t[0], t[1], t[2], val, dx, dy, dz);
    const T ih = (T)rh;
    const T ihx = quad_get<0>(ih), ihy = quad_get<1>(ih), ihz = quad_get<2>(ih);
    T u, G[3];
    if (normalize_first<MODE>()) {
        u = val;
        G[0] = dx * ihx;
        G[1] = dy * ihy;
        G[2] = dz * ihz;
        if (NORM2) {
            const T u0 = quad_get<0>(u), u1 = quad_get<1>(u), u2 = quad_get<2>(u);
            n2 = jdot(u0, u1, u2, u0, u1, u2);
        }
    } else {
        const T v[3] = {quad_get<0>(val), quad_get<1>(val), quad_get<2>(val)};
        const T bn = sqrt(norm2<T, S, MODE>(v[0], v[1], v[2]));
        const T inv = bn > (T)1e-300 ? (T)1 / bn : (T)0;
        const T uu[3] = {v[0] * inv, v[1] * inv, v[2] * inv};
        u = val * inv;
        const T Gb[3] = {dx * ihx, dy * ihy, dz * ihz};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const T ug = along(uu[0], uu[1], uu[2], quad_get<0>(Gb[j]), quad_get<1>(Gb[j]), quad_get<2>(Gb[j]));
            G[j] = fma(-u, ug, Gb[j]) * inv;
        }
        if (NORM2) n2 = jdot(uu[0], uu[1], uu[2], uu[0], uu[1], uu[2]);
    }
    kx = sigma * u;
    k1 = sigma * jdot(G[0], G[1], G[2], quad_get<0>(d1), quad_get<1>(d1), quad_get<2>(d1));
    k2 = sigma * jdot(G[0], G[1], G[2], quad_get<0>(d2), quad_get<1>(d2), quad_get<2>(d2));
    if (a.sphere) {
        const T m = (T)geo_inverse_scale(a, c, x);
        kx *= m;
        k1 *= m;
        k2 *= m;
    }
    return n2;
}

#define QSQ_GEO_STAGES(STAGE)                                                                         \
    STAGE(1, (T)ck::a21)                                                                              \
    STAGE(2, (T)ck::a31, (T)ck::a32)                                                                  \
    STAGE(3, (T)ck::a41, (T)ck::a42, (T)ck::a43)                                                      \
    STAGE(4, (T)ck::a51, (T)ck::a52, (T)ck::a53, (T)ck::a54)                                          \
    STAGE(5, (T)ck::a61, (T)ck::a62, (T)ck::a63, (T)ck::a64, (T)ck::a65)

// One attempt in physical coordinates: positions FP64, stage arithmetic in T;
// the same error norm, controller, limits and statuses as on uniform grids.
template <typename T, typename S, int MODE>
__device__ __forceinline__ void geo_attempt(const S *nodes, const GeoAxis &a, const StepOpts &o, T rtol, T atol, int c3,
                                            const Records &rec, QuadState<T> &st, GeoCell<S> &cell, QuadCount &cnt)
{
    const int c = c3 == 3 ? 2 : c3;
    int stop = -1;
    T Kx[6], K1[6], K2[6];
    if (st.attempts >= o.max_steps) {
        stop = QSQ_END_MAX_STEPS;
    } else {
        // first stage (also the null test at the current point)
        const T un2 = geo_rhs<T, S, MODE, true>(nodes, a, c, st.X, st.sigma, st.D1, st.D2, Kx[0], K1[0], K2[0], cell);
        ++cnt.ev;
        if (un2 < (T)1e-12) stop = QSQ_END_NULL;
    }
    if (stop < 0) {
        T hs = st.h < (T)o.h_max ? st.h : (T)o.h_max;
        bool last = false;
        if (o.max_length > 0.0 && (double)hs >= o.max_length - st.s) {
            hs = (T)(o.max_length - st.s);
            last = true;
        }
#define QSQ_GSTAGE(ST, ...)                                                                                         \
    {                                                                                                              \
        const T c_[] = {__VA_ARGS__};                                                                              \
        T ax = 0, a1 = 0, a2 = 0;                                                                                  \
        _Pragma("unroll") for (int j = 0; j < ST; ++j)                                                             \
        {                                                                                                          \
            ax = fma(c_[j], Kx[j], ax);                                                                            \
            a1 = fma(c_[j], K1[j], a1);                                                                            \
            a2 = fma(c_[j], K2[j], a2);                                                                            \
        }                                                                                                          \
        geo_rhs<T, S, MODE, false>(nodes, a, c, advance(st.X, hs, ax), st.sigma, fma(hs, a1, st.D1),                \
                                   fma(hs, a2, st.D2), Kx[ST], K1[ST], K2[ST], cell);                              \
    }
        QSQ_GEO_STAGES(QSQ_GSTAGE)
#undef QSQ_GSTAGE
        cnt.ev += 5;
        const T b[3] = {ck_b5(Kx[0], Kx[2], Kx[3], Kx[5]), ck_b5(K1[0], K1[2], K1[3], K1[5]),
                        ck_b5(K2[0], K2[2], K2[3], K2[5])};
        const T e[3] = {ck_e(Kx[0], Kx[2], Kx[3], Kx[4], Kx[5]), ck_e(K1[0], K1[2], K1[3], K1[4], K1[5]),
                        ck_e(K2[0], K2[2], K2[3], K2[4], K2[5])};
        const double Xn = advance(st.X, hs, b[0]);
        const T yo[3] = {(T)st.X, st.D1, st.D2};
        const T yn[3] = {(T)Xn, fma(hs, b[1], st.D1), fma(hs, b[2], st.D2)};
        T err = 0, fsum = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            err = fmax(err, fabs(hs * e[k]) / err_scale(atol, rtol, yo[k], yn[k]));
            const T f = yn[k] + e[k];
            fsum += quad_get<0>(f);
            fsum += quad_get<1>(f);
            fsum += quad_get<2>(f);
        }
        err = fmax(fmax(quad_get<0>(err), quad_get<1>(err)), quad_get<2>(err));
        ++st.attempts;
        ++cnt.att;
        const bool out = quad_any(!(Xn >= a.lo && Xn <= a.hi));
        if (!isfinite(fsum)) {
            stop = QSQ_END_NONFINITE;
        } else if (err > (T)1) {
            const T f = (T)0.9 * (T)pow((double)err, -0.25);
            st.h = hs * (f > (T)0.2 ? f : (T)0.2);
            if ((double)st.h < o.hmin) stop = QSQ_END_UNDERFLOW;
        } else if (out) {
            quad_put(rec, c3, st, st.s, (double)hs, kPendingLand);
            st.active = false;
            ++cnt.land;
        } else {
            st.X = Xn;
            st.D1 = yn[1];
            st.D2 = yn[2];
            if (last) {
                st.s = o.max_length;
                stop = QSQ_END_MAX_LENGTH;
            } else {
                st.s += (double)hs;
                const T f = err > (T)0 ? (T)0.9 * (T)pow((double)err, -0.2) : (T)5;
                st.h = hs * (f < (T)5 ? f : (T)5);
            }
        }
    }
    if (stop >= 0) {
        quad_put(rec, c3, st, st.s, 0.0, stop);
        st.active = false;
    }
}

template <typename T, typename S, int MODE>
__global__ void __launch_bounds__(kQuadWg) k_trace_geo(TraceJob job)
{
    const int c3 = (int)(threadIdx.x & 3), c = c3 == 3 ? 2 : c3;
    const int64_t total = *job.rec.n_work, P = 2 * job.rec.cap;
    if (total <= 0) return;
    const StepOpts &o = job.o;
    const T rtol = (T)o.rtol, atol = (T)o.atol;
    const S *nodes = static_cast<const S *>(job.nodes) + c;
    const GeoAxis a = geo_axis(job.g, c);
    QuadState<T> st{};
    GeoCell<S> cell{};
    cell.key = -1;
    QuadCount cnt{};
    quad_drive(
        job, total, st.active,
        [&](int64_t rec) {
            st.rec = rec;
            st.sigma = rec >= job.rec.cap ? (T)-1 : (T)1;
            st.X = job.rec.y[c * P + rec];
            st.D1 = (T)job.rec.y[(3 + c) * P + rec];
            st.D2 = (T)job.rec.y[(6 + c) * P + rec];
            st.s = 0.0;
            st.h = (T)o.h_init;
            st.attempts = 0;
            ++cnt.act;
        },
        [&] { geo_attempt<T, S, MODE>(nodes, a, o, rtol, atol, c3, job.rec, st, cell, cnt); });
    if (job.work) quad_count(job.work, cnt);
}

// ---------------------------------------------------------------------------
// FP64 landing.  The step length that ends on a face needs the position only
// (eq. (2) does not involve the deviations), so the root find steps one value
// per lane; the step to the root is then taken once with all nine.
// ---------------------------------------------------------------------------
// the lane's position component at the end of a Cash-Karp step of length h
template <typename S, int MODE>
__device__ __forceinline__ double geo_step_x(const S *nodes, const GeoAxis &a, int c, double sigma, double x, double h,
                                             double k0, GeoCell<S> &cell)
{
    typedef double T;   // of the stage table
    double K[6];
    K[0] = k0;
    auto slope = [&](double xs) {
        double t[3], rh;
        geo_corners<double, S>(nodes, a, xs, t, rh, cell);
        const double val = lerp_val<double>((double)cell.v[0], (double)cell.v[1], (double)cell.v[2], (double)cell.v[3],
                                            (double)cell.v[4], (double)cell.v[5], (double)cell.v[6], (double)cell.v[7],
                                            t[0], t[1], t[2]);
        double u = val;
        if (!normalize_first<MODE>()) {
            const double v[3] = {quad_get<0>(val), quad_get<1>(val), quad_get<2>(val)};
            const double bn = sqrt(norm2<double, S, MODE>(v[0], v[1], v[2]));
            u = val * (bn > 1e-300 ? 1.0 / bn : 0.0);
        }
        double k = sigma * u;
        if (a.sphere) k *= geo_inverse_scale(a, c, xs);
        return k;
    };
#define QSQ_GLSTAGE(ST, ...)                                                          \
    {                                                                                 \
        const double c_[] = {__VA_ARGS__};                                            \
        double ax = 0;                                                                \
        _Pragma("unroll") for (int j = 0; j < ST; ++j) ax = fma(c_[j], K[j], ax);     \
        K[ST] = slope(fma(h, ax, x));                                                 \
    }
    QSQ_GEO_STAGES(QSQ_GLSTAGE)
#undef QSQ_GLSTAGE
    return fma(h, ck_b5(K[0], K[2], K[3], K[5]), x);
}

// For every face the trial step crosses, Illinois regula falsi from the secant
// point on the face gap of the FP64 step's end over its length (|gap| <=
// gtol); the face reached first (the shortest length; exact ties keep the
// lower face) takes the line, the state is stepped there and snapped onto it.
template <typename S, int MODE>
__global__ void __launch_bounds__(kQuadWg) k_land_geo(TraceJob job)
{
    typedef double T;   // of the stage table
    const int c3 = (int)(threadIdx.x & 3), c = c3 == 3 ? 2 : c3;
    const int64_t total = *job.rec.n_land, P = 2 * job.rec.cap;
    const S *nodes = static_cast<const S *>(job.nodes) + c;
    const GeoAxis a = geo_axis(job.g, c);
    const double gtol = job.o.gtol;
    GeoCell<S> cell{};
    cell.key = -1;
    for (int64_t it = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2; it < total;
         it += ((int64_t)gridDim.x * blockDim.x) >> 2) {
        const int64_t r = job.rec.work2[it];
        const double sigma = r >= job.rec.cap ? -1.0 : 1.0;
        const double x = job.rec.y[c * P + r], d1 = job.rec.y[(3 + c) * P + r], d2 = job.rec.y[(6 + c) * P + r];
        const double s = job.rec.s[r], hs = job.rec.h[r];
        double Kx[6], K1[6], K2[6];
        geo_rhs<double, S, MODE, false>(nodes, a, c, x, sigma, d1, d2, Kx[0], K1[0], K2[0], cell);
        // signed distances beyond the six faces, at the quad's point whose component the lane holds
        double glo, ghi;
        auto gap_of = [&](int f) {
            const double v = (f & 1) ? ghi : glo;
            return (f >> 1) == 0 ? quad_get<0>(v) : (f >> 1) == 1 ? quad_get<1>(v) : quad_get<2>(v);
        };
        auto gap_at = [&](double h, int f) {
            const double xe = h > 0.0 ? geo_step_x<S, MODE>(nodes, a, c, sigma, x, h, Kx[0], cell) : x;
            glo = a.lo - xe;
            ghi = xe - a.hi;
            return gap_of(f);
        };
        double best = INFINITY, gmax = -INFINITY, gend[6];
        int face = -1, fmax_ = 0;
        gap_at(hs, 0);
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            gend[f] = gap_of(f);
            if (gend[f] > gmax) {
                gmax = gend[f];
                fmax_ = f;
            }
        }
#pragma unroll 1
        for (int f = 0; f < 6; ++f) {
            double ge = gend[0];
#pragma unroll
            for (int k = 1; k < 6; ++k) ge = f == k ? gend[k] : ge;
            if (!(ge > 0.0)) continue;
            double lo = 0.0, hi = hs, ga = gap_at(lo, f), gb = ge, root;
            if (ga >= 0.0) {
                root = 0.0;
            } else {
                int side = 0;
                root = -1.0;
                for (int k = 0; k < 200 && root < 0.0; ++k) {
                    const double h = landing_secant(lo, ga, hi, gb);
                    const double gc = gap_at(h, f);
                    if (fabs(gc) <= gtol) {
                        root = h;
                    } else if (gc > 0.0) {
                        hi = h;
                        gb = gc;
                        if (side == +1) ga *= 0.5;
                        side = +1;
                    } else {
                        lo = h;
                        ga = gc;
                        if (side == -1) gb *= 0.5;
                        side = -1;
                    }
                    if (root < 0.0 && hi - lo <= 1e-15 * hs) root = ga > -gb ? lo : hi;
                }
                if (root < 0.0) root = ga > -gb ? lo : hi;
            }
            if (root < best) {
                best = root;
                face = f;
            }
        }
        if (face < 0) {
            // the trial step left the box in FP32 but the FP64 step does not:
            // end on the face nearest the FP64 end
            best = hs;
            face = fmax_;
        }
        double xl = x, l1 = d1, l2 = d2;
        if (best > 0.0) {
#define QSQ_GFSTAGE(ST, ...)                                                                                        \
    {                                                                                                              \
        const double c_[] = {__VA_ARGS__};                                                                         \
        double ax = 0, a1 = 0, a2 = 0;                                                                             \
        _Pragma("unroll") for (int j = 0; j < ST; ++j)                                                             \
        {                                                                                                          \
            ax = fma(c_[j], Kx[j], ax);                                                                            \
            a1 = fma(c_[j], K1[j], a1);                                                                            \
            a2 = fma(c_[j], K2[j], a2);                                                                            \
        }                                                                                                          \
        geo_rhs<double, S, MODE, false>(nodes, a, c, fma(best, ax, x), sigma, fma(best, a1, d1), fma(best, a2, d2), \
                                        Kx[ST], K1[ST], K2[ST], cell);                                             \
    }
            QSQ_GEO_STAGES(QSQ_GFSTAGE)
#undef QSQ_GFSTAGE
            xl = fma(best, ck_b5(Kx[0], Kx[2], Kx[3], Kx[5]), x);
            l1 = fma(best, ck_b5(K1[0], K1[2], K1[3], K1[5]), d1);
            l2 = fma(best, ck_b5(K2[0], K2[2], K2[3], K2[5]), d2);
        }
        if (c == (face >> 1)) xl = (face & 1) ? a.hi : a.lo;
        if (c3 < 3) {
            job.rec.y[c * P + r] = xl;
            job.rec.y[(3 + c) * P + r] = l1;
            job.rec.y[(6 + c) * P + r] = l2;
        } else {
            job.rec.s[r] = s + best;
            job.rec.h[r] = 0.0;
            job.rec.status[r] = face;
        }
    }
}
#undef QSQ_GEO_STAGES
