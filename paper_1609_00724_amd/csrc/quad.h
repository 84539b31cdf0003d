// Stepping with four lanes per half-line (a quad of adjacent lanes): lane c of
// the quad holds component c of the position and of both deviation vectors and
// evaluates component c of the field (lane 3 repeats lane 2, or idles along on
// values that nothing reads), and the values
// that every component needs (cell fractions, deviations) cross the quad by
// DPP moves.  An attempt is a serial chain of six evaluations; a lane that does
// a third of the components issues about a third of the instructions (640
// vector instructions against 1490), so the chain is shorter: 2.4 us an
// attempt against 5.4 where one line is all a SIMD has.  The lane's state (18
// stage slopes and 8 corner values instead of 54 and 24) lets four waves stay
// resident on a SIMD instead of two.  Included by trace.hip
// after the evaluation helpers it shares with the one-lane kernel; every
// operation on a component is the one-lane kernel's, in its order, so the
// results are the same bit for bit.
#pragma once

template <int K>
__device__ __forceinline__ int quad_get(int v) { return __builtin_amdgcn_mov_dpp(v, 0x55 * K, 0xf, 0xf, true); }
template <int K>
__device__ __forceinline__ float quad_get(float v) { return __int_as_float(quad_get<K>(__float_as_int(v))); }
template <int K>
__device__ __forceinline__ double quad_get(double v)
{
    return __hiloint2double(quad_get<K>(__double2hiint(v)), quad_get<K>(__double2loint(v)));
}

// the lane's share of a line's grid: axis c of it
template <typename T>
struct QuadGeom {
    int n;              // nodes along the axis
    int ka;             // records from one cell to the next along the axis (lane 3: 0)
    double o, ih, lo, hi;
    uint32_t sy, sz;    // bytes to the next node record along y and z
    T iha;              // 1 / spacing of the lane's axis
    T iht[3];           // 1 / spacing of every axis
};

template <typename T>
struct QuadState {
    double X, s;        // position component; length (the same in the quad's lanes)
    T D1, D2;           // deviation components
    T h, sigma;
    int attempts;
    int64_t rec;
    bool active, have_k1;
    T Kx0, K10, K20;    // first-stage slopes
};

// the 8 corner values (component c) of the cell the quad evaluated last
template <typename T>
struct QuadCell {
    int key;
    T v[8];
};

template <typename T, typename S>
__device__ __forceinline__ T quad_load(const char *p)
{
    if constexpr (std::is_same<S, Bf16>::value)
        return (T)__uint_as_float((uint32_t)*reinterpret_cast<const uint16_t *>(p) << 16);
    else
        return (T)*reinterpret_cast<const S *>(p);
}

// bytes of one value of a node record
template <typename S>
constexpr int value_bytes() { return std::is_same<S, Bf16>::value ? 2 : (int)sizeof(S); }

// floor(q) kept within [lo, hi] (lo for a NaN)
__device__ __forceinline__ float clamp_floor(float q, float lo, float hi)
{
    return __builtin_amdgcn_fmed3f(floorf(q), lo, hi);
}
__device__ __forceinline__ double clamp_floor(double q, double lo, double hi) { return fmin(fmax(floor(q), lo), hi); }

// reference cell of an attempt along the lane's axis: the offsets that the
// cell index may take from it, and its share of the record key
template <typename T>
struct QuadRef {
    int ib, key0;
    T flo, fhi;
};

template <typename T>
__device__ __forceinline__ QuadRef<T> quad_ref(const QuadGeom<T> &g, int ib)
{
    return {ib, __mul24(ib, g.ka), (T)-ib, (T)(g.n - 2 - ib)};
}

// Values (the lane's component) of the K records of one stencil row, K = 3 or
// 4.  FP32 records: lane l of the quad loads record l whole (16 bytes; the
// quad's loads fall in one or two cache lines, one access instead of K), and a
// 4 x 4 transpose across the quad hands every lane its component of all four.
// Other types: the lane's component of each record.  off: byte offset of the
// row; ox: of the quad lane's record in it; oc: of the lane's component of
// records 0 .. K - 1.
template <typename T, typename S, int K>
__device__ __forceinline__ void quad_row(const char *recs, uint32_t off, uint32_t ox, const uint32_t oc[K], int c3, T v[K])
{
    if constexpr (std::is_same<S, float>::value) {
        const float4 r = *reinterpret_cast<const float4 *>(recs + (off + ox));
        float a0 = r.x, a1 = r.y, a2 = r.z, a3 = r.w;
        const bool odd = c3 & 1, high = c3 & 2;
        // swap across lanes 1 apart, then 2 apart
        const auto x1 = [](float w) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(w), 0xb1, 0xf, 0xf, true)); };
        const auto x2 = [](float w) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(w), 0x4e, 0xf, 0xf, true)); };
        const float s0 = x1(a0), s1 = x1(a1), s2 = x1(a2), s3 = x1(a3);
        a0 = odd ? s1 : a0;
        a1 = odd ? a1 : s0;
        a2 = odd ? s3 : a2;
        a3 = odd ? a3 : s2;
        const float t0 = x2(a0), t1 = x2(a1), t2 = x2(a2), t3 = x2(a3);
        const float o[4] = {high ? t2 : a0, high ? t3 : a1, high ? a2 : t0, high ? a3 : t1};
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = (T)o[k];
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = quad_load<T, S>(recs + (off + oc[k]));
    }
}

// Value and grid-unit gradient of record component comp (lane 3 of the FP32
// transpose: the fourth) by the separable stencil sum of order K - 1 at cell ci, fraction t of the lane's axis: along x per
// row, then y, then z, in stencil_sum's order.  Each lane forms its own axis'
// weights and the quad shares them.
template <typename T, typename S, int K>
__device__ __forceinline__ void quad_stencil(const char *recs, int n, uint32_t sy, uint32_t sz, int c3, int comp, int ci,
                                             T t, T &val, T &dx, T &dy, T &dz)
{
    constexpr uint32_t VB = value_bytes<S>(), RB = 4 * VB;
    const int c = c3 == 3 ? 2 : c3;
    int s0;
    T w[K], dw[K];
    axis_stencil<K, T>(ci, t, n, s0, w, dw);
    // byte offsets of the lane's axis' stencil nodes (the last may lie past
    // the grid, with weight zero)
    const uint32_t st = c == 0 ? RB : c == 1 ? sy : sz;
    uint32_t off[K];
#pragma unroll
    for (int k = 0; k < K; ++k) off[k] = (uint32_t)(s0 + k < n - 1 ? s0 + k : n - 1) * st;
    uint32_t oc[K], oy[K], oz[K], ox = 0;
    T wx[K], wy[K], wz[K], dwx[K], dwy[K], dwz[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t o = (uint32_t)quad_get<0>((int)off[k]);
        oc[k] = o + VB * (uint32_t)comp;
        if (k == c3 || (k == K - 1 && c3 > k)) ox = o;
        oy[k] = (uint32_t)quad_get<1>((int)off[k]);
        oz[k] = (uint32_t)quad_get<2>((int)off[k]);
        wx[k] = quad_get<0>(w[k]);
        wy[k] = quad_get<1>(w[k]);
        wz[k] = quad_get<2>(w[k]);
        dwx[k] = quad_get<0>(dw[k]);
        dwy[k] = quad_get<1>(dw[k]);
        dwz[k] = quad_get<2>(dw[k]);
    }
    val = dx = dy = dz = (T)0;
#pragma unroll
    for (int kz = 0; kz < K; ++kz) {
        T v[K][K], ay = 0, axy = 0, ayy = 0;
#pragma unroll
        for (int ky = 0; ky < K; ++ky) quad_row<T, S, K>(recs, oz[kz] + oy[ky], ox, oc, c3, v[ky]);
#pragma unroll
        for (int ky = 0; ky < K; ++ky) {
            T rx = 0, drx = 0;
#pragma unroll
            for (int kx = 0; kx < K; ++kx) {
                rx = fma(wx[kx], v[ky][kx], rx);
                drx = fma(dwx[kx], v[ky][kx], drx);
            }
            ay = fma(wy[ky], rx, ay);
            axy = fma(wy[ky], drx, axy);
            ayy = fma(dwy[ky], rx, ayy);
        }
        val = fma(wz[kz], ay, val);
        dx = fma(wz[kz], axy, dx);
        dy = fma(wz[kz], ayy, dy);
        dz = fma(dwz[kz], ay, dz);
        // one z plane's rows in flight, not all of the stencil's
        __builtin_amdgcn_sched_barrier(0);
    }
}

// One evaluation at grid-unit reference r plus offset q (the lane's axis) for
// deviations d1, d2 (the lane's components); returns |u|^2 if NORM2.  `recs`
// points at the records, `c3` is the lane's place in its quad.  Record keys and byte
// offsets fit 32 bits and the axis products 24 bits (the launcher checks).
template <typename T, typename S, int MODE, bool NORM2>
__device__ __forceinline__ T quad_rhs(const char *recs, const QuadGeom<T> &g, int c3, const QuadRef<T> &r, T q, T d1,
                                      T d2, T &kx, T &k1, T &k2, QuadCell<T> &cell)
{
    const int c = c3 == 3 ? 2 : c3;
    constexpr uint32_t VB = value_bytes<S>(), RB = 4 * VB;
    // cell and fraction as cell_of gives them
    const T fl = clamp_floor(q, r.flo, r.fhi), t = q - fl;
    const int ifl = (int)fl;
    T val, dx, dy, dz;
    if constexpr (interp_order<MODE>() > 1) {
        quad_stencil<T, S, interp_order<MODE>() + 1>(recs, g.n, g.sy, g.sz, c3, c, r.ib + ifl, t, val, dx,
                                                        dy, dz);
    } else {
        // the record key of the cell, summed over the axes (lane 3 adds nothing)
        int key = __mul24(ifl, g.ka) + r.key0;
        key += __builtin_amdgcn_mov_dpp(key, 0xb1, 0xf, 0xf, true);   // lanes 1 0 3 2
        key += __builtin_amdgcn_mov_dpp(key, 0x4e, 0xf, 0xf, true);   // lanes 2 3 0 1
        if (key != cell.key) {
            cell.key = key;
            const uint32_t o0 = (uint32_t)key * RB + VB * (uint32_t)c, o1 = o0 + g.sy, o2 = o0 + g.sz, o3 = o1 + g.sz;
            cell.v[0] = quad_load<T, S>(recs + o0);
            cell.v[1] = quad_load<T, S>(recs + o0 + RB);
            cell.v[2] = quad_load<T, S>(recs + o1);
            cell.v[3] = quad_load<T, S>(recs + o1 + RB);
            cell.v[4] = quad_load<T, S>(recs + o2);
            cell.v[5] = quad_load<T, S>(recs + o2 + RB);
            cell.v[6] = quad_load<T, S>(recs + o3);
            cell.v[7] = quad_load<T, S>(recs + o3 + RB);
        }
        lerp_tree<T>(cell.v[0], cell.v[1], cell.v[2], cell.v[3], cell.v[4], cell.v[5], cell.v[6], cell.v[7],
                     quad_get<0>(t), quad_get<1>(t), quad_get<2>(t), val, dx, dy, dz);
    }
    const T a0 = quad_get<0>(d1), a1 = quad_get<1>(d1), a2 = quad_get<2>(d1);
    const T b0 = quad_get<0>(d2), b1 = quad_get<1>(d2), b2 = quad_get<2>(d2);
    T u, G[3], n2 = 0;
    if (normalize_first<MODE>()) {
        u = val;
        G[0] = dx * g.iht[0];
        G[1] = dy * g.iht[1];
        G[2] = dz * g.iht[2];
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
        const T Gb[3] = {dx * g.iht[0], dy * g.iht[1], dz * g.iht[2]};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const T ug = along(uu[0], uu[1], uu[2], quad_get<0>(Gb[j]), quad_get<1>(Gb[j]), quad_get<2>(Gb[j]));
            G[j] = fma(-u, ug, Gb[j]) * inv;
        }
        if (NORM2) n2 = jdot(uu[0], uu[1], uu[2], uu[0], uu[1], uu[2]);
    }
    kx = u;
    k1 = jdot(G[0], G[1], G[2], a0, a1, a2);
    k2 = jdot(G[0], G[1], G[2], b0, b1, b2);
    return n2;
}

// end record of the quad's line
template <typename T>
__device__ __forceinline__ void quad_put(const Records &r, int c, const QuadState<T> &st, double s, double h, int status)
{
    const int64_t P = 2 * r.cap, i = st.rec;
    if (c < 3) {
        r.y[c * P + i] = st.X;
        r.y[(3 + c) * P + i] = (double)st.D1;
        r.y[(6 + c) * P + i] = (double)st.D2;
    } else {
        r.s[i] = s;
        r.h[i] = h;
        r.status[i] = status;
        r.attempts[i] = st.attempts;
    }
}

struct QuadCount {
    unsigned int att, ev, act, land;   // of the lines this lane leads
};

// a flag that holds in any of the quad's first three lanes (lane 3 repeats lane 2)
__device__ __forceinline__ bool quad_any(bool f)
{
    int v = f ? 1 : 0;
    v |= __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true);
    v |= __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true);
    return v != 0;
}

// One step attempt of the quad's line (the one-lane kernel's order: step cap,
// null, trial, accept or reject, exit); writes the end record and clears
// st.active when the line ends.  Every branch is taken by whole quads.
template <typename T, typename S, int MODE, bool EULER>
__device__ __forceinline__ void quad_attempt(const char *recs, const QuadGeom<T> &g, const StepOpts &o, T rtol,
                                             T atol, T hmax, double hmin, int c3,
                                             const Records &rec, QuadState<T> &st, QuadCell<T> &cell, QuadCount &cnt)
{
    int stop = -1;
    if (st.attempts >= o.max_steps) stop = QSQ_END_MAX_STEPS;
    QuadRef<T> ref{};
    T fb = 0;
    if (stop < 0) {
        const double xg = (st.X - g.o) * g.ih;
        const double fl = floor(xg);
        ref = quad_ref<T>(g, (int)fl);
        fb = (T)fma(st.X - g.o, g.ih, -fl);
        if (EULER || !st.have_k1) {
            const T un2 = quad_rhs<T, S, MODE, true>(recs, g, c3, ref, fb, st.D1, st.D2, st.Kx0, st.K10,
                                                             st.K20, cell);
            ++cnt.ev;
            if (un2 < (T)1e-12) stop = QSQ_END_NULL;   // NaN: not a null (the step reports it)
            st.have_k1 = true;
        }
    }
    if (stop < 0) {
        T hs = EULER ? st.h : (st.h < hmax ? st.h : hmax);
        bool last = false;
        if (o.max_length > 0.0 && (double)hs >= o.max_length - st.s) {
            hs = (T)(o.max_length - st.s);
            last = true;
        }
        const T hsig = st.sigma * hs;
        double Xn;
        T D1n, D2n, err = 0, fpart;
        if constexpr (EULER) {
            Xn = advance(st.X, hsig, st.Kx0);
            D1n = fma(hsig, st.K10, st.D1);
            D2n = fma(hsig, st.K20, st.D2);
            fpart = ((T)Xn + D1n) + D2n;
            ++cnt.att;
        } else {
            T Kx[6], K1[6], K2[6];
            Kx[0] = st.Kx0;
            K1[0] = st.K10;
            K2[0] = st.K20;
#define QSQ_QSTAGE(ST, ...)                                                                                        \
    {                                                                                                              \
        const T c_[] = {__VA_ARGS__};                                                                              \
        T ax = 0, a1 = 0, a2 = 0;                                                                                  \
        _Pragma("unroll") for (int j = 0; j < ST; ++j)                                                             \
        {                                                                                                          \
            ax = fma(c_[j], Kx[j], ax);                                                                            \
            a1 = fma(c_[j], K1[j], a1);                                                                            \
            a2 = fma(c_[j], K2[j], a2);                                                                            \
        }                                                                                                          \
        quad_rhs<T, S, MODE, false>(recs, g, c3, ref, fma(hsig * ax, g.iha, fb), fma(hsig, a1, st.D1),        \
                                            fma(hsig, a2, st.D2), Kx[ST], K1[ST], K2[ST], cell);                   \
    }
            QSQ_QSTAGE(1, (T)ck::a21)
            QSQ_QSTAGE(2, (T)ck::a31, (T)ck::a32)
            QSQ_QSTAGE(3, (T)ck::a41, (T)ck::a42, (T)ck::a43)
            QSQ_QSTAGE(4, (T)ck::a51, (T)ck::a52, (T)ck::a53, (T)ck::a54)
            QSQ_QSTAGE(5, (T)ck::a61, (T)ck::a62, (T)ck::a63, (T)ck::a64, (T)ck::a65)
#undef QSQ_QSTAGE
            const T bx = ck_b5(Kx[0], Kx[2], Kx[3], Kx[5]);
            const T b1 = ck_b5(K1[0], K1[2], K1[3], K1[5]);
            const T b2 = ck_b5(K2[0], K2[2], K2[3], K2[5]);
            const T ex = ck_e(Kx[0], Kx[2], Kx[3], Kx[4], Kx[5]);
            const T e1 = ck_e(K1[0], K1[2], K1[3], K1[4], K1[5]);
            const T e2 = ck_e(K2[0], K2[2], K2[3], K2[4], K2[5]);
            Xn = advance(st.X, hsig, bx);
            D1n = fma(hsig, b1, st.D1);
            D2n = fma(hsig, b2, st.D2);
            const T xo = (T)st.X, xn = (T)Xn;
            err = fmax(err, err_ratio(fabs(hs * ex), err_scale(atol, rtol, xo, xn)));
            err = fmax(err, err_ratio(fabs(hs * e1), err_scale(atol, rtol, st.D1, D1n)));
            err = fmax(err, err_ratio(fabs(hs * e2), err_scale(atol, rtol, st.D2, D2n)));
            err = fmax(fmax(quad_get<0>(err), quad_get<1>(err)), quad_get<2>(err));
            fpart = (xn + D1n) + (D2n + ex) + (e1 + e2);
            ++cnt.att;
            cnt.ev += 5;
        }
        T fsum = 0;
        fsum += quad_get<0>(fpart);
        fsum += quad_get<1>(fpart);
        fsum += quad_get<2>(fpart);
        ++st.attempts;
        const bool out = quad_any(c3 < 3 && !(Xn >= g.lo && Xn <= g.hi));
        if (!isfinite(fsum)) {
            stop = QSQ_END_NONFINITE;
        } else if (!EULER && err > (T)1) {
            // reject: shrink, keep k1 (y is unchanged)
            const T f = (T)0.9 * (T)exp2((T)-0.25 * (T)log2(err));
            st.h = hs * (f > (T)0.2 ? f : (T)0.2);
            if ((double)st.h < hmin) stop = QSQ_END_UNDERFLOW;
        } else if (out) {
            // the step that leaves the box: hand over to FP64 landing
            quad_put(rec, c3, st, st.s, (double)hs, kPendingLand);
            st.active = false;
            ++cnt.land;
        } else {
            st.X = Xn;
            st.D1 = D1n;
            st.D2 = D2n;
            st.have_k1 = false;
            if (last) {
                st.s = o.max_length;
                stop = QSQ_END_MAX_LENGTH;
            } else {
                st.s += (double)hs;
                if (!EULER) {
                    const T f = err > (T)0 ? (T)0.9 * (T)exp2((T)-0.2 * (T)log2(err)) : (T)5;
                    st.h = hs * (f < (T)5 ? f : (T)5);
                }
            }
        }
    }
    if (stop >= 0) {
        quad_put(rec, c3, st, st.s, 0.0, stop);
        st.active = false;
    }
}

// the lane's axis of a grid (c: the lane's component, 0..2; dup: lane 3)
template <typename T, typename S>
__device__ __forceinline__ QuadGeom<T> quad_geom(const Geom &g, int c, bool dup)
{
    QuadGeom<T> q;
    q.n = c == 0 ? g.n[0] : c == 1 ? g.n[1] : g.n[2];
    q.o = c == 0 ? g.o[0] : c == 1 ? g.o[1] : g.o[2];
    q.ih = c == 0 ? g.ih[0] : c == 1 ? g.ih[1] : g.ih[2];
    q.lo = c == 0 ? g.lo[0] : c == 1 ? g.lo[1] : g.lo[2];
    q.hi = c == 0 ? g.hi[0] : c == 1 ? g.hi[1] : g.hi[2];
#pragma unroll
    for (int d = 0; d < 3; ++d) q.iht[d] = (T)g.ih[d];
    q.iha = (T)q.ih;
    q.sy = 4u * value_bytes<S>() * (uint32_t)g.n[0];
    q.sz = q.sy * (uint32_t)g.n[1];
    q.ka = c == 0 ? 1 : c == 1 ? g.n[0] : g.n[0] * g.n[1];
    if (dup) q.ka = 0;
    return q;
}

// Work distribution of the four-lane kernels, up to 16 half-lines per wave.  A
// list of fewer than 16 lines per SIMD is spread over one wave per SIMD (a
// wave with fewer lines waits for fewer cell moves); a longer one goes 16
// lines per wave, and what does not fit the grid at first goes, with one
// atomic per chunk of 16, to the quads that fall idle.  start(record) sets up
// the quad's line, attempt() takes one step and clears `active` at its end.
constexpr int kQuadWg = 256, kQuadLines = 16;

template <typename Start, typename Attempt>
__device__ __forceinline__ void quad_drive(const TraceJob &job, int64_t total, bool &active, Start start, Attempt attempt)
{
    const int lane = (int)(threadIdx.x & 63), qi = lane >> 2;
    const int64_t wave = (int64_t)blockIdx.x * (kQuadWg / 64) + (threadIdx.x >> 6);
    const int per = total >= (int64_t)job.simds * kQuadLines ? kQuadLines : (int)((total + job.simds - 1) / job.simds);
    unsigned long long *count = job.counter + kPartCounter;
    int64_t item = wave * per + qi;
    if (qi >= per || item >= total) item = -1;
    // the counter may hold items past the first of every wave
    bool more = total > (int64_t)gridDim.x * (kQuadWg / 64) * per;
    int64_t cnext = 0, cend = 0;   // the wave's unassigned items [cnext, cend)
    for (;;) {
        if (!active && item >= 0) {
            start((int64_t)job.rec.work[item]);
            active = true;
        }
        if (__ballot(active) == 0 && !more) break;
        if (active) attempt();
        item = -1;
        const uint64_t need = __ballot(!active);
        if (more && need) {
            // items for the idle quads: what is left of the wave's chunk, then a fresh one
            const int j = __popcll(need & ((1ull << (lane & ~3)) - 1ull)) >> 2, k = __popcll(need) >> 2;
            const int64_t avail = cend - cnext;
            if (j < avail) item = cnext + j;
            if (avail < k) {
                unsigned long long b = 0;
                if (lane == 0) b = atomicAdd(count, (unsigned long long)kQuadLines);
                const int64_t fresh = (int64_t)__shfl(b, 0);
                more = fresh < total;
                cend = more ? min(fresh + kQuadLines, total) : fresh;
                if (j >= avail && fresh + (j - avail) < cend) item = fresh + (j - avail);
                cnext = min(fresh + (k - avail), cend);
            } else {
                cnext += k;
            }
            if (active) item = -1;
        }
    }
}

// Work counters: one lane of each quad counts its lines, and a workgroup adds
// its four sums with one instruction.  Every workgroup of the grid adds to the
// same 32 bytes, one after the other (10 ns each): with four atomics per wave,
// stepping of 65 536 half-lines of a volume (64^2 x 32 cells, 8 cells a step)
// took 223 us, against 57 so and 60 without counters; a 256^2 map of the same
// field with its levels 0.58 against 0.34 ms.
__device__ __forceinline__ void quad_count(unsigned long long *work, const QuadCount &cnt)
{
    __shared__ unsigned long long sums[kQuadWg / 64][4];
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long v[4] = {cnt.att, cnt.ev, cnt.act, cnt.land};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (lane & 3) v[k] = 0;
#pragma unroll
        for (int s = 32; s >= 4; s >>= 1) v[k] += __shfl_xor(v[k], s);
        if (lane == 0) sums[threadIdx.x >> 6][k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        unsigned long long sum = 0;
#pragma unroll
        for (int w = 0; w < kQuadWg / 64; ++w) sum += sums[w][threadIdx.x];
        if (sum) atomicAdd(&work[threadIdx.x], sum);
    }
}

// Stepping kernel of the lists that quad_list gives four lanes a line
template <typename T, typename S, int MODE, bool BATCH, bool EULER>
__global__ void __launch_bounds__(kQuadWg) k_trace_quad(TraceJob job)
{
    const StepOpts &o = job.o;
    const int c3 = (int)(threadIdx.x & 3), c = c3 == 3 ? 2 : c3;
    const int64_t total = *job.rec.n_work;
    if (total > job.quad_max) return;   // the one-lane kernel's call
    const int64_t P = 2 * job.rec.cap;
    const T rtol = (T)o.rtol, atol = (T)o.atol;
    T hmax = (T)o.h_max;
    double h_init = o.h_init, hmin = o.hmin;
    const char *recs = static_cast<const char *>(job.nodes);
    QuadGeom<T> g = quad_geom<T, S>(job.g, c, c3 == 3);
    QuadState<T> st{};
    QuadCell<T> cell{};
    cell.key = -1;
    QuadCount cnt{};
    quad_drive(
        job, total, st.active,
        [&](int64_t rec) {
            st.rec = rec;
            const int dir = rec >= job.rec.cap ? 1 : 0;
            if constexpr (BATCH) {
                const SetDesc &sd = job.sets[job.set_of[dir ? rec - job.rec.cap : rec]];
                g = quad_geom<T, S>(sd.g, c, c3 == 3);
                recs = in_global<char>(sd.nodes);
                h_init = sd.h_init;
                hmin = sd.hmin;
                hmax = (T)sd.h_max;
                cell.key = -1;   // another field
            }
            // the seed pass left x0 and the frame (eq. 9) in the record
            st.sigma = dir ? (T)-1 : (T)1;
            st.X = job.rec.y[c * P + rec];
            st.D1 = (T)job.rec.y[(3 + c) * P + rec];
            st.D2 = (T)job.rec.y[(6 + c) * P + rec];
            st.s = 0.0;
            st.h = (T)h_init;
            st.attempts = 0;
            st.have_k1 = false;
            ++cnt.act;
        },
        [&] { quad_attempt<T, S, MODE, EULER>(recs, g, o, rtol, atol, hmax, hmin, c3, job.rec, st, cell, cnt); });
    if (job.work) quad_count(job.work, cnt);
}
