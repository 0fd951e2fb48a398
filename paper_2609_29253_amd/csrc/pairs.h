// One voxel-transducer pair: its quadrants on the parameter rectangle, built once
// per pair and swept into a sink (the kernels' histograms or gathers).
#pragma once

#include "area.h"

namespace patop {

#if defined(__clang__)
typedef __attribute__((address_space(3))) double LdsDouble;
#else
typedef double LdsDouble;
#endif

// frame coordinates of a voxel (Sec. 4.1 / Sec. 4.2 frames), FP64
__device__ __forceinline__ void frame_coords(const TrDev& T, int ix, int iy, int iz, double x[3])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) x[a] = fma(T.g[a][0], ix, fma(T.g[a][1], iy, fma(T.g[a][2], iz, T.base[a])));
}

// the work-group's copy of kArcTable (no barrier here)
template <int STRIDE>
__device__ __forceinline__ void load_arc_table(double* tab)
{
    for (int i = threadIdx.x; i < kArcTab; i += STRIDE) tab[i] = kArcTable[i];
}

// ---------------------------------------------------------------------------
// per-pair geometry: reflected quadrants of the parameter rectangle
// (Eq. uvminmax; Eq. folded_intervals for the cylinder), built one at a time
// ---------------------------------------------------------------------------

// Two reflected intervals that share an end point, [e, p] and [e, q] (or [p, e]
// and [q, e]), cover the same parameter region as the interval between e and
// the nearer of p, q counted twice plus the remainder counted once.  Sweeping
// the merged form visits each bin of the shared part once instead of twice.
struct WInt {
    double lo[2], hi[2];
    float w[2];
    int n;
};

// intervals [0, A] and [0, B] (A, B >= 0), Eq. uvminmax with the origin inside.
// MERGE: the shared-part form above; else the two intervals as they are, which
// an approximation that is not additive over sub-intervals (the trapezoidal
// I_l: the chord of a split arc is not the chord of the arc) must use.
template <bool MERGE = true>
__device__ __forceinline__ void split_at_zero(double A, double B, WInt& I)
{
    if (MERGE) {
        double m = fmin(A, B), M = fmax(A, B);
        I.lo[0] = 0.0; I.hi[0] = m; I.w[0] = 2.0f;
        I.lo[1] = m;   I.hi[1] = M; I.w[1] = 1.0f;
    } else {
        I.lo[0] = 0.0; I.hi[0] = A; I.w[0] = 1.0f;
        I.lo[1] = 0.0; I.hi[1] = B; I.w[1] = 1.0f;
    }
    I.n = 2;
}

// the reflected intervals of [lo, hi] about 0 (Eq. uvminmax)
template <bool MERGE = true>
__device__ __forceinline__ void fold_line(double lo, double hi, WInt& I)
{
    if (lo < 0.0 && 0.0 < hi) { split_at_zero<MERGE>(-lo, hi, I); return; }
    double a = fabs(lo), b = fabs(hi);
    I.lo[0] = fmin(a, b); I.hi[0] = fmax(a, b); I.w[0] = 1.0f;
    I.lo[1] = I.hi[1] = 0.0; I.w[1] = 0.0f;
    I.n = 1;
}

template <int NW>
struct PlanarPair {
    WInt U, V;
    double z2;
    const double* tab;
    __device__ __forceinline__ void bind(double*, const double2*, const double* t, const TrDev*, int, int, int)
    {
        tab = t;
    }
    __device__ __forceinline__ void setup(const TrDev& T, const double x[3], double)
    {
        double L1 = T.p[0], L2 = T.p[1];
        fold_line(-L1 - x[0], L1 - x[0], U);
        fold_line(-L2 - x[1], L2 - x[1], V);
        z2 = x[2] * x[2];
    }
    __device__ __forceinline__ void agree(bool) {}
    // bins wlo .. whi of each quadrant reach the sink; each edge is evaluated
    // on its own, so the walk starts at max(mfirst, wlo)
    template <class Sink>
    __device__ __forceinline__ void sweep(int wlo, int whi, Sink& sink, double r0)
    {
        // the lane's non-empty quadrants first, so lanes step through their k-th
        // quadrant together
        int list = 0, nq = 0;
#pragma unroll
        for (int qi = 0; qi < 4; ++qi) {
            const int i = qi >> 1, j = qi & 1;
            const bool ok = i < U.n && j < V.n && (i ? U.hi[1] > U.lo[1] : U.hi[0] > U.lo[0]) &&
                            (j ? V.hi[1] > V.lo[1] : V.hi[0] > V.lo[0]);
            if (ok) { list |= qi << (2 * nq); ++nq; }
        }
#pragma unroll 1
        for (int t = 0; t < nq; ++t) {
            const int qi = (list >> (2 * t)) & 3;
            const int i = qi >> 1, j = qi & 1;
            const double a = i ? U.lo[1] : U.lo[0], b = i ? U.hi[1] : U.hi[0];
            const double c = j ? V.lo[1] : V.lo[0], d = j ? V.hi[1] : V.hi[0];
            const float w = (i ? U.w[1] : U.w[0]) * (j ? V.w[1] : V.w[0]);
            if constexpr (NW >= 2) {
                PlaneQuad q;
                plane_setup(q, a, b, c, d, z2, w, r0);
                plane_sweep(q, wlo, whi, tab, sink);
            } else {
                ArcQuad<0> q;   // the plane's own coordinates, weight 1
                q.base2 = z2;
                q.wN = a; q.oN = a * a;
                q.wF = b; q.oF = b * b;
                q.P[0] = 0.5 * w; q.Q[0] = w;
                arc_finish<0, 1>(q, c, d, r0);
                arc_sweep<0, 1, NW>(q, r0, wlo, whi, tab, sink);
            }
        }
    }
};

__device__ __forceinline__ double wrap_pi(double u)
{
    if (u <= -M_PI) u += 2.0 * M_PI;
    if (u <= -M_PI) u += 2.0 * M_PI;
    if (u > M_PI) u -= 2.0 * M_PI;
    if (u > M_PI) u -= 2.0 * M_PI;
    return u;
}

// The interval ends of the folded quadrants live in LDS (one column per thread,
// kBoxSlots doubles), read back per quadrant: kept in registers they would be
// live through every sweep and pushed to scratch memory at three or four waves
// per SIMD.
constexpr int kBoxSlots = 8;

// MERGE of the folded intervals holds for every I_l that is a difference of a
// function of the end points (exact, tables); not for the chord.
template <int NW, int IL, int STRIDE = kThreads>   // STRIDE: threads of the work-group (the table's row)
struct CylinderPair {
    static constexpr bool kMerge = IL != kIlTrapezoid;
    CyPair P;
    double* box;             // this thread's column of the LDS box table
    int list, nq;            // non-empty quadrants (2 bits each, in sweep order) and their number
    int wbits;               // quadrant weights: bits 0/1 the U intervals, 2/3 the V intervals (set = 2)
    __device__ __forceinline__ void bind(double* table, const double2* lut, const double*, const TrDev*, int, int, int)
    {
        box = table + threadIdx.x;
        P.lut = lut;
    }
    __device__ __forceinline__ void setup(const TrDev& T, const double x[3], double)
    {
        WInt U, V;
        double R = T.p[0], th = T.p[1], Lz = T.p[2];
        // a voxel on the focal line (rho = 0, Sec. 4.2) has no angular position;
        // rounding of its frame coordinates leaves rho at ~1e-16 of them, which
        // is snapped to 0 so that its angle is 0 rather than an arbitrary one
        double rho = sqrt64(x[0] * x[0] + x[1] * x[1]);
        if (rho <= 1e-10 * R) rho = 0.0;
        double thi = (rho > 0.0) ? atan2_full(x[1], x[0]) : 0.0;
        P.R = R;
        P.dm = fabs(R - rho);
        P.mu = 4.0 * R * rho;
        P.imu = P.mu > 0.0 ? rcp64_full(P.mu) : 0.0;
        double u1 = wrap_pi(-th - thi), u2 = wrap_pi(th - thi);
        // Eq. folded_intervals (merged where the areas are exact, see split_at_zero)
        if (u1 < 0.0 && 0.0 < u2) {
            split_at_zero<kMerge>(-u1, u2, U);
        } else if (u2 < u1) {
            // [u1, pi] and [-u2, pi]
            if (!kMerge) {
                U.lo[0] = u1;  U.hi[0] = M_PI; U.w[0] = 1.0f;
                U.lo[1] = -u2; U.hi[1] = M_PI; U.w[1] = 1.0f;
            } else {
                double m = fmax(u1, -u2), M = fmin(u1, -u2);
                U.lo[0] = m; U.hi[0] = M_PI; U.w[0] = 2.0f;
                U.lo[1] = M; U.hi[1] = m;    U.w[1] = 1.0f;
            }
            U.n = 2;
        } else if (0.0 <= u1) {
            U.lo[0] = u1; U.hi[0] = u2; U.w[0] = 1.0f; U.n = 1;
        } else {
            U.lo[0] = -u2; U.hi[0] = -u1; U.w[0] = 1.0f; U.n = 1;
        }
        fold_line<kMerge>(-Lz - x[2], Lz - x[2], V);
        // the non-empty quadrants in decreasing order of their number of bins
        // (nearest to farthest corner, estimated in FP32): the wave steps
        // through every lane's t-th quadrant together, so the lanes' longest
        // sweeps share one trip count
        bool ok[4];
        float len[4];
        {
            const float muf = (float)P.mu, dm2 = (float)(P.dm * P.dm);
            float pa[2], pb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float sa = __sinf(0.5f * (float)(i < U.n ? U.lo[i] : 0.0));
                const float sb = __sinf(0.5f * (float)(i < U.n ? U.hi[i] : 0.0));
                pa[i] = fmaf(muf * sa, sa, dm2);
                pb[i] = fmaf(muf * sb, sb, dm2);
            }
#pragma unroll
            for (int qi = 0; qi < 4; ++qi) {
                const int i = qi >> 1, j = qi & 1;
                ok[qi] = i < U.n && j < V.n && (i ? U.hi[1] > U.lo[1] : U.hi[0] > U.lo[0]) &&
                         (j ? V.hi[1] > V.lo[1] : V.hi[0] > V.lo[0]);
                const float c = (float)(j < V.n ? V.lo[j] : 0.0), d = (float)(j < V.n ? V.hi[j] : 0.0);
                len[qi] = ok[qi] ? fmaxf(sqrt_t(fmaf(d, d, pb[i])) - sqrt_t(fmaf(c, c, pa[i])), 0.0f) : -1.0f;
            }
        }
        list = 0;
        nq = 0;
#pragma unroll
        for (int qi = 0; qi < 4; ++qi) {
            int rank = 0;
#pragma unroll
            for (int qj = 0; qj < 4; ++qj)
                rank += (qj != qi) && (len[qj] > len[qi] || (len[qj] == len[qi] && qj < qi));
            if (ok[qi]) { list |= qi << (2 * rank); ++nq; }
        }
        wbits = (U.w[0] > 1.5f ? 1 : 0) | (U.w[1] > 1.5f ? 2 : 0) | (V.w[0] > 1.5f ? 4 : 0) |
                (V.w[1] > 1.5f ? 8 : 0);
        box[0 * STRIDE] = U.lo[0]; box[1 * STRIDE] = U.hi[0];
        box[2 * STRIDE] = U.lo[1]; box[3 * STRIDE] = U.hi[1];
        box[4 * STRIDE] = V.lo[0]; box[5 * STRIDE] = V.hi[0];
        box[6 * STRIDE] = V.lo[1]; box[7 * STRIDE] = V.hi[1];
    }
    __device__ __forceinline__ void quadrant(int qi, double& a, double& b, double& c, double& d, double& w) const
    {
        const int i = qi >> 1, j = qi & 1;
        a = box[(2 * i) * STRIDE]; b = box[(2 * i + 1) * STRIDE];
        c = box[(4 + 2 * j) * STRIDE]; d = box[(5 + 2 * j) * STRIDE];
        w = (double)((1 + ((wbits >> i) & 1)) * (1 + ((wbits >> (2 + j)) & 1)));
    }
    __device__ __forceinline__ void agree(bool) {}
    // bins wlo .. whi of each quadrant reach the sink; each edge is evaluated
    // on its own, so the walk starts at max(mfirst, wlo)
    template <class Sink>
    __device__ __forceinline__ void sweep(int wlo, int whi, Sink& sink, double r0)
    {
#pragma unroll 1
        for (int t = 0; t < nq; ++t) {
            double a, b, c, d, w;
            quadrant((list >> (2 * t)) & 3, a, b, c, d, w);
            CyQuad q;
            cy_setup(q, P, a, b, c, d, r0);
            cy_sweep<NW, IL>(q, P, r0, wlo, whi, w, sink);
        }
    }
};

// Which levels of the weight's polynomials serve a pair, whose u-intervals end at the
// cosines [c0, c1] and [cm, cp] (where ok): least <= level <= most (most = -1: none).
// They cover |tau| <= eta of x = w^2 / mu on its side of pi/2.  The recurrence of the
// J_j loses (vmax^2 / (mu (1 - xc)))^n roundings, so voxels closer to the focal line
// than kappa, and within 1e-7 R of it, keep the elliptic integral.  So do, with FP64
// input and output, those whose interval reaches u = pi, although the weight fits
// them and is closer there (worst bin of a pair against 30 digits, elements of an arc:
// 5e-14 to 2.5e-13 against 5e-12 to 9e-11, as the integral's end points round there by up to
// 1e-8 of a bin): taking it moves the FP64 signals of such arrays by up to 2.5e-9,
// where 1e-9 of the earlier ones was kept.
struct ArcFit {
    int least, most;
    __host__ __device__ bool fits() const { return least <= most; }
};
template <int NW>
__host__ __device__ inline ArcFit arc_fit(double R, double rho, double c0, double c1, double cm, double cp, bool ok0,
                                          bool ok1, double vmax, bool inpi)
{
    constexpr int top = Levels<NW>::n - 1;
    const double mu = 4.0 * R * rho, v2 = vmax * vmax;
    ArcFit r{0, mu >= 4e-7 * R * R && !(NW >= 2 && inpi) ? top : -1};
    for (int i = 0; i < 2; ++i) {
        if (!(i ? ok1 : ok0)) continue;
        const double ca = i ? cm : c0, cb = i ? cp : c1, g = ca + cb > 0.0 ? 0.5 : -0.5;
        const double xa = fma(-g, ca, 0.5), xb = fma(-g, cb, 0.5);
        const double one = 1.0 - 0.5 * (xa + xb), del = 0.5 * fabs(xb - xa), m1 = mu * one;
        const int least = (del > Weight<NW, 0>::eta * one) + (del > Weight<NW, 1>::eta * one) +
                          (top > 2 && del > Weight<NW, top - 1>::eta * one) + (del > Weight<NW, top>::eta * one);
        const int most = (v2 <= Weight<NW, 0>::kappa * m1) + (v2 <= Weight<NW, 1>::kappa * m1) +
                         (top > 2 && v2 <= Weight<NW, top - 1>::kappa * m1) + (v2 <= Weight<NW, top>::kappa * m1) - 1;
        r.least = r.least > least ? r.least : least;
        r.most = r.most < most ? r.most : most;
    }
    return r;
}

// One pair by its elliptic integrals, out of line: the few pairs that need it
// would otherwise cost every other one registers (inlined, 84 were spilled; now
// 20 to 47, outside the loops over edges).  The sink travels by value, with LDS
// pointers typed as such.
template <int NW, int STRIDE, class Sink>
__device__ __attribute__((noinline)) Sink carlson_pair(const TrDev* tr, int ix, int iy, int iz, int wlo, int whi,
                                                        double r0, LdsDouble* box, Sink sink)
{
    const TrDev T = *tr;
    double x[3];
    frame_coords(T, ix, iy, iz, x);
    CylinderPair<NW, kIlExact, STRIDE> pair;
    pair.box = (double*)box;
    pair.P.lut = nullptr;
    pair.setup(T, x, r0);
    pair.sweep(wlo, whi, sink, r0);
    return sink;
}

// Exact I_l: the quadrants as weighted areas (arc_sweep), for a pair whose
// folded u-intervals the weight's polynomials cover, else Carlson's integral
// (CylinderPair).  The ends of the intervals are kept as cos and sin, which the
// frame coordinates give without an inverse function.
template <int NW, int STRIDE>
struct ArcCylinderPair {
    double R, rho;
    double* box;             // this thread's column of the LDS box table
    const double* tab;
    int list, nq;            // non-empty quadrants (2 bits each, in sweep order) and their number
    int bits;                // bit 0 / 1: U / V interval 0 has weight 2; bit 2 / 3: U interval 0 ends at
                             // u = 0 / pi; bits 4-5: the weight's least level; bits 6-8: the number of
                             // levels that serve from the lowest on, 0 for Carlson's path
    int level;               // the pair's own, the wave's after agree()
    const TrDev* tr;         // the pair, for Carlson's path
    int ix, iy, iz;
    __device__ __forceinline__ void bind(double* table, const double2*, const double* t, const TrDev* T, int x, int y,
                                         int z)
    {
        box = table + threadIdx.x;
        tab = t;
        tr = T;
        ix = x;
        iy = y;
        iz = z;
    }
    // w^2 / mu = sin^2(u/2) from cos u and sin u, without cancellation for small u
    static __device__ __forceinline__ double half_sin2(double c, double s)
    {
        return c >= 0.0 ? s * s * rcp_nw<NW>(fma(2.0, c, 2.0)) : fma(-0.5, c, 0.5);
    }
    __device__ __forceinline__ void setup(const TrDev& T, const double x[3], double r0)
    {
        R = T.p[0];
        const double n2 = fma(x[0], x[0], x[1] * x[1]);
        const double ir = rsq64(fmax(n2, 1e-300));
        rho = n2 * ir;
        const double ct = x[0] * ir, st = fabs(x[1]) * ir;   // cos and sin of |theta_i|
        // u = |theta_i| -+ theta_max (Eq. folded_intervals; the sign of theta_i
        // does not matter): [0, -u-] twice and [-u-, u+] when 0 is inside, [2 pi -
        // u+, pi] twice and [u-, 2 pi - u+] when pi is, else [u-, u+]
        const double cm = fma(ct, T.cth, st * T.sth), sm = fma(st, T.cth, -ct * T.sth);
        const double cp = fma(ct, T.cth, -st * T.sth), sp = fma(st, T.cth, ct * T.sth);
        const bool in0 = sm < 0.0, inpi = !in0 && sp < 0.0;
        WInt V;
        fold_line(-T.p[2] - x[2], T.p[2] - x[2], V);
        const double c0 = in0 ? 1.0 : inpi ? cp : cm, c1 = in0 ? cm : inpi ? -1.0 : cp;
        const bool uok[2] = {c0 > c1, (in0 || inpi) && cm > cp};
        const double vmax = V.n == 2 ? V.hi[1] : V.hi[0];
        bits = (in0 || inpi ? 1 : 0) | (V.n == 2 ? 2 : 0) | (in0 ? 4 : 0) | (inpi ? 8 : 0);
        const ArcFit fit = arc_fit<NW>(R, rho, c0, c1, cm, cp, uok[0], uok[1], vmax, inpi);
        level = 0;
        if (!fit.fits()) return;
        level = fit.least;
        // the non-empty quadrants in decreasing order of their number of bins
        // (nearest to farthest corner, estimated in FP32): the wave steps
        // through every lane's t-th quadrant together, so the lanes' longest
        // sweeps share one trip count
        bool ok[4];
        float len[4];
        {
            const float b2 = (float)fma(R, R, rho * rho), r2 = (float)(2.0 * R * rho);
            const float p0 = fmaf(-r2, (float)c0, b2), p1 = fmaf(-r2, (float)c1, b2);
            const float pm = fmaf(-r2, (float)cm, b2), pp = fmaf(-r2, (float)cp, b2);
            const float pa[2] = {p0, pm}, pb[2] = {p1, pp};
#pragma unroll
            for (int qi = 0; qi < 4; ++qi) {
                const int i = qi >> 1, j = qi & 1;
                ok[qi] = uok[i] && j < V.n && (j ? V.hi[1] > V.lo[1] : V.hi[0] > V.lo[0]);
                const float c = (float)(j < V.n ? V.lo[j] : 0.0), d = (float)(j < V.n ? V.hi[j] : 0.0);
                len[qi] = ok[qi] ? fmaxf(sqrt_t(fmaf(d, d, pb[i])) - sqrt_t(fmaf(c, c, pa[i])), 0.0f) : -1.0f;
            }
        }
        list = 0;
        nq = 0;
#pragma unroll
        for (int qi = 0; qi < 4; ++qi) {
            int rank = 0;
#pragma unroll
            for (int qj = 0; qj < 4; ++qj)
                rank += (qj != qi) && (len[qj] > len[qi] || (len[qj] == len[qi] && qj < qi));
            if (ok[qi]) { list |= qi << (2 * rank); ++nq; }
        }
        bits |= (fit.least << 4) | (fit.most + 1) << 6;
        box[0 * STRIDE] = cm; box[1 * STRIDE] = fabs(sm);
        box[2 * STRIDE] = cp; box[3 * STRIDE] = fabs(sp);
        box[4 * STRIDE] = V.lo[0]; box[5 * STRIDE] = V.hi[0]; box[6 * STRIDE] = V.hi[1];
    }
    // One level of the weight for the wave's lanes, which are neighbouring voxels; a lane
    // it does not serve takes Carlson's path.  All the cube's voxels take part, whether
    // or not they have a coefficient, so the forward of any volume, alone or beside
    // others, by cubes or by time tiles, and the adjoint use the same areas (to the
    // rounding of the arc's angle, whose series the active lanes choose: 2e-15 of a
    // signal).  The sparse forward's waves are of listed voxels: its areas differ by
    // the weight's error.
    __device__ __forceinline__ void agree(bool valid)
    {
        const int own = valid ? (bits >> 4) & 3 : 0;
        level = __any(own > 2) ? 3 : __any(own > 1) ? 2 : __any(own > 0) ? 1 : 0;
    }
    // p(om) = scale (1 - x)^(-1/2): Weight's polynomial in tau = al om + be, expanded
    template <class Wt>
    static __device__ __forceinline__ void weight(ArcQuad<Wt::n>& q, double al, double be, double scale)
    {
        constexpr int N = Wt::n;
        double p[N + 1];
#pragma unroll
        for (int i = 0; i <= N; ++i) p[i] = 0.0;
        p[0] = Wt::c[N];
#pragma unroll
        for (int j = N - 1; j >= 0; --j) {
#pragma unroll
            for (int i = N - j; i > 0; --i) p[i] = fma(be, p[i], al * p[i - 1]);
            p[0] = fma(be, p[0], Wt::c[j]);
        }
#pragma unroll
        for (int j = 0; j <= N; ++j) {
            p[j] *= scale;
            q.P[j] = p[j] * (1.0 / (2 * j + 2));
            q.Q[j] = p[j] * (1.0 / (2 * j + 1));
        }
    }
    template <class Wt, int S, class Sink>
    __device__ __forceinline__ void arc(double xN, double xF, double c, double d, double w, double mu, double r0,
                                        int wlo, int whi, Sink& sink) const
    {
        constexpr int N = Wt::n;
        ArcQuad<N> q;
        const double b = S > 0 ? R - rho : R + rho;
        q.base2 = b * b;
        const double o1 = mu * xN, o2 = mu * xF;
        q.wN = sqrt64<NW>(o1); q.oN = S * o1;
        q.wF = sqrt64<NW>(o2); q.oF = S * o2;
        const double xc = 0.5 * (xN + xF), ione = rcp_nw<NW>(1.0 - xc);
        const double smu = rsq64<NW>(mu);   // 1 / sqrt(mu)
        weight<Wt>(q, S * ione * (smu * smu), -xc * ione, S * w * 2.0 * R * (smu * sqrt64<NW>(ione)));
        arc_finish<N, S>(q, c, d, r0);
        arc_sweep<N, S, NW>(q, r0, wlo, whi, tab, sink);
    }
    template <class Wt, class Sink>
    __device__ __forceinline__ void arcs(int wlo, int whi, Sink& sink, double r0) const
    {
        const double mu = 4.0 * R * rho;
#pragma unroll 1
        for (int t = 0; t < nq; ++t) {
            const int qi = (list >> (2 * t)) & 3;
            const int i = qi >> 1, j = qi & 1;
            double ca = box[0 * STRIDE], sa = box[1 * STRIDE], cb = box[2 * STRIDE], sb = box[3 * STRIDE];
            if (i == 0 && (bits & 4)) { cb = ca; sb = sa; ca = 1.0; sa = 0.0; }
            if (i == 0 && (bits & 8)) { ca = cb; sa = sb; cb = -1.0; sb = 0.0; }
            const double c = j ? box[5 * STRIDE] : box[4 * STRIDE], d = j ? box[6 * STRIDE] : box[5 * STRIDE];
            const double w = (double)((1 + ((bits & 1) & ~i)) * (1 + (((bits >> 1) & 1) & ~j)));
            if (ca + cb > 0.0)   // the middle of [a, b] is below pi/2
                arc<Wt, 1>(half_sin2(ca, sa), half_sin2(cb, sb), c, d, w, mu, r0, wlo, whi, sink);
            else
                arc<Wt, -1>(half_sin2(-ca, sa), half_sin2(-cb, sb), c, d, w, mu, r0, wlo, whi, sink);
        }
    }
    // bins wlo .. whi of each quadrant reach the sink; each edge is evaluated
    // on its own, so the walk starts at max(mfirst, wlo)
    template <int LEVEL, class Sink>
    __device__ __forceinline__ void arcs_or_carlson(int wlo, int whi, Sink& sink, double r0)
    {
        if ((bits >> 6) <= LEVEL)
            sink.take(carlson_pair<NW, STRIDE>(tr, ix, iy, iz, wlo, whi, r0, (LdsDouble*)box, sink.give()));
        else
            arcs<Weight<NW, LEVEL>>(wlo, whi, sink, r0);
    }
    template <class Sink>
    __device__ __forceinline__ void sweep(int wlo, int whi, Sink& sink, double r0)
    {
        if (Levels<NW>::n > 3 && level == 3)
            arcs_or_carlson<Levels<NW>::n - 1>(wlo, whi, sink, r0);
        else if (level == 2)
            arcs_or_carlson<2>(wlo, whi, sink, r0);
        else if (level == 1)
            arcs_or_carlson<1>(wlo, whi, sink, r0);
        else
            arcs_or_carlson<0>(wlo, whi, sink, r0);
    }
};

// Areas are FP64 in both variants (they are differences between edges).  With
// FP32 input and output one correction step after the FP32 seeds of the square
// roots and reciprocals (2^-46 after it) is enough; the FP64 variant takes two
// after the FP64 ones.
template <class Real> struct Newton { static constexpr int value = 2; };
template <> struct Newton<float> { static constexpr int value = 1; };

// IL: how the cylinder's I_l is evaluated (kIlExact, kIlCarlson, kIlTrapezoid, kIlTable);
// the planar area is exact either way
template <int SHAPE, class Real, int IL, int STRIDE = kThreads> struct PairOf;
template <class Real, int IL, int STRIDE> struct PairOf<0, Real, IL, STRIDE> {
    using type = PlanarPair<Newton<Real>::value>;
};
template <class Real, int IL, int STRIDE> struct PairOf<1, Real, IL, STRIDE> {
    using type = CylinderPair<Newton<Real>::value, IL, STRIDE>;
};
template <class Real, int STRIDE> struct PairOf<1, Real, kIlExact, STRIDE> {
    using type = ArcCylinderPair<Newton<Real>::value, STRIDE>;
};
template <class Real, int STRIDE> struct PairOf<1, Real, kIlCarlson, STRIDE> {
    using type = CylinderPair<Newton<Real>::value, kIlExact, STRIDE>;
};

}  // namespace patop
