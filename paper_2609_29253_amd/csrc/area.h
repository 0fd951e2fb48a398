// Shell areas |M_i^m| of one voxel on one transducer, device side.
//
// A bin m is the radial interval [r0 + m - 1, r0 + m) in units of dr = c/(U fs).
// Both geometries use the paper's separable form (Sec. 4, Eq. separable): the
// squared distance is psi(u) + v^2 on a parameter rectangle D, which is split
// into at most four quadrants reflected to u, v >= 0 (Eq. uvminmax, folded
// intervals Eq. folded_intervals for the cylinder), each of the form
// [a, b] x [c, d].  A sweep walks the bins a quadrant touches (between its
// nearest corner distance D_ac and farthest D_bd, Eq. closedform_rminrmax) and
// hands each bin's area to a sink.
//
// Exact areas (planar, Sec. 4.1, and cylinder, Sec. 4.2): the closed form as the
// difference of an elementary function between the bin's two edges (arc_sweep),
// with the cylinder's curvature as a polynomial weight.  Elliptic integrals are
// left to the quadrants whose weight the polynomials do not cover.
//
// Cylinder (Sec. 4.2): psi(u) = (R - rho)^2 + 4 R rho sin^2(u/2).  Alg. 4 is
// followed literally (triples carried from edge to edge, Eq. area_D_l_xi,
// Eq. cyl_Il), in FP64: the cylinder's I_l is a difference of nearly equal
// elliptic integrals.  E(beta/2, nu) - E(alpha/2, nu) is evaluated by Legendre's
// addition theorem, E(phi) - E(psi) = E(sigma) - nu sin phi sin psi sin sigma, so
// only one Carlson evaluation, at the amplitude sigma of the difference, is needed
// (E = s R_F(c^2, 1 - nu s^2, 1) - nu/3 s^3 R_D(c^2, 1 - nu s^2, 1), valid for
// nu > 1 whenever nu s^2 <= 1, Lemma exact_integral).  The half angles of the
// clamped inverse Phi (Eq. alphabeta) come from
//   sin^2(u/2) = (s - v^2 - (R - rho)^2) / (4 R rho),
//   1 - nu sin^2(u/2) = v^2 / (s - (R - rho)^2),
// so arccos is never evaluated.
//
// Two cheaper I_l replace the Carlson evaluation (selected by IL): the chord of
// the level curve (Eq. trapezoid_Il) and the lookup tables of E~, F~ (Sec. 4.2,
// LUT paragraph), E(beta/2) - E(alpha/2) read off bilinearly at both end points.
#pragma once

#include <hip/hip_runtime.h>

#include "patop_internal.h"

namespace patop {

// ---------------------------------------------------------------------------
// small numeric helpers
// ---------------------------------------------------------------------------

// Seeds of the FP64 reciprocal and reciprocal square root.  NW = 1 (one
// correction step, the kernels with FP32 input and output): the FP32 instructions
// v_rcp_f32 / v_rsq_f32 (1 ulp, 2^-23), which on gfx950 cost, with their two
// conversions, about half of v_rcp_f64 / v_rsq_f64; one Newton step then leaves
// 2^-46 (rcp) and 1.5 x 2^-46 (rsq) relative error.  Their arguments must lie
// in the FP32 normal range (or be <= 0 where the result is not used).  NW >= 2:
// the FP64 instructions (~2^-24), two steps to full precision.
template <int NW>
__device__ __forceinline__ double rcp_seed(double x)
{
    if (NW == 1) return (double)__builtin_amdgcn_rcpf((float)x);
    return __builtin_amdgcn_rcp(x);
}
template <int NW>
__device__ __forceinline__ double rsq_seed(double x)
{
    if (NW == 1) return (double)__builtin_amdgcn_rsqf((float)x);
    return __builtin_amdgcn_rsq(x);
}

// the offset that keeps square-root arguments positive (and, for NW = 1, in
// the FP32 normal range of the seeds); below any length or cosine that enters
// a sum here
template <int NW> struct Tiny { static constexpr double value = 1e-300; };
template <> struct Tiny<1> { static constexpr double value = 1e-30; };

// 1/x with one Newton step
template <int NW = 2>
__device__ __forceinline__ double rcp64(double x)
{
    double r = rcp_seed<NW>(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// a * b + c as one three-operand v_fma_f64 with the addend c in a register.
// Horner steps add a loop-invariant constant; left to itself the compiler
// copies it into the destination of a two-operand v_fmac_f64, one extra
// instruction per step.  b is a register too ("v") or, for a constant
// multiplier, a scalar register ("s").
__device__ __forceinline__ double fma_vvv(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ double fma_vsv(double a, double b, double c)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// 1/x with a second Newton step (full precision)
__device__ __forceinline__ double rcp64_full(double x)
{
    double r = rcp64(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// v_rsq_f64 is accurate to ~2^-24: each Newton step doubles the correct bits
// (one step: ~2^-48, two: full precision)
template <int NEWTON = 2>
__device__ __forceinline__ double rsq64(double x)
{
    double r = rsq_seed<NEWTON>(x);
#pragma unroll
    for (int i = 0; i < NEWTON; ++i) {
        double h = 0.5 * x * r;
        r = fma(r, fma(-h, r, 0.5), r);
    }
    return r;
}

// sqrt of x > 0 from y = v_rsq_f64(x) (relative error ~2^-24): g = x y is
// corrected by the residual x - g^2 times h = y/2 (one step: ~2^-48); two
// steps first refine g and h together (Goldschmidt), then take the residual
// step (full precision)
template <int NEWTON = 2>
__device__ __forceinline__ double sqrt64_pos(double x)
{
    const double y = rsq_seed<NEWTON>(x);
    double g = x * y, h = 0.5 * y;
    if (NEWTON >= 2) {
        const double r = fma(-g, h, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
    }
    return fma(fma(-g, g, x), h, g);
}

// sqrt(max(x, tiny)): branch free; returns sqrt(tiny) (1e-150, or 1e-15 with the
// FP32 seeds) instead of 0 for x <= 0, below any length or cosine that enters a
// sum here
template <int NEWTON = 2>
__device__ __forceinline__ double sqrt64(double x)
{
    return sqrt64_pos<NEWTON>(fmax(x, Tiny<NEWTON>::value));
}

// FP32 square root as the one v_sqrt_f32 (1 ulp); the IEEE-rounded sqrtf the
// compiler emits otherwise adds a denormal rescale and a correction step
// (some 15 instructions)
__device__ __forceinline__ float sqrt_t(float x) { return __builtin_amdgcn_sqrtf(fmaxf(x, 0.0f)); }

// ---------------------------------------------------------------------------
// areas as differences of a weighted area in a plane: planar quadrants, and
// cylinder quadrants with the exact I_l
// ---------------------------------------------------------------------------
// With w = sqrt(mu) sin(u/2) the cylinder's level curve psi(u) + v^2 = r^2 is the
// circle w^2 + v^2 = K, K = r^2 - (R - rho)^2, and with t = sqrt(mu) cos(u/2) the
// hyperbola v^2 - t^2 = K, K = r^2 - (R + rho)^2; the surface element R du dv
// becomes h dw dv with the weight h = 2 R / sqrt(mu (1 - x)), x = w^2 / mu
// (resp. t^2 / mu).  h is smooth away from x = 1, so each quadrant takes it as a
// polynomial p in om = S w^2 (S = +1 circle, -1 hyperbola), on the side of u =
// pi/2 that keeps x away from 1, and the area nearer than r,
//   int p(om) [clamp(y, c, d) - c] dw,   y = sqrt(K - om),
// is elementary: with J_j = int om^j y dw,
//   (2j + 2) J_j = (2j - 1) K J_{j-1} - w om^{j-1} y^3,   2 J_0 = w y + K Lambda,
// Lambda = int dw / y the angle (or hyperbolic angle) the arc subtends.  An error
// eps of p changes each area by at most eps of itself, whatever the cancellation
// between edges, and costs no elliptic integral: two square roots, one inverse
// function and about 6 N + 35 further FP64 operations per edge, with no loop
// whose length differs between lanes.  A rectangle is the case h = 1, N = 0, with FP32
// input and output; with FP64 it has a form of its own (PlaneQuad).
//
// The sweep is bound by VALU issue (1.02 of the SIMD cycles on 256^3 x 512
// rectangles, at four cycles a wave instruction; FP32 ones issue faster): 71 instructions per edge of a
// rectangle, 113 to 137 of a cylinder, where Carlson's integral by Legendre's
// addition theorem took 271 per edge and a walk of FP32 pieces between the
// rectangle's corners 194 per bin.  With FP32 input and output A went from 448 to
// 265 ms on 256^3 x 512 rectangles and from 142 to 65 ms on 128^3 x 256 cylinders
// (the order and number of the work-groups in it: 275 -> 263 and 69 -> 61, with weights
// of a lower degree).  Errors of the FP32 signals against 64 bits, 32^3 x 64
// rectangles: 1.5e-7 -> 2.6e-8.
//
// End points of the arc: alpha starts clamped at the quadrant's near end N (u =
// a) and moves along the line v = d once K passes the corner (N, d); beta moves
// along v = c until the corner (F, c) and is then clamped at the far end F.

// h's factor (1 - x)^(-1/2) = (1 - xc)^(-1/2) (1 - tau)^(-1/2), tau = (x - xc) /
// (1 - xc): interpolants of degree n at Chebyshev nodes on |tau| <= eta, by level.
// Relative error with FP32 input and output 1.9e-11, 2.2e-11, 2.3e-11 and 5.7e-11, three
// orders below the output's rounding: about what Carlson's integral leaves in the median,
// less in the worst (worst bin of a pair over its largest, median / 95 % / worst, Carlson and this: elements
// of a scan at U = 1 1.7e-11 / 2.4e-10 / 2.3e-9 and 2.0e-11 / 7e-11 / 1.1e-10, at U = 11 2.1e-10 /
// 1.9e-9 / 2e-8 and 3.3e-11 / 5e-10 / 1e-9, of an arc 5e-8 / 1.4e-7 / 1.7e-7 and 1.1e-11 /
// 1.8e-11 / 2e-11); with FP64 6.2e-14, 1.0e-13 and 3.3e-13.  A / A^T of 128^3 x 256 cylinders,
// A^T of the scan of 200^3 x 64 in ms: 64.6 / 67.8, 73.1; without the first level 66.1 /
// 69.0, 72.8; degrees 4, 5, 7 on 0.04, 0.08, 0.16, which leave 1.6e-9 whatever the element,
// 62.1 / 64.6, 67.6.  kappa bounds vmax^2 / (mu (1 - xc)), whose n-th power multiplies the
// roundings of the J_j.
template <int NW, int LEVEL> struct Weight;
// (levels, the lowest degree first)
template <int NW> struct Levels { static constexpr int n = 3; };
template <> struct Levels<1> { static constexpr int n = 4; };
template <> struct Weight<1, 0> {
    static constexpr int n = 4;
    static constexpr double eta = 0.0165, kappa = 3.2;
    static constexpr double c[n + 1] = {
        1.0, 0.49999999429819714, 0.374999994773313, 0.31258376819134176, 0.27351428791320237};
};
template <> struct Weight<1, 1> {
    static constexpr int n = 5;
    static constexpr double eta = 0.038, kappa = 2.6;
    static constexpr double c[n + 1] = {
        1.0000000000212659, 0.5000000000197475, 0.3749997349316204, 0.31249975385743234, 0.27392681105161915,
        0.24654812125416245};
};
template <> struct Weight<1, 2> {
    static constexpr int n = 7;
    static constexpr double eta = 0.104, kappa = 2.0;
    static constexpr double c[n + 1] = {
        0.9999999999785899, 0.4999999999797752, 0.37500006332410346, 0.3125000598183644, 0.27340827460690964,
        0.24606614306016883, 0.22989139768446637, 0.2135395082670361};
};
template <> struct Weight<1, 3> {
    static constexpr int n = 8;
    static constexpr double eta = 0.16, kappa = 1.8;
    static constexpr double c[n + 1] = {
        1.0, 0.49999999704787307, 0.3749999971941834, 0.3125015348867947, 0.27343895879424956,
        0.2458789227748675, 0.2253817687557605, 0.22053917177169305, 0.20689706937941357};
};
template <> struct Weight<2, 0> {
    static constexpr int n = 7;
    static constexpr double eta = 0.05, kappa = 1.3;
    static constexpr double c[n + 1] = {
        0.9999999999999398, 0.49999999999994316, 0.37500000077050993, 0.31250000072773826, 0.27343595956342226,
        0.24609229508034408, 0.2265708771687404, 0.21040290777839668};
};
template <> struct Weight<2, 1> {
    static constexpr int n = 8;
    static constexpr double eta = 0.08, kappa = 1.2;
    static constexpr double c[n + 1] = {
        1.0, 0.49999999998891637, 0.37499999998946937, 0.3125000230808288, 0.27343752192922083,
        0.24608078231340225, 0.22557361695740225, 0.21216685744128233, 0.19894030261705037};
};
template <> struct Weight<2, 2> {
    static constexpr int n = 10;
    static constexpr double eta = 0.16, kappa = 1.0;
    static constexpr double c[n + 1] = {
        1.0, 0.5000000000212094, 0.3750000000203339, 0.31249998344974184, 0.2734374841330066,
        0.2460973593854478, 0.2255893978103804, 0.20915235533051377, 0.19607355491324047, 0.1978170102153056,
        0.1880321370533884};
};

// Lambda's inverse function f, f(x) = x + x^3 P(x^2): P by interpolation at Chebyshev
// nodes of x^2, for atan (S = 1) and atanh (S = -1), on x <= 1/8 and on x <=
// 0.42; relative error 2e-15 and 1.3e-13 (NW = 1), 7e-18 and 5e-17 (NW = 2)
template <int S, int NW> struct ArcSeries;
template <> struct ArcSeries<1, 1> {
    static constexpr double lo[5] = {
        -0.33333333333319803, 0.19999999956695652, -0.14285692082379586, 0.11107119763160542,
        -0.08796919798324465};
    static constexpr double hi[8] = {
        -0.3333333333325081, 0.19999999940043187, -0.14285707102889028, 0.11110781342546695,
        -0.09083412043223445, 0.0759848113690192, -0.05998786787867099, 0.03245379438372544};
};
template <> struct ArcSeries<1, 2> {
    static constexpr double lo[6] = {
        -0.33333333333333287, 0.19999999999790477, -0.14285714129116034, 0.1111106826170422,
        -0.09085599506798686, 0.07387718384425714};
    static constexpr double hi[11] = {
        -0.3333333333333333, 0.19999999999994217, -0.14285714284398277, 0.11111110993987848,
        -0.09090903726254194, 0.0769216368130413, -0.06664240513226126, 0.05855828347679443,
        -0.05073475931846312, 0.03889055030264144, -0.018764922473679908};
};
template <> struct ArcSeries<-1, 1> {
    static constexpr double lo[5] = {
        0.3333333333334781, 0.19999999953686995, 0.1428573796423765, 0.11106881256020994, 0.09398126834838963};
    static constexpr double hi[9] = {
        0.3333333333334639, 0.19999999988024808, 0.14285716086836603, 0.1111100729792487, 0.09093888604356387,
        0.07644687050656893, 0.0710737704056635, 0.03570834279784205, 0.11354190728849271};
};
template <> struct ArcSeries<-1, 2> {
    static constexpr double lo[6] = {
        0.3333333333333328, 0.20000000000227505, 0.14285714116012183, 0.11111157356123932, 0.09085223469123827,
        0.08013059813075277};
    static constexpr double hi[11] = {
        0.3333333333333336, 0.19999999999964782, 0.1428571429367304, 0.11111110411784622, 0.09090940491443848,
        0.0769148899584336, 0.06679888190163528, 0.05746567311921013, 0.06144227524817444,
        0.013262917513335266, 0.11309973802991415};
};

// atan(k / 32) and log(1 + k / 32), k = 0..32: the work-group copies them to LDS
// (kArcTab doubles) for the arguments above those
constexpr int kArcNodes = 33;
constexpr int kArcTab = 2 * kArcNodes;
static __device__ const double kArcTable[kArcTab] = {
    0.0, 0.031239833430268277, 0.06241880999595735, 0.09347678115858947, 0.12435499454676144,
    0.15499674192394097, 0.18534794999569476, 0.21535769969773805, 0.24497866312686414, 0.2741674511196588,
    0.3028848683749714, 0.3310960767041321, 0.35877067027057225, 0.38588266939807375, 0.4124104415973873,
    0.43833655985795783, 0.4636476090008061, 0.48833395105640554, 0.5123894603107377, 0.5358112379604637,
    0.5585993153435624, 0.5807563535676704, 0.6022873461349642, 0.6231993299340659, 0.6435011087932844,
    0.6632029927060933, 0.6823165548747481, 0.7008544078844502, 0.7188299996216245, 0.7362574289814281,
    0.7531512809621944, 0.7695264804056583, 0.7853981633974483,
    0.0, 0.030771658666753687, 0.06062462181643484, 0.08961215868968714, 0.11778303565638346,
    0.1451820098444979, 0.17185025692665923, 0.19782574332991987, 0.22314355131420976, 0.24783616390458127,
    0.27193371548364176, 0.2954642128938359, 0.3184537311185346, 0.3409265869705932, 0.3629054936893685,
    0.38441169891033206, 0.4054651081081644, 0.4260843953109001, 0.44628710262841953, 0.46608972992459924,
    0.4855078157817008, 0.5045560107523953, 0.5232481437645479, 0.5415972824327444, 0.5596157879354227,
    0.5773153650348236, 0.5947071077466928, 0.6118015411059929, 0.6286086594223741, 0.6451379613735847,
    0.661398482245365, 0.6773988235918061, 0.6931471805599453,
};

template <int S, int NW>
__device__ __forceinline__ double arc_series(double X)
{
    // X -+ X^3/3 + X^5/5 ... (S = +1 atan, -1 atanh) of a table's rest, |X| <= 1/64
    const double u = X * X;
    double p = NW == 1 ? 1.0 / 5 : fma(u, S > 0 ? -1.0 / 7 : 1.0 / 7, 1.0 / 5);
    p = fma(u, p, S > 0 ? -1.0 / 3 : 1.0 / 3);
    return fma(X * u, p, X);
}

// x + x^3 P(x^2)
template <int M>
__device__ __forceinline__ double arc_series(double x, const double (&c)[M])
{
    const double u = x * x;
    double p = c[M - 1];
#pragma unroll
    for (int j = M - 2; j >= 0; --j) p = fma(p, u, c[j]);
    return fma(x * u, p, x);
}

// 1/x to the accuracy of the variant: one Newton step on the FP32 seed, or two
// on the FP64 one
template <int NW>
__device__ __forceinline__ double rcp_nw(double x) { return NW >= 2 ? rcp64_full(x) : rcp64<1>(x); }

// num / den to the accuracy of the variant
template <int NW>
__device__ __forceinline__ double arc_quotient(double num, double den)
{
    const double r = NW >= 2 ? rcp64(den) : rcp_seed<1>(den), q = num * r;
    return fma(fma(-q, den, num), r, q);
}

// atan(num / den), num >= 0, den > 0, num <= den (beyond it only by rounding): the node k / 32 next to
// the quotient, by its FP32 estimate, and the series at the tangent of the rest
template <int NW>
__device__ __forceinline__ double arc_atan(double num, double den, const double* tab)
{
    const float t = (float)num * __builtin_amdgcn_rcpf((float)den);
    const float kf = rintf(fminf(fmaxf(t * 32.0f, 0.0f), 32.0f));
    const double G = (double)(kf * (1.0f / 32));
    const double X = fma(-G, den, num) * rcp_nw<NW>(fma(G, num, den));
    return tab[(int)kf] + arc_series<1, NW>(X);
}

// log(a / b), a >= b > 0 (below it only by rounding): exponent and the leading
// five bits of the quotient's FP32 estimate, then log of the rest = 2 atanh
template <int NW>
__device__ __forceinline__ double arc_log(double a, double b, const double* tab)
{
    const float qf = (float)a * __builtin_amdgcn_rcpf((float)b);
    const int g = __float_as_int(qf);
    const double G = (double)__int_as_float(g & 0x7ffc0000);
    const int k = (g >> 18) & 31, e = ((g >> 23) & 255) - 127;
    const double Gb = G * b;
    const double X = (a - Gb) * rcp_nw<NW>(a + Gb);
    return fma((double)e, 0.6931471805599453, fma(2.0, arc_series<-1, NW>(X), tab[kArcNodes + k]));
}

// one quadrant [N, F] x [c, d]: om and w of both ends, the squared distance of
// the plane, and p's coefficients p_j as P = p_j / (2j + 2) and Q = p_j / (2j + 1)
// times everything that multiplies the area
template <int N>
struct ArcQuad {
    double base2, oN, wN, oF, wF, c, d, c2, d2;
    double P[N + 1], Q[N + 1];
    double S0, S1;          // the area function at the nearest and the farthest corner
    int mfirst, mlast;      // bins touched
};

template <int N>
__device__ __forceinline__ double horner(const double* q, double x)
{
    double a = q[N];
#pragma unroll
    for (int j = N - 1; j >= 0; --j) a = fma(a, x, q[j]);
    return a;
}

// corners, the area function there and the bins; P and Q set
template <int N, int S>
__device__ __forceinline__ void arc_finish(ArcQuad<N>& q, double c, double d, double r0)
{
    q.c = c; q.d = d; q.c2 = c * c; q.d2 = d * d;
    q.S0 = q.wN * (d - c) * horner<N>(q.Q, q.oN);
    q.S1 = q.wF * (d - c) * horner<N>(q.Q, q.oF);
    q.mfirst = (int)floor(sqrt64(q.base2 + (q.oN + q.c2)) - r0) + 1;
    q.mlast = (int)ceil(sqrt64(q.base2 + (q.oF + q.d2)) - r0);
}

// The area function at radius r strictly between the nearest and the farthest
// corner (its value at the corners is S0 and S1: it is the area nearer than r
// plus S0)
template <int N, int S, int NW>
__device__ __forceinline__ double arc_edge(const ArcQuad<N>& q, double r, const double* tab)
{
    const double K = fma(r, r, -q.base2);
    bool onD, onC;
    double oa, ob, ea, eb;   // om at the end points, and the squares of what the roots give
    if constexpr (N == 0) {
        onD = K > q.oN + q.d2;
        onC = K < q.oF + q.c2;
        ea = K - (onD ? q.d2 : q.oN);
        eb = K - (onC ? q.c2 : q.oF);
        oa = ob = 0.0;
    } else {
        const double od = K - q.d2, oc = K - q.c2;
        onD = od > q.oN;
        onC = oc < q.oF;
        oa = fmax(od, q.oN);
        ob = fmin(oc, q.oF);
        ea = onD ? S * od : K - q.oN;
        eb = onC ? S * oc : K - q.oF;
    }
    const double ra = sqrt64<NW>(ea), rb = sqrt64<NW>(eb);
    const double wa = onD ? ra : q.wN, ya = onD ? q.d : ra;
    const double wb = onC ? rb : q.wF, yb = onC ? q.c : rb;
    // Lambda: twice atan or atanh of num / den, the half angle, whose denominator
    // stays positive.  The branches are the wave's: on 256^3 voxels x 512 rectangles
    // nearly all arguments are below 1/8 (median 0.03), on 128^3 x 256 cylinders
    // below 0.42 (median 0.14)
    double num, den;
    if (S > 0) {
        num = fma(wb, ya, -wa * yb);
        den = K + fma(wa, wb, ya * yb);
    } else {
        num = (wb + yb) - (wa + ya);
        den = (wb + yb) + (wa + ya);
    }
    const double x = arc_quotient<NW>(num, den);
    double lam;   // Lambda / 2
    if (__any(!(fabs(x) <= 0.42)))
        lam = S > 0 ? arc_atan<NW>(num, den, tab) : -0.5 * arc_log<NW>(wa + ya, wb + yb, tab);
    else if (__any(fabs(x) > 0.125))
        lam = arc_series(x, ArcSeries<S, NW>::hi);
    else
        lam = arc_series(x, ArcSeries<S, NW>::lo);
    if constexpr (N == 0) {
        const double Ba = wa * fma(ya, q.P[0], -q.d * q.Q[0]);
        return fma(q.Q[0] * K, lam, fma(wb, fma(yb, q.P[0], -q.c * q.Q[0]), -Ba));   // Q = 2 P
    } else {
        // (2j + 2) D[j] = p_j + (2j + 1) K D[j + 1]: the sum of p_j J_j is
        // D[0] (w y + K Lambda) - w y^3 (D[1] + D[2] om + ...)
        double D[N + 1];
        D[N] = q.P[N];
#pragma unroll
        for (int j = N; j > 0; --j) D[j - 1] = fma(K * ((2.0 * j - 1.0) / (2.0 * j)), D[j], q.P[j - 1]);
        const double Ba = wa * fma(ya, fma(-ya * ya, horner<N - 1>(D + 1, oa), D[0]), -q.d * horner<N>(q.Q, oa));
        const double Bb = wb * fma(yb, fma(-yb * yb, horner<N - 1>(D + 1, ob), D[0]), -q.c * horner<N>(q.Q, ob));
        return fma(D[0] * (K + K), lam, Bb - Ba);
    }
}

// ---------------------------------------------------------------------------
// rectangles with FP64 input and output
// ---------------------------------------------------------------------------
// The area function above is of the size of K = r^2 - |x3|^2, and away from the
// element's axis K is the square of thousands of bins where a bin's area is a few:
// its differences keep 2^-53 K.  Here everything is counted from the quadrant's
// nearest corner (a, c) at distance D: t = r - D, q = r^2 - D^2 = t (t + 2 D), the
// end points' offsets from the corner as quotients of q and of its differences
// with E = d^2 - c^2 and F = b^2 - a^2, and the area nearer than r as
//   pa (d - c) + (pb - pa)(va + vb) / 2 + K (atan x - x / (1 + x^2)):
// the strip beside the arc, the trapezoid under its chord, and the segment between
// chord and arc, x = tan(Lambda / 2) = ((pb - pa) + (va - vb)) / (wa + wb + ya + yb).
// t > 0 from the first edge on, so no edge can fall on the corner or inside it.
//
// Two quotients more than arc_edge<0>: A^T of 32^3 x 64 rectangles in FP64 66.8 us
// against 58.4 (427 by the walk of pieces between corners that both replace).
// Errors of the worst bin against 40 digits, of the pair's largest bin, medians of this
// form, of arc_edge<0> and of the walk: 0.5 x 3 mm at 50 MHz, 20 to 60 mm away on
// the axis 4e-15, 2e-14, 1e-13; 30 degrees off it 1.6e-14, 3e-13, 3e-14; 85 degrees 1.8e-14,
// 2.6e-12, 1.6e-14; the same at U = 11, 60 degrees 1e-13, 1.1e-11, 1.7e-14 (the area nearer
// than the edge is 1000 bins there); 0.2 mm at U = 11, 60 degrees 5e-14, 3.5e-11, 7e-14;
// 0.1 mm at U = 61, 60 degrees 2.6e-13, 2.9e-10, 3.5e-13.
struct PlaneQuad {
    double pos, D2, a, c, a2, c2, E, F, G, H;   // D - r0, 2 D, the near corner and its squares, d^2 - c^2,
                                                // b^2 - a^2, b - a, d - c
    double w;                                   // weight of the quadrant
    double S0, S1;
    int mfirst, mlast;
};

// (atan x - x / (1 + x^2)) / x^3 by interpolation at Chebyshev nodes of x^2, on x <= 1/8
// and on x <= 0.42; relative error 4e-17 and 6e-17
static constexpr double kSegmentLo[7] = {
    0.6666666666666666, -0.7999999999998448, 0.8571428569838612, -0.8888888277343502,
    0.9090796942525528, -0.922018712775229, 0.8835386887333297};
static constexpr double kSegmentHi[12] = {
    0.6666666666666666, -0.7999999999999372, 0.857142857125834, -0.8888888870770899,
    0.9090908091655334, -0.9230736588703263, 0.933265379587792, -0.9402379872042317,
    0.9386152534074689, -0.8972906398300687, 0.7271671936388654, -0.3539903641493709};

template <int M>
__device__ __forceinline__ double segment_series(double u, const double (&c)[M])
{
    double p = c[M - 1];
#pragma unroll
    for (int j = M - 2; j >= 0; --j) p = fma(p, u, c[j]);
    return p;
}

__device__ __forceinline__ void plane_setup(PlaneQuad& q, double a, double b, double c, double d, double z2, double w,
                                            double r0)
{
    q.a = a; q.c = c;
    q.a2 = a * a; q.c2 = c * c;
    q.G = b - a; q.H = d - c;
    q.F = q.G * (b + a); q.E = q.H * (d + c);
    const double D = sqrt64(z2 + (q.a2 + q.c2));
    q.D2 = D + D;
    q.pos = D - r0;
    q.w = w;
    q.S0 = 0.0;
    q.S1 = w * q.G * q.H;
    q.mfirst = (int)floor(q.pos) + 1;
    q.mlast = (int)ceil(sqrt64(z2 + fma(b, b, d * d)) - r0);
}

// sqrt(b^2 + n) - b for n >= 0, b >= 0 to full relative precision: n / (b + sqrt(b^2 + n))
// from the seeds of root and reciprocal (2^-23), then two steps on x^2 + 2 b x = n
// with the root's seed for the slope
__device__ __forceinline__ double plane_offset(double n, double b)
{
    const double s2 = fmax(fma(b, b, n), Tiny<2>::value);
    const double y = __builtin_amdgcn_rsq(s2), h = -0.5 * y, b2 = b + b;
    double x = n * __builtin_amdgcn_rcp(fma(s2, y, b));
    x = fma(fma(x, x + b2, -n), h, x);
    return fma(fma(x, x + b2, -n), h, x);
}

// the area nearer than the outer edge of bin m, mfirst <= m < mlast
__device__ __forceinline__ double plane_edge(const PlaneQuad& Q, int m, const double* tab)
{
    const double t = m - Q.pos, q = t * (t + Q.D2);
    const double qE = q - Q.E, qF = q - Q.F;
    const bool onD = qE > 0.0, onC = qF < 0.0;
    // each end point's offset n / (base + sqrt(base^2 + n)) along the line it is on
    const double na = onD ? qE : q, nb = onC ? q : qF;
    const double ba = onD ? Q.a : Q.c, bb = onC ? Q.a : Q.c;
    const double fa = plane_offset(na, ba), fb = plane_offset(nb, bb);
    const double pa = onD ? fa : 0.0, va = onD ? Q.H : fa;
    const double pb = onC ? fb : Q.G, vb = onC ? 0.0 : fb;
    const double dp = pb - pa, sv = va + vb;
    const double num = dp + (va - vb), den = fma(2.0, Q.a + Q.c, (pa + pb) + sv);
    const double x = arc_quotient<2>(num, den), u = x * x;
    const double K = q + (Q.a2 + Q.c2);
    double seg;   // K (atan x - x / (1 + x^2))
    if (__any(!(fabs(x) <= 0.42)))
        seg = K * (arc_atan<2>(num, den, tab) - x * rcp64_full(1.0 + u));
    else if (__any(fabs(x) > 0.125))
        seg = K * (x * u) * segment_series(u, kSegmentHi);
    else
        seg = K * (x * u) * segment_series(u, kSegmentLo);
    return Q.w * fma(pa, Q.H, fma(0.5 * dp, sv, seg));
}

// ---------------------------------------------------------------------------
// the walk over a quadrant's bins
// ---------------------------------------------------------------------------

// hand the bins wlo .. whi of the quadrant to sink(m, area).  Every edge is
// evaluated on its own, from its number, so a walk that the window clips starts
// there, with the same areas bit for bit; the first and the last edge of the
// quadrant lie outside its corners and are set (S0, S1), which also makes every
// lane's loop one edge shorter
template <class Quad, class Edge, class Sink>
__device__ __forceinline__ void sweep_edges(const Quad& q, int wlo, int whi, Edge edge, Sink& sink)
{
    const int mb = max(q.mfirst, wlo), me = min(q.mlast, whi);
    if (mb > me) return;
    const bool tail = me == q.mlast;
    const int mend = tail ? me - 1 : me;   // the last edge evaluated
    double s0 = q.S0;
    if (mb > q.mfirst) s0 = edge(mb - 1);
    for (int m = mb; m <= mend; ++m) {
        const auto w = sink.fetch(m);   // what the bin's sum needs from memory, under way while the edge is evaluated
        const double s1 = edge(m);
        sink.add(m, s1 - s0, w);
        s0 = s1;
    }
    if (tail) sink(me, q.S1 - s0);
}

template <int N, int S, int NW, class Sink>
__device__ __forceinline__ void arc_sweep(const ArcQuad<N>& q, double r0, int wlo, int whi, const double* tab,
                                          Sink& sink)
{
    sweep_edges(q, wlo, whi, [&](int m) { return arc_edge<N, S, NW>(q, r0 + m, tab); }, sink);
}

template <class Sink>
__device__ __forceinline__ void plane_sweep(const PlaneQuad& q, int wlo, int whi, const double* tab, Sink& sink)
{
    sweep_edges(q, wlo, whi, [&](int m) { return plane_edge(q, m, tab); }, sink);
}

// ---------------------------------------------------------------------------
// cylinder quadrant by its arc integrals I_l (FP64): the trapezoidal and the
// tabulated I_l, and the exact one where arc_sweep does not serve
// ---------------------------------------------------------------------------

struct CyPair {
    double R, dm, mu, imu;       // radius, |R - rho|, 4 R rho, 1/mu (0 when rho = 0)
    const double2* lut;          // E~, F~ tables (lookup-table I_l only)
};

// how the cylinder's I_l is evaluated
enum : int {
    kIlExact = 0,       // exact (as weighted areas where they serve, in the pair sweeps)
    kIlTrapezoid = 1,   // chord of the level curve, Eq. trapezoid_Il
    kIlTable = 2,       // lookup tables of E~ and F~ (Sec. 4.2, LUT paragraph)
    kIlCarlson = 3,     // exact, by Carlson's integral for every pair, Eq. cyl_Il
};

struct CyQuad {
    double a, b, c, d;
    double sa, ca, sb, cb;          // sin, cos of a/2 and b/2
    double Qac, Qad, Qbc, Qbd;       // squared corner distances psi(a or b) + (c or d)^2
    double psia, psib;               // psi(a), psi(b) = (R - rho)^2 + mu sin^2 of the half angle
    double sa2, cb2;                // sin^2(a/2), cos^2(b/2)
    int mfirst, mlast;
};

struct CyEdge {
    double sa, ca, da;   // alpha/2: sin, cos, Delta = sqrt(1 - nu sin^2)
    double sb, cb, db;   // beta/2
    double I;
};

// sin and cos of x in [0, pi/2] (a half angle of the folded interval [0, pi]):
// Taylor series through x^23 and x^22, whose first omitted terms are below
// 2e-18 on that range, so no argument reduction is needed
__device__ __forceinline__ void sincos_quarter(double x, double& s, double& c)
{
    const double y = x * x;
    double ps = -1.0 / 25852016738884976640000.0;              // -1/23!
    ps = fma(y, ps, 1.0 / 51090942171709440000.0);            // 1/21!
    ps = fma(y, ps, -1.0 / 121645100408832000.0);             // -1/19!
    ps = fma(y, ps, 1.0 / 355687428096000.0);                 // 1/17!
    ps = fma(y, ps, -1.0 / 1307674368000.0);                  // -1/15!
    ps = fma(y, ps, 1.0 / 6227020800.0);                      // 1/13!
    ps = fma(y, ps, -1.0 / 39916800.0);                       // -1/11!
    ps = fma(y, ps, 1.0 / 362880.0);                          // 1/9!
    ps = fma(y, ps, -1.0 / 5040.0);                           // -1/7!
    ps = fma(y, ps, 1.0 / 120.0);                             // 1/5!
    ps = fma(y, ps, -1.0 / 6.0);                              // -1/3!
    s = fma(x * y, ps, x);
    double pc = 1.0 / 1124000727777607680000.0;               // 1/22!
    pc = fma(y, pc, -1.0 / 2432902008176640000.0);            // -1/20!
    pc = fma(y, pc, 1.0 / 6402373705728000.0);                // 1/18!
    pc = fma(y, pc, -1.0 / 20922789888000.0);                 // -1/16!
    pc = fma(y, pc, 1.0 / 87178291200.0);                     // 1/14!
    pc = fma(y, pc, -1.0 / 479001600.0);                      // -1/12!
    pc = fma(y, pc, 1.0 / 3628800.0);                         // 1/10!
    pc = fma(y, pc, -1.0 / 40320.0);                          // -1/8!
    pc = fma(y, pc, 1.0 / 720.0);                             // 1/6!
    pc = fma(y, pc, -1.0 / 24.0);                             // -1/4!
    pc = fma(y, pc, 0.5);
    c = fma(-y, pc, 1.0);
}

__device__ __forceinline__ void cy_setup(CyQuad& q, const CyPair& P, double a, double b, double c,
                                         double d, double r0)
{
    q.a = a; q.b = b; q.c = c; q.d = d;
    double sa, ca, sb, cb;
    sincos_quarter(0.5 * a, sa, ca);
    sincos_quarter(0.5 * b, sb, cb);
    q.sa = sa; q.ca = ca; q.sb = sb; q.cb = cb;
    const double psia = fma(P.mu * sa, sa, P.dm * P.dm);
    const double psib = fma(P.mu * sb, sb, P.dm * P.dm);
    q.psia = psia;
    q.psib = psib;
    q.Qac = psia + c * c;
    q.Qad = psia + d * d;
    q.Qbc = psib + c * c;
    q.Qbd = psib + d * d;
    q.sa2 = sa * sa;
    q.cb2 = cb * cb;
    q.mfirst = (int)floor(sqrt64(q.Qac) - r0) + 1;   // nearest and farthest corners
    q.mlast = (int)ceil(sqrt64(q.Qbd) - r0);
}

// one end point of the level curve on the line v (Eq. alphabeta), half-angle form;
// isK = 1/sqrt(r^2 - (R - rho)^2); Qav, Qbv = psi(a or b) + v^2.  r^2 - Q is
// one fma: its error is that of the rounded Q, as for (r - sqrt Q)(r + sqrt Q)
template <int NW>
__device__ __forceinline__ void cy_endpoint(const CyQuad& q, const CyPair& P, double r, double v,
                                            double Qav, double Qbv, double isK, double& s, double& c,
                                            double& dl)
{
    double qa = fma(r, r, -Qav);                // r^2 - v^2 - psi(a)
    if (!(qa > 0.0)) {
        s = q.sa; c = q.ca;
        dl = sqrt64<NW>(fma(r, r, -q.psia)) * isK;
        return;
    }
    double qb = fma(r, r, -Qbv);                // r^2 - v^2 - psi(b)
    if (!(qb < 0.0)) {
        s = q.sb; c = q.cb;
        dl = sqrt64<NW>(fma(r, r, -q.psib)) * isK;
        return;
    }
    // sin^2 = (qa + mu sa^2) / mu and cos^2 = (mu cb^2 - qb) / mu, both > 0 here
    s = sqrt64_pos<NW>(fma(qa, P.imu, q.sa2));
    c = sqrt64_pos<NW>(fma(-qb, P.imu, q.cb2));
    dl = v * isK;
}

// E(sigma, nu) from sin, cos and Delta of sigma: E = s R_F(c^2, D^2, 1) -
// nu s^3 R_D(c^2, D^2, 1) / 3 (DLMF 19.25.9), with Carlson's duplication and
// the series of DLMF 19.36.1-2 through degree 7.  Their truncation error is
// ~eps^8 / 4 for eps = max |1 - x_i / A|, so the duplication stops once
// eps < 1/35 (relative error ~1e-13; 4e-15 measured over amplitudes to 1.55
// rad and nu sin^2 up to 0.99999) in the FP64 kernels and once eps < 1/12
// (truncation 2e-11 measured, 5e-10 with the FP32 series terms below) in the
// FP32-I/O ones (NW = 1), whose outputs round at 6e-8: that saves most lanes a
// duplication step, and on 128^3 voxels x 256 cylinders moves the signals'
// error against FP64 from 5.7e-8 to 6.9e-8 (relative L2).
// TABLE: stop at eps < 1e-4 instead (truncation far below rounding) and also
// return F = s R_F(c^2, D^2, 1).
// The duplication runs on 4^n times the n-th iterates: a step then adds
// lambda to each (no scaling), the stopping test compares 4^n A_n with the
// fixed initial deviation, and the factors 2^n that the scaling leaves on
// R_F and on the R_D series are applied once at the end.  With c^2, D^2 <= 1
// = z, z stays the largest argument, so A_D = (x + y + 3z)/5 >= A_F = (x + y
// + z)/3 and the test needs A_F only.  x and y start at c^2 + tiny and D^2 +
// tiny (tiny = 1e-300, or 1e-30 for the FP32 seeds of NW = 1, which changes
// R_F and R_D by ~1e-15 relative at most), so every square root in the loop
// has a positive argument.
template <int NW, bool TABLE = false>
__device__ __forceinline__ double ellip_e_scd(double s, double c, double dl, double nu, double* f_out = nullptr)
{
    double x = fma(c, c, Tiny<NW>::value), y = fma(dl, dl, Tiny<NW>::value), z = 1.0;
    double sx = fabs(c), sy = dl, sz = 1.0;
    double AF = (x + y + z) * (1.0 / 3.0);
    double AD = (x + y + 3.0 * z) * 0.2;
    // largest |A - x_i| over both means: z is the largest argument and A_D >= A_F
    const double dev = fmax(z - AF, AD - fmin(x, y));
    const double thr = (TABLE ? 1.0e4 : (NW == 1 ? 12.0 : 35.0)) * dev;
    const int itmax = TABLE ? 40 : 12;
    double p2 = 1.0, sumD = 0.0;
    if (thr >= AF) {
        // the first step, with z = sqrt(z) = 1
        const double lam = fma(sx, sy, sx + sy);
        z += lam;
        sumD = rcp64<NW>(z);
        x += lam;
        y += lam;
        AF += lam;
        p2 = 2.0;
        sx = sqrt64_pos<NW>(x);
        sy = sqrt64_pos<NW>(y);
        sz = sqrt64_pos<NW>(z);
#pragma unroll 1
        for (int it = 1; it < itmax && thr >= AF; ++it) {
            double lam = fma(sx, sy, fma(sx, sz, sy * sz));
            sumD = fma(p2, rcp64<NW>(sz * (z + lam)), sumD);
            x += lam;
            y += lam;
            z += lam;
            AF += lam;
            p2 *= 2.0;
            sx = sqrt64_pos<NW>(x);
            sy = sqrt64_pos<NW>(y);
            sz = sqrt64_pos<NW>(z);
        }
    }
    AD = (x + y + 3.0 * z) * 0.2;
    double rAF = rsq64<NW>(AF), iAF = rAF * rAF;
    double X = (AF - x) * iAF, Y = (AF - y) * iAF, Z = -X - Y;
    if constexpr (NW == 1) {
        // FP32-I/O kernels: the series' corrections to 1 are O(eps^2) <= ~7e-3
        // (eps < 1/12 at the stop), so FP32 (twice the FP64 rate on gfx950)
        // leaves ~5e-10 relative error on E; the deviations X, Y themselves
        // are formed in FP64
        const float xf = (float)X, yf = (float)Y, zf = -xf - yf;
        const float e2 = fmaf(xf, yf, -zf * zf), e3 = xf * yf * zf;
        const float df = fmaf(e2, fmaf(e2, fmaf(e2, -5.0f / 208.0f, 1.0f / 24.0f), -0.1f),
                              e3 * fmaf(e2, fmaf(e2, 1.0f / 16.0f, -3.0f / 44.0f), fmaf(e3, 3.0f / 104.0f, 1.0f / 14.0f)));
        const double rf = (1.0 + (double)df) * rAF * p2;
        const double rAD = rsq64<NW>(AD), iAD = rAD * rAD;
        const float xd = (float)((AD - x) * iAD), yd = (float)((AD - y) * iAD);
        const float zd = -(xd + yd) * (1.0f / 3.0f);
        const float xy = xd * yd, z2 = zd * zd;
        const float d2 = fmaf(-6.0f, z2, xy), d3 = fmaf(3.0f, xy, -8.0f * z2) * zd, d4 = 3.0f * (xy - z2) * z2,
                    d5 = xy * z2 * zd;
        float t2 = fmaf(d3, 45.0f / 272.0f, fmaf(d2, -1.0f / 16.0f, 9.0f / 88.0f));
        t2 = fmaf(d2, t2, fmaf(d3, -9.0f / 52.0f, fmaf(d4, 3.0f / 20.0f, fmaf(d5, -9.0f / 68.0f, -3.0f / 14.0f))));
        const float t3 = fmaf(d3, 3.0f / 40.0f, fmaf(d4, -9.0f / 68.0f, 1.0f / 6.0f));
        const float dd = fmaf(d2, t2, fmaf(d3, t3, fmaf(d4, -3.0f / 22.0f, d5 * (3.0f / 26.0f))));
        const double rd = fma(p2 * (1.0 + (double)dd) * iAD, rAD, 3.0 * sumD);
        if (TABLE) *f_out = s * rf;
        return s * fma(-(nu * (1.0 / 3.0)) * (s * s), rd, rf);
    }
    double E2 = fma(X, Y, -Z * Z), E3 = X * Y * Z;
    // 1 - E2/10 + E3/14 + E2^2/24 - 3 E2 E3/44 - 5 E2^3/208 + 3 E3^2/104 + E2^2 E3/16
    double sf = fma(E2, fma_vvv(E2, fma_vsv(E2, -5.0 / 208.0, 1.0 / 24.0), -0.1), 1.0);
    sf = fma(E3, fma_vvv(E2, fma_vsv(E2, 1.0 / 16.0, -3.0 / 44.0), fma_vsv(E3, 3.0 / 104.0, 1.0 / 14.0)), sf);
    double rf = sf * rAF * p2;
    double rAD = rsq64<NW>(AD), iAD = rAD * rAD;
    X = (AD - x) * iAD;
    Y = (AD - y) * iAD;
    Z = -(X + Y) * (1.0 / 3.0);
    double XY = X * Y, Z2 = Z * Z;
    double D2 = XY - 6.0 * Z2, D3 = (3.0 * XY - 8.0 * Z2) * Z, D4 = 3.0 * (XY - Z2) * Z2, D5 = XY * Z2 * Z;
    // 1 - 3 D2/14 + D3/6 + 9 D2^2/88 - 3 D4/22 - 9 D2 D3/52 + 3 D5/26 - D2^3/16 + 3 D3^2/40
    //   + 3 D2 D4/20 + 45 D2^2 D3/272 - 9 (D3 D4 + D2 D5)/68, grouped by powers of D2 and D3
    double t2 = fma(D3, 45.0 / 272.0, fma_vsv(D2, -1.0 / 16.0, 9.0 / 88.0));
    t2 = fma(D2, t2, fma(D3, -9.0 / 52.0, fma(D4, 3.0 / 20.0, fma_vsv(D5, -9.0 / 68.0, -3.0 / 14.0))));
    double t3 = fma(D3, 3.0 / 40.0, fma_vsv(D4, -9.0 / 68.0, 1.0 / 6.0));
    double ser = fma(D2, t2, fma(D3, t3, fma(D4, -3.0 / 22.0, fma(D5, 3.0 / 26.0, 1.0))));
    double rd = fma(p2 * ser * iAD, rAD, 3.0 * sumD);
    if (TABLE) *f_out = s * rf;
    return s * fma(-(nu * (1.0 / 3.0)) * (s * s), rd, rf);
}

// ---------------------------------------------------------------------------
// lookup tables of E~(s, nu) = E(arcsin s, nu) and F~(s, nu) = F(arcsin s, nu)
// ---------------------------------------------------------------------------
// Both axes use the power-law grid of Eq. LUT_sampling, x_n = top (1 - (1 -
// n/(N-1))^4), n = 0..N-1, top = 1 - 1e-16, which crowds the nodes towards the
// logarithmic singularity of F at (1, 1).  Node (s_i, nu_j) holds {E~, F~} at
// index j N + i, so the four corners of a cell are two 32-byte pairs.
constexpr double kLutTop = 1.0 - 1e-16;
constexpr double kLutInvTop = 1.0 / kLutTop;

// node x_n; n / (N - 1) as the product with the rounded reciprocal plus one
// correction step (the correctly rounded quotient)
__device__ __forceinline__ double lut_node(int n)
{
    constexpr double inv = 1.0 / (double)(kLutN - 1);
    const double dn = (double)n;
    double q = dn * inv;
    q = fma(fma(-q, (double)(kLutN - 1), dn), inv, q);
    const double t = 1.0 - q;
    return kLutTop * (1.0 - t * t * t * t);
}

// the grid cell [x_n, x_{n+1}] holding x, by the inverse of the grid map,
// t = 1 - (1 - x/top)^(1/4) (two square roots), and the weight of x in it,
// linear in the coordinate: (x - x_n) / (x_{n+1} - x_n)
template <int NW>
__device__ __forceinline__ void lut_cell(double x, int& n, double& w)
{
    const double y = fmin(fmax(x * kLutInvTop, 0.0), 1.0);
    const double p = (1.0 - sqrt64<NW>(sqrt64<NW>(1.0 - y))) * (double)(kLutN - 1);
    n = max(0, min((int)p, kLutN - 2));
    const double x0 = lut_node(n), x1 = lut_node(n + 1);
    const double d = x1 - x0;
    w = (fmin(x, kLutTop) - x0) * (NW >= 2 ? rcp64_full(d) : rcp64(d));
}

// bilinear E~ and F~ at (s, nu), nu's cell (j, wn) given
template <int NW>
__device__ __forceinline__ void lut_ef(const double2* __restrict__ T, double s, int j, double wn, double& E,
                                       double& F)
{
    int i;
    double ws;
    lut_cell<NW>(s, i, ws);
    const double2* r = T + (j * kLutN + i);
    const double2 a = r[0], b = r[1], c = r[kLutN], d = r[kLutN + 1];
    const double e0 = fma(ws, b.x - a.x, a.x), e1 = fma(ws, d.x - c.x, c.x);
    const double f0 = fma(ws, b.y - a.y, a.y), f1 = fma(ws, d.y - c.y, c.y);
    E = fma(wn, e1 - e0, e0);
    F = fma(wn, f1 - f0, f0);
}

// E(beta/2, nu) - E(alpha/2, nu) from the sines of the half angles by the
// tables: E~ directly for nu <= 1; for nu > 1 the reciprocal-modulus form
// (Eq. reciprocal_modulus) E(t, nu) = sqrt(nu) [E~(sqrt(nu) sin t, 1/nu) -
// (1 - 1/nu) F~(sqrt(nu) sin t, 1/nu)], whose first argument stays <= 1 by
// Lemma exact_integral.  Both end points share the nu cell.
template <int NW>
__device__ __forceinline__ double lut_de(const double2* __restrict__ T, double sa, double sb, double nu)
{
    const bool rec = nu > 1.0;
    const double inu = NW >= 2 ? rcp64_full(nu) : rcp64(nu);
    const double q = rec ? inu : nu;
    const double g = rec ? sqrt64<NW>(nu) : 1.0;
    const double cf = rec ? 1.0 - inu : 0.0;
    int j;
    double wn;
    lut_cell<NW>(q, j, wn);
    double Ea, Fa, Eb, Fb;
    lut_ef<NW>(T, g * sa, j, wn, Ea, Fa);
    lut_ef<NW>(T, g * sb, j, wn, Eb, Fb);
    return g * fma(-cf, Fb - Fa, Eb - Ea);
}

// asin(u) for 0 <= u <= 0.05: odd Taylor series through u^11 (the first
// omitted term is < 5e-18 relative)
__device__ __forceinline__ double asin_small(double u)
{
    double y = u * u;
    double p = 63.0 / 2816;
    p = fma(y, p, 35.0 / 1152);
    p = fma(y, p, 5.0 / 112);
    p = fma(y, p, 3.0 / 40);
    p = fma(y, p, 1.0 / 6);
    return fma(u * y, p, u);
}

// atan(t) for 0 <= t <= 1: four halvings of the angle, tan(x/2) = t / (1 +
// sqrt(1 + t^2)), take t below tan(pi/64) < 0.05, where the odd Taylor series
// through t^13 has its first omitted term below 3e-20 relative.  Its
// coefficients 1/3 .. 1/13 are taken over the common denominator 45045, so
// each is an integer that the instruction encodes as a literal.
__device__ __forceinline__ double atan_unit(double t)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) t *= rcp64_full(1.0 + sqrt64_pos(fma(t, t, 1.0)));
    const double y = t * t, y2 = y * y, y3 = y2 * y;
    const double p = 45045.0 - 15015.0 * y + 9009.0 * y2 - 6435.0 * y3 + 5005.0 * (y2 * y2) -
                     4095.0 * (y2 * y3) + 3465.0 * (y3 * y3);
    return (16.0 / 45045.0) * t * p;
}

// atan2(y, x) on the full circle from atan_unit of min/max(|x|, |y|), with
// the octant restored by reflections; 0 for x = y = 0
__device__ __forceinline__ double atan2_full(double y, double x)
{
    const double ax = fabs(x), ay = fabs(y);
    const double mn = fmin(ax, ay), mx = fmax(ax, ay);
    double a = mx > 0.0 ? atan_unit(mn * rcp64_full(mx)) : 0.0;
    if (ay > ax) a = 0.5 * M_PI - a;
    if (x < 0.0) a = M_PI - a;
    return copysign(a, y);
}

// Alg. 4 triple at the edge of radius r: half-angle state of alpha, beta and I
// (Eq. cyl_Il; the chord of the level curve, Eq. trapezoid_Il, or the tables)
template <int NW, int IL = kIlExact>
__device__ __forceinline__ void cy_edge(const CyQuad& q, const CyPair& P, double r, CyEdge& E)
{
    // K = r^2 - (R - rho)^2 = 2 R rho + b(r).  K <= 0: the shell misses the
    // surface, r^2 - v^2 - psi(a) <= 0 on both lines, so both end points clamp
    // at a (no branch of their own) and I = 0; their Delta (and 1/sqrt K) are
    // then not finite and not used
    double K = (r - P.dm) * (r + P.dm);
    double isK = rsq64<NW>(K);
    cy_endpoint<NW>(q, P, r, q.d, q.Qad, q.Qbd, isK, E.sa, E.ca, E.da);
    cy_endpoint<NW>(q, P, r, q.c, q.Qac, q.Qbc, isK, E.sb, E.cb, E.db);
    double cr = fma(E.sb, E.ca, -E.cb * E.sa);   // sin(beta/2 - alpha/2)
    if (!(cr > 0.0 && K > 0.0)) { E.I = 0.0; return; }
    if (IL == kIlTrapezoid) {
        // (beta - alpha)/2 (Psi(alpha) + Psi(beta)) with Psi = sqrt(K) Delta
        const double cs = fma(E.cb, E.ca, E.sb * E.sa);   // cos(beta/2 - alpha/2)
        const double sg = (cr <= 0.05 && cs > 0.0) ? asin_small(cr) : atan2_full(cr, cs);
        E.I = K * isK * sg * (E.da + E.db);
        return;
    }
    double nu = P.mu * isK * isK;
    if (IL == kIlTable) {
        E.I = 2.0 * K * isK * lut_de<NW>(P.lut, E.sa, E.sb, nu);
        return;
    }
    const double sbda = E.sb * E.da, sbsa = E.sb * E.sa, dd = E.db * E.da, nss = nu * sbsa;
    double den = fma(E.cb, E.cb, sbda * sbda);   // 1 - nu sin^2 sin^2
    double idn = rcp64<NW>(den);
    double ss = fma(sbda, E.ca, -E.sa * (E.cb * E.db)) * idn;
    double cs = fma(E.cb, E.ca, sbsa * dd) * idn;
    double ds = fma(nss, E.cb * E.ca, dd) * idn;
    double es = ellip_e_scd<NW>(ss, cs, ds, nu);
    E.I = 2.0 * K * isK * fma(-nss, ss, es);
}

// The steps of both end-point angles between consecutive edges (negative
// steps count as zero).  The half angles lie in [0, pi/2], so the cosine of a
// half step is >= 0, and a step whose half-step sine cr is <= 0.05 is 2 asin(cr)
// by the short series, with no division; unless every active lane of the wave
// has such steps, 2 atan2(cr, cos).
__device__ __forceinline__ void angle_steps(const CyEdge& E0, const CyEdge& E1, double& da, double& db)
{
    const double cra = fma(E1.sa, E0.ca, -E1.ca * E0.sa), crb = fma(E1.sb, E0.cb, -E1.cb * E0.sb);
    const double ua = fmax(cra, 0.0), ub = fmax(crb, 0.0);
    if (__all(fmax(ua, ub) <= 0.05)) {
        da = 2.0 * asin_small(ua);
        db = 2.0 * asin_small(ub);
        return;
    }
    const double dta = fma(E1.ca, E0.ca, E1.sa * E0.sa), dtb = fma(E1.cb, E0.cb, E1.sb * E0.sb);
    da = cra > 0.0 ? 2.0 * atan2_full(cra, dta) : 0.0;
    db = crb > 0.0 ? 2.0 * atan2_full(crb, dtb) : 0.0;
}

template <int NW, int IL, class Sink>
__device__ __forceinline__ void cy_sweep(const CyQuad& q, const CyPair& P, double r0, int wlo, int whi,
                                         double wgt, Sink& sink)
{
    const int mb = max(q.mfirst, wlo), me = min(q.mlast, whi);
    if (mb > me) return;
    const double wR = wgt * P.R;
    // Eq. area_D_l_xi, times J0 = R, between the edges Ea (inner) and Eb (outer)
    auto shell = [&](int m, const CyEdge& Ea, const CyEdge& Eb) {
        double dal, dbe;
        angle_steps(Ea, Eb, dal, dbe);
        sink(m, wR * fma(dal, q.d, fma(-q.c, dbe, Eb.I - Ea.I)));
    };
    // The inner edge of the first bin, r0 + mfirst - 1, does not pass the
    // nearest corner and the outer edge of the last one, r0 + mlast, is past
    // the farthest: there both end points sit at u = a (resp. u = b) and I = 0,
    // so these two edges are set rather than evaluated (a walk the window
    // clips evaluates its end edges).  Every lane's loop is one edge shorter.
    auto corner_edge = [](double s, double c, CyEdge& E) {
        E.sa = s; E.ca = c; E.da = 1.0;
        E.sb = s; E.cb = c; E.db = 1.0;
        E.I = 0.0;
    };
    CyEdge E0, E1;
    if (mb > q.mfirst)
        cy_edge<NW, IL>(q, P, r0 + (mb - 1), E0);
    else
        corner_edge(q.sa, q.ca, E0);
    const bool tail = me == q.mlast;
    const int mend = tail ? me - 1 : me;   // the last edge evaluated
    // two shells per trip, the edge records alternating roles (no copies)
    int m = mb;
    for (; m < mend; m += 2) {
        cy_edge<NW, IL>(q, P, r0 + m, E1);
        shell(m, E0, E1);
        cy_edge<NW, IL>(q, P, r0 + (m + 1), E0);
        shell(m + 1, E1, E0);
    }
    if (m == mend) {
        cy_edge<NW, IL>(q, P, r0 + m, E1);
        shell(m, E0, E1);
        if (tail) {
            corner_edge(q.sb, q.cb, E0);
            shell(me, E1, E0);
        }
    } else if (tail) {
        corner_edge(q.sb, q.cb, E1);
        shell(me, E0, E1);
    }
}

}  // namespace patop
