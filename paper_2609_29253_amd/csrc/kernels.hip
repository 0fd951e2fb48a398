// Device kernels of the patop library (gfx950).
//
// Forward A (Alg. 1):
//   1. k_fill            f <- 0  (FP64 fine-bin coefficients, [B][K][Mcount])
//   2. k_fwd_wave /      closed form: one work-group of one wave per (4 x 4 x 4
//      k_fwd_quad        voxel cube, chunk of transducers): for each transducer,
//                        every voxel of the cube adds p0 * |M_i^m| (Alg. 3, Eq.
//                        ui_area) into an LDS FP64 histogram covering the cube's
//                        bin window, which the wave then adds to f with FP64
//                        atomics, with no work-group barrier.  Quadrature: one
//                        256-thread work-group per (voxel brick, chunk), p0 * dA / r
//                        into the bin of each surface point (Alg. 2, Eq.
//                        def_f_point).  Sparse forward: k_support_count / _scan /
//                        _write list the voxels that are nonzero in some volume,
//                        and k_fwd_sparse_wave strides waves of 64 of them.  Time
//                        tiles: k_fwd_tile owns a (transducer, tile) of f.
//   3. k_fir             s_hat[l] = sum_j G[j] scale[m] f[m], m = U l - j (FP64): the
//                        convolution with h followed by the block average D_U
//                        (Eq. discrete_conv, Eq. def_downsampling) as one
//                        polyphase filter G[j] = 1/U sum_{l'=1..U} h[j + l'];
//                        scale[m] = U fs dr^2 / (c tau_{m-1/2}) (surface, Eq.
//                        ui_area) or U fs dr (points).
// Adjoint A^T (Alg. 5-7):
//   1. k_adjw            W[m] = scale[m] sum_l G[U l - m] y[l]: transpose of the
//                        block average and correlation with the reversed kernel.
//   2. k_adj_wave /      one work-group per (cube of one wave, or brick for the
//      k_adj_quad        quadrature, chunk of transducers): W of the bin window is
//                        staged in LDS, every voxel gathers sum_m |M_i^m| W[m]
//                        (FP32 or FP64 per transducer) and accumulates over
//                        transducers in FP64.
//   3. k_finish          cast of the FP64 sums (cleared by k_adjw) when transducer
//                        chunks were split over work-groups.
#include <hip/hip_runtime.h>

#include "area.h"
#include "kernels.h"
#include "pairs.h"
#include "plan.h"

namespace patop {

// ---------------------------------------------------------------------------
// utilities
// ---------------------------------------------------------------------------

__global__ void k_fill(double* __restrict__ p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

template <class Real>
__global__ void k_finish(const double* __restrict__ z, Real* __restrict__ out, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (Real)z[i];
}

__device__ __forceinline__ int floordiv(int a, int b)
{
    int q = a / b;
    return (q * b > a) ? q - 1 : q;
}

// the voxel owned by this thread and the box of the work-group's brick
struct Brick {
    int64_t idx;
    int ix, iy, iz;
    bool valid;
    double lo[3], hi[3];   // axis-aligned box of the brick's voxel centres (global)
};

// axis-aligned box of brick bid's voxel centres (global coordinates)
__device__ __forceinline__ void brick_box(const KParams& P, int bid, double lo[3], double hi[3])
{
    const int bxi = bid % P.nbx, byi = (bid / P.nbx) % P.nby, bzi = bid / (P.nbx * P.nby);
    const int x0 = bxi * kBrickX, y0 = byi * kBrickY, z0 = bzi * kBrickZ;
    const int x1 = (int)min((int64_t)(x0 + kBrickX), P.n[0]) - 1;
    const int y1 = (int)min((int64_t)(y0 + kBrickY), P.n[1]) - 1;
    const int z1 = (int)min((int64_t)(z0 + kBrickZ), P.n[2]) - 1;
    lo[0] = P.origin[0] + x0 * P.w; hi[0] = P.origin[0] + x1 * P.w;
    lo[1] = P.origin[1] + y0 * P.w; hi[1] = P.origin[1] + y1 * P.w;
    lo[2] = P.origin[2] + z0 * P.w; hi[2] = P.origin[2] + z1 * P.w;
}

// Column of a work-group's cube or brick in its row of nx.  Work-groups go to the 32 shader
// engines in turn, and an engine without a free slot holds up the others: where
// 32 divides nx, each engine would see the same columns of the volume in every
// row, and the costliest would set the pace (128^3 x 256 cylinders: 2.5 waves per
// SIMD resident of 4 possible, and 3.96 with each row starting at a column of its
// own: A 69.3 -> 64.1 ms, A^T 80.8 -> 68.2, with weights of a lower degree than now;
// 256^3 x 512 rectangles A 275 -> 263).
__device__ __forceinline__ unsigned spread_column(unsigned id, unsigned row, unsigned nx)
{
    return (id - row * nx + (((row + 1) * 0x9e3779b9u) >> 16)) % nx;
}

__device__ __forceinline__ void brick_setup(const KParams& P, int bid, Brick& Bk)
{
    const int bxi = bid % P.nbx, byi = (bid / P.nbx) % P.nby, bzi = bid / (P.nbx * P.nby);
    const int x0 = bxi * kBrickX, y0 = byi * kBrickY, z0 = bzi * kBrickZ;
    // each wave owns a 4 x 4 x 4 sub-cube of the brick: the most compact set of
    // 64 voxels, so that their sweeps over a transducer have similar lengths
    // and quadrant counts (less divergence than an 8 x 8 x 1 slab)
    const int v = threadIdx.x, w = v >> 6, l = v & 63;
    Bk.ix = x0 + (w & 1) * 4 + (l & 3);
    Bk.iy = y0 + (w >> 1) * 4 + ((l >> 2) & 3);
    Bk.iz = z0 + (l >> 4);
    Bk.valid = Bk.ix < P.n[0] && Bk.iy < P.n[1] && Bk.iz < P.n[2];
    Bk.idx = Bk.valid ? Bk.ix + P.n[0] * (Bk.iy + P.n[1] * (int64_t)Bk.iz) : 0;
    brick_box(P, bid, Bk.lo, Bk.hi);
}

// shells that any voxel of the box [lo, hi] can reach on transducer T
// (bounding sphere; Eq. rmin_rmax bounds each pair's range inside it), clipped
// to the kept shells [Jlo, Jhi]: empty (wlo > whi) if none
__device__ __forceinline__ void box_window(const KParams& P, const double lo3[3], const double hi3[3],
                                           const TrDev& T, int& wlo, int& whi)
{
    double dd = 0.0, dm = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double o = fmax(0.0, fmax(lo3[a] - T.cen[a], T.cen[a] - hi3[a]));
        dd += o * o;
        double f = fmax(fabs(lo3[a] - T.cen[a]), fabs(hi3[a] - T.cen[a]));
        dm += f * f;
    }
    double dlo = fmax(sqrt(dd) - T.rad, 0.0), dhi = sqrt(dm) + T.rad;
    int64_t lo = (int64_t)floor(dlo - P.r0);
    int64_t hi = (int64_t)ceil(dhi - P.r0) + 1;
    lo = max(lo, P.Jlo);
    hi = min(hi, P.Jhi);
    wlo = (int)lo;
    whi = (int)hi;
}

__device__ __forceinline__ void brick_window(const KParams& P, const Brick& Bk, const TrDev& T, int& wlo,
                                             int& whi)
{
    box_window(P, Bk.lo, Bk.hi, T, wlo, whi);
}

// shells that the voxel at frame coordinates x can reach on transducer T: from
// its distances to the nearest and the farthest point of the surface (Eq.
// rmin_rmax), in closed form.  Planar: the rectangle's nearest and farthest
// points in its plane.  Cylinder: |x - y|^2 = R^2 + rho^2 - 2 R rho cos(delta)
// + (z - x3)^2 for the point y at angle gap delta from the voxel's direction,
// whose smallest gap is 0 inside the angular range and |theta_i| - theta_max
// outside it, and largest min(pi, |theta_i| + theta_max); rho cos(delta) from
// the frame coordinates and cos / sin of theta_max, with no angle computed.
// floor / ceil keep a shell of margin for rounding: [lo, hi] holds every bin of
// every quadrant sweep of the pair.
template <int SHAPE>
__device__ __forceinline__ void pair_range(const TrDev& T, const double x[3], double r0, int& lo, int& hi)
{
    double dmin2, dmax2;
    if (SHAPE == 0) {
        const double du = fmax(0.0, fabs(x[0]) - T.p[0]), dv = fmax(0.0, fabs(x[1]) - T.p[1]);
        const double eu = fabs(x[0]) + T.p[0], ev = fabs(x[1]) + T.p[1];
        const double z2 = x[2] * x[2];
        dmin2 = fma(du, du, fma(dv, dv, z2));
        dmax2 = fma(eu, eu, fma(ev, ev, z2));
    } else {
        const double R = T.p[0], ax1 = fabs(x[1]);
        const double rho2 = fma(x[0], x[0], x[1] * x[1]);
        const double rho = sqrt64<1>(rho2);
        const bool inside = fma(x[0], T.sth, -ax1 * T.cth) >= 0.0;   // |theta_i| <= theta_max
        const double cmin = inside ? rho : fma(x[0], T.cth, ax1 * T.sth);
        const double cmax = x[0] < -T.cth * rho ? -rho : fma(x[0], T.cth, -ax1 * T.sth);
        const double vmin = fmax(0.0, fabs(x[2]) - T.p[2]), vmax = fabs(x[2]) + T.p[2];
        const double base = fma(R, R, rho2);
        dmin2 = fma(vmin, vmin, fma(-2.0 * R, cmin, base));
        dmax2 = fma(vmax, vmax, fma(-2.0 * R, cmax, base));
    }
    // FP32 roots (off by less than 2e-7), moved outward by twice that
    lo = (int)floor((double)(sqrt_t((float)dmin2) * (1.0f - 4e-7f)) - r0);
    hi = (int)ceil((double)(sqrt_t((float)dmax2) * (1.0f + 4e-7f)) - r0) + 1;
}

// minimum of v over the 64 lanes, all active, as a scalar: shifts by 1, 2, 4 and 8
// within rows of 16 lanes, then two broadcasts across rows, each fused with its
// minimum (a permute through LDS per step takes four times the instructions)
__device__ __forceinline__ int wave_min(int v)
{
    constexpr int none = 0x7fffffff;
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x111, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x112, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x114, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x118, 0xf, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x142, 0xa, 0xf, false));
    v = min(v, __builtin_amdgcn_update_dpp(none, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// [min lo, max hi] over the lanes of the wave that take part (others pass
// INT_MAX / INT_MIN), clipped to the kept shells [Jlo, Jhi]
__device__ __forceinline__ void wave_window(const KParams& P, int lo, int hi, int& wlo, int& whi)
{
    wlo = max(wave_min(lo), (int)P.Jlo);
    whi = min(~wave_min(~hi), (int)P.Jhi);
}

// ---------------------------------------------------------------------------
// forward, closed-form areas
// ---------------------------------------------------------------------------

// sparse forward: transducers per work item, and the strided grid in units of
// 256 threads (4 x 4096 one-wave work-groups: 64 waves per CU at 256 CUs)
constexpr int kSparseChunk = 16;
constexpr int kSparseGrid = 4096;

// Waves per SIMD the closed-form kernels are built for (one-wave work-groups in
// the dense and sparse forward and the adjoint, 256-thread ones in the time
// tiles).  The planar kernels hold 90-128 VGPRs without spills (five waves up to 96),
// except FP64 with eight volumes (140 in the adjoint: three).  Cylinders for one or
// two volumes: four, in 128 VGPRs with spills outside the loops over edges; with
// more volumes the spills grow and they keep three.
template <int SHAPE, class AT, int NB>
constexpr int closed_waves()
{
    return SHAPE == 1 ? (NB <= 2 ? 4 : 3) : (sizeof(AT) == 8 && NB == 8 ? 3 : 4);
}

// ---------------------------------------------------------------------------
// forward, closed-form areas, one wave per work-group
// ---------------------------------------------------------------------------

constexpr int kWave = 64;          // threads of a one-wave work-group: a 4 x 4 x 4 voxel cube

// orders a one-wave work-group's LDS operations before it against those after
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS window of a one-wave work-group, in bytes, shared by its volumes.  Planar:
// with the arc table 7568 bytes, so that twenty-one of them fit a CU (the kernels
// run at five waves per SIMD).  Cylinders keep their 4 KB table of interval ends
// there too and run sixteen per CU.
template <int SHAPE>
constexpr int wave_window_bytes()
{
    return SHAPE == 1 ? 4096 : 7040;
}

// Where a sweep's areas go.  fetch(m) reads what bin m's sum needs, before the area
// is known; add(m, area, fetched) finishes it.  give() and take() carry the sink to
// and from a function that is not inlined.

__device__ __forceinline__ void lds_add(double* p, double v)
{
    __builtin_amdgcn_ds_atomic_fadd_f64((LdsDouble*)p, v);
}
__device__ __forceinline__ void lds_add(LdsDouble* p, double v) { __builtin_amdgcn_ds_atomic_fadd_f64(p, v); }

// forward: p0 * area into the LDS histogram of each volume (`stride` bins apart)
template <int NB, class Ptr = double*>
struct Scatter {
    Ptr hist;
    int stride, first;
    double p0[NB];
    __device__ __forceinline__ int fetch(int) const { return 0; }
    __device__ __forceinline__ void add(int m, double area, int)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b) lds_add(&hist[b * stride + (m - first)], p0[b] * area);
    }
    __device__ __forceinline__ void operator()(int m, double area) { add(m, area, 0); }
    __device__ __forceinline__ Scatter<NB, LdsDouble*> give() const
    {
        Scatter<NB, LdsDouble*> s;
        s.hist = (LdsDouble*)hist;
        s.stride = stride;
        s.first = first;
#pragma unroll
        for (int b = 0; b < NB; ++b) s.p0[b] = p0[b];
        return s;
    }
    __device__ __forceinline__ void take(const Scatter<NB, LdsDouble*>&) {}
};

// adjoint: area times each volume's W, summed
template <int NB, class AT, class Real, class Ptr = const Real*>
struct Gather {
    using Lds = const __attribute__((address_space(3))) Real*;
    Ptr Ws;
    int stride, first;
    AT part[NB];
    struct Vals {
        Real w[NB];
    };
    __device__ __forceinline__ Vals fetch(int m) const
    {
        Vals v;
#pragma unroll
        for (int b = 0; b < NB; ++b) v.w[b] = Ws[b * stride + (m - first)];
        return v;
    }
    __device__ __forceinline__ void add(int, double area, const Vals& v)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b) part[b] = fma((AT)area, (AT)v.w[b], part[b]);
    }
    __device__ __forceinline__ void operator()(int m, double area) { add(m, area, fetch(m)); }
    __device__ __forceinline__ Gather<NB, AT, Real, Lds> give() const
    {
        Gather<NB, AT, Real, Lds> s;
        s.Ws = (Lds)Ws;
        s.stride = stride;
        s.first = first;
#pragma unroll
        for (int b = 0; b < NB; ++b) s.part[b] = part[b];
        return s;
    }
    __device__ __forceinline__ void take(const Gather<NB, AT, Real, Lds>& s)
    {
#pragma unroll
        for (int b = 0; b < NB; ++b) part[b] = s.part[b];
    }
};

struct Count {
    int n;
    __device__ __forceinline__ int fetch(int) const { return 0; }
    __device__ __forceinline__ void add(int, double, int) { ++n; }
    __device__ __forceinline__ void operator()(int, double) { ++n; }
    __device__ __forceinline__ Count give() const { return *this; }
    __device__ __forceinline__ void take(const Count& s) { n = s.n; }
};

// First voxel of a one-wave work-group's cube
__device__ __forceinline__ void wave_cube(const KParams& P, int& x0, int& y0, int& z0)
{
    const unsigned ncx = (P.n[0] + 3) / 4, ncy = (P.n[1] + 3) / 4, row = blockIdx.x / ncx;
    x0 = (int)spread_column(blockIdx.x, row, ncx) * 4;
    y0 = (int)(row % ncy) * 4;
    z0 = (int)(row / ncy) * 4;
}

// The wave's 64 voxels (one per lane; `valid` false for lanes without one)
// against transducers kperm[kbeg .. kend): per transducer the window is the
// union of the lanes' pair ranges, swept in passes of HW shells.  The wave owns
// its LDS window: it clears it, sweeps into it and adds it to f with no
// work-group barrier, only the ordering of its own LDS operations.
template <int SHAPE, class AT, int NB, class Real, int IL>
__device__ __forceinline__ void fwd_wave_voxels(const KParams& P, int ix, int iy, int iz, bool valid, int64_t idx,
                                                int kbeg, int kend, const Real* __restrict__ coef,
                                                double* __restrict__ f, double* hist, double* box, double* tab)
{
    constexpr int HE = wave_window_bytes<SHAPE>() / (int)sizeof(double);
    constexpr int HW = HE / NB;          // shells per pass
    const int l = threadIdx.x;
    double p0[NB];
    bool nz = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        p0[b] = valid ? (double)coef[b * P.N + idx] : 0.0;
        nz |= p0[b] != 0.0;
    }
    if (!__any(nz)) return;
    load_arc_table<kWave>(tab);   // after the cubes without a coefficient have left
    wave_lds_order();
    const int S = P.step;
    const int64_t Mhi = P.Mlo + P.Mcount - 1;
    for (int kk = kbeg; kk < kend; ++kk) {
        const int k = P.kperm[kk];
        int wlo, whi;
        typename PairOf<SHAPE, Real, IL, kWave>::type pair;
        pair.bind(box, P.lut, tab, P.tr + k, ix, iy, iz);
        {
            const TrDev T = P.tr[k];
            double x[3];
            frame_coords(T, ix, iy, iz, x);
            int lo = 0x7fffffff, hi = -0x7fffffff - 1;
            if (nz) pair_range<SHAPE>(T, x, P.r0, lo, hi);   // lanes whose volumes are all zero add nothing
            wave_window(P, lo, hi, wlo, whi);
            if (wlo > whi) continue;   // no shell kept: a cylinder's set-up costs more than all else here
            pair.setup(T, x, P.r0);
            pair.agree(valid);
        }
        for (int plo = wlo; plo <= whi; plo += HW) {
            const int phi = min(whi, plo + HW - 1);
            const int wn = phi - plo + 1;
            for (int i = l; i < wn; i += kWave)
#pragma unroll
                for (int b = 0; b < NB; ++b) hist[b * HW + i] = 0.0;
            wave_lds_order();
            if (nz) {
                Scatter<NB> sink;
                sink.hist = hist;
                sink.stride = HW;
                sink.first = plo;
#pragma unroll
                for (int b = 0; b < NB; ++b) sink.p0[b] = p0[b];
                pair.sweep(plo, phi, sink, P.r0);
            }
            wave_lds_order();
            for (int i = l; i < wn * S; i += kWave) {
                const int jj = S == 1 ? i : i / S;   // (no division on the fine grid)
                const int64_t m = (int64_t)(plo + jj - 1) * S + 1 + (i - jj * S);
                if (m < P.Mlo || m > Mhi) continue;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    double v = hist[b * HW + jj];
                    if (v != 0.0) unsafeAtomicAdd(&f[((int64_t)b * P.K + k) * P.Mcount + (m - P.Mlo)], v * S);
                }
            }
            wave_lds_order();
        }
    }
}

// Dense forward: one work-group of one wave per (4 x 4 x 4 voxel cube, chunk
// of transducers).
template <int SHAPE, class AT, int NB, class Real, int IL>
__global__ __launch_bounds__(kWave, (closed_waves<SHAPE, AT, NB>())) void k_fwd_wave(KParams P,
                                                                                     const Real* __restrict__ coef,
                                                                                     double* __restrict__ f)
{
    __shared__ double hist[wave_window_bytes<SHAPE>() / sizeof(double)];   // [NB][shells per pass]
    __shared__ double box[SHAPE == 1 ? kBoxSlots * kWave : 1];
    __shared__ double tab[kArcTab];
    int x0, y0, z0;
    wave_cube(P, x0, y0, z0);
    const int l = threadIdx.x;
    const int ix = x0 + (l & 3), iy = y0 + ((l >> 2) & 3), iz = z0 + (l >> 4);
    const bool valid = ix < P.n[0] && iy < P.n[1] && iz < P.n[2];
    const int64_t idx = valid ? ix + P.n[0] * (iy + P.n[1] * (int64_t)iz) : 0;
    const int kbeg = blockIdx.y * P.kchunk;
    fwd_wave_voxels<SHAPE, AT, NB, Real, IL>(P, ix, iy, iz, valid, idx, kbeg, min(P.nk, kbeg + P.kchunk), coef, f,
                                             hist, box, tab);
}

// Sparse forward: work items (64 consecutive entries of the support list, a
// chunk of P.kchunk transducers), strided over a fixed grid of one-wave
// work-groups, since their number is known on the device only.  The list holds
// the nonzero voxels brick by brick in Morton order and, inside a brick, 4 x 4
// x 4 cube by cube, so 64 consecutive entries lie in a few neighbouring cubes
// and their pair ranges overlap.
template <int SHAPE, class AT, int NB, class Real, int IL>
__global__ __launch_bounds__(kWave, (closed_waves<SHAPE, AT, NB>())) void k_fwd_sparse_wave(
    KParams P, const Real* __restrict__ coef, double* __restrict__ f)
{
    __shared__ double hist[wave_window_bytes<SHAPE>() / sizeof(double)];   // [NB][shells per pass]
    __shared__ double box[SHAPE == 1 ? kBoxSlots * kWave : 1];
    __shared__ double tab[kArcTab];
    const int64_t total = *P.sup_total;
    const int64_t groups = (total + kWave - 1) / kWave;
    // fewer transducers an item where the grid would be left with work-groups idle
    // (200^3 voxels, 1 in 400 nonzero, x 64 at U = 11: 1250 items of 16)
    const int kchunk = (int)min((int64_t)P.kchunk, max((int64_t)1, groups * P.nk / gridDim.x));
    const int64_t nchunks = (P.nk + kchunk - 1) / kchunk;
    const int64_t items = groups * nchunks;
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int64_t g = it / nchunks;
        const int64_t e = g * kWave + threadIdx.x;
        const bool valid = e < total;
        const int64_t idx = valid ? (int64_t)P.sup_list[e] : 0;
        const int ix = (int)(idx % P.n[0]), iy = (int)((idx / P.n[0]) % P.n[1]), iz = (int)(idx / (P.n[0] * P.n[1]));
        const int kbeg = (int)(it % nchunks) * kchunk;
        fwd_wave_voxels<SHAPE, AT, NB, Real, IL>(P, ix, iy, iz, valid, idx, kbeg, min(P.nk, kbeg + kchunk), coef,
                                                 f, hist, box, tab);
    }
}

// ---------------------------------------------------------------------------
// forward, closed-form areas, by (transducer, time tile): output-stationary
// ---------------------------------------------------------------------------

// One work-group per (transducer, tile of `tile` consecutive shells).  It owns
// the tile's fine bins of f for every volume of the launch, so f needs neither
// a fill nor atomics: the group scans the bricks, keeps those whose window
// meets the tile, and for each runs the pair setup and the sweep clipped to
// the tile into its LDS histogram, then stores the tile.  Work items come in
// the order of items[] (estimated cost, largest first) so that the in-order
// dispatch of work-groups balances the tail of the launch.
template <int SHAPE, class AT, int NB, class Real, int IL>
__global__ __launch_bounds__(kThreads, (closed_waves<SHAPE, AT, NB>())) void k_fwd_tile(
    KParams P, const int32_t* __restrict__ items, int tile, int ntiles, int nbricks, const Real* __restrict__ coef,
    double* __restrict__ f)
{
    extern __shared__ double hist[];   // [NB][tile]
    __shared__ double box[SHAPE == 1 ? kBoxSlots * kThreads : 1];
    __shared__ double tab[kArcTab];
    __shared__ int cand[kThreads];
    __shared__ int ncand;
    const int item = items[blockIdx.x];
    const int kk = item / ntiles, t = item - kk * ntiles;
    const int k = P.kperm[kk];
    const int tlo = (int)P.Jlo + t * tile;
    const int thi = min((int)P.Jhi, tlo + tile - 1);
    for (int i = threadIdx.x; i < NB * tile; i += kThreads) hist[i] = 0.0;
    load_arc_table<kThreads>(tab);   // ordered by the barriers before the first sweep
    for (int c0 = 0; c0 < nbricks; c0 += kThreads) {
        const int b = c0 + threadIdx.x;
        bool hit = false;
        if (b < nbricks) {
            double lo[3], hi[3];
            brick_box(P, b, lo, hi);
            int wlo, whi;
            box_window(P, lo, hi, P.tr[k], wlo, whi);
            hit = wlo <= thi && whi >= tlo;
        }
        __syncthreads();   // the previous list has been consumed (the histogram cleared)
        if (threadIdx.x == 0) ncand = 0;
        __syncthreads();
        if (hit) cand[atomicAdd(&ncand, 1)] = b;
        __syncthreads();
        const int nc = ncand;
        for (int i = 0; i < nc; ++i) {
            Brick Bk;
            brick_setup(P, cand[i], Bk);
            double p0[NB];
            bool nz = false;
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                p0[v] = Bk.valid ? (double)coef[v * P.N + Bk.idx] : 0.0;
                nz |= p0[v] != 0.0;
            }
            if (!__syncthreads_or(nz)) continue;
            typename PairOf<SHAPE, Real, IL>::type pair;
            pair.bind(box, P.lut, tab, P.tr + k, Bk.ix, Bk.iy, Bk.iz);
            {
                const TrDev T = P.tr[k];
                double x[3];
                frame_coords(T, Bk.ix, Bk.iy, Bk.iz, x);
                pair.setup(T, x, P.r0);
                pair.agree(Bk.valid);
            }
            if (nz) {
                Scatter<NB> sink;
                sink.hist = hist;
                sink.stride = tile;
                sink.first = tlo;
#pragma unroll
                for (int v = 0; v < NB; ++v) sink.p0[v] = p0[v];
                // every edge is evaluated on its own (those outside a quadrant
                // are set, as in the cube forward), so a tile's areas are the
                // cube forward's (see ArcCylinderPair::agree)
                pair.sweep(tlo, thi, sink, P.r0);
            }
        }
    }
    __syncthreads();
    // shell j holds the fine bins (j - 1) step + 1 .. j step, its area split
    // evenly over them (Remark 1), as in the cube forward
    const int S = P.step;
    const int64_t Mhi = P.Mlo + P.Mcount - 1;
    const int wn = thi - tlo + 1;
    for (int i = threadIdx.x; i < wn * S; i += kThreads) {
        const int jj = i / S;
        const int64_t m = (int64_t)(tlo + jj - 1) * S + 1 + (i - jj * S);
        if (m < P.Mlo || m > Mhi) continue;
#pragma unroll
        for (int v = 0; v < NB; ++v) f[((int64_t)v * P.K + k) * P.Mcount + (m - P.Mlo)] = hist[v * tile + jj] * S;
    }
}

// Estimated work of each (transducer, time tile) item of a shape group: the
// shells of every brick's window that fall in the tile, summed over the bricks
// (integers, so the FP64 sums are exact and independent of their order).
// One thread per (brick, transducer); cost[kk ntiles + t].
__global__ __launch_bounds__(kThreads) void k_tile_cost(KParams P, int nbricks, int tile, int ntiles,
                                                        double* __restrict__ cost)
{
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= (int64_t)nbricks * P.nk) return;
    const int b = (int)(g % nbricks), kk = (int)(g / nbricks);
    double lo[3], hi[3];
    brick_box(P, b, lo, hi);
    int wlo, whi;
    box_window(P, lo, hi, P.tr[P.kperm[kk]], wlo, whi);
    if (wlo > whi) return;
    const int J0 = (int)P.Jlo;
    for (int t = (wlo - J0) / tile; t <= (whi - J0) / tile; ++t) {
        const int a = max(wlo, J0 + t * tile), z = min(whi, J0 + t * tile + tile - 1);
        atomicAdd(&cost[(int64_t)kk * ntiles + t], (double)(z - a + 1));
    }
}

// ---------------------------------------------------------------------------
// adjoint, closed-form areas
// ---------------------------------------------------------------------------

// One work-group of one wave per (4 x 4 x 4 voxel cube, chunk of transducers):
// the wave stages its own window of W in LDS and gathers, with no work-group
// barrier, only the ordering of its own LDS operations.
template <int SHAPE, class AT, int NB, class Real, int IL>
__global__ __launch_bounds__(kWave, (closed_waves<SHAPE, AT, NB>())) void k_adj_wave(KParams P,
                                                                                     const Real* __restrict__ W,
                                                                                     Real* __restrict__ out,
                                                                                     double* __restrict__ z64,
                                                                                     int direct)
{
    constexpr int HE = wave_window_bytes<SHAPE>() / (int)sizeof(Real);
    __shared__ Real Ws[HE];              // [NB][HB]
    constexpr int HB = HE / NB;          // shells per pass
    __shared__ double box[SHAPE == 1 ? kBoxSlots * kWave : 1];
    __shared__ double tab[kArcTab];
    int x0, y0, z0;
    wave_cube(P, x0, y0, z0);
    const int l = threadIdx.x;
    const int ix = x0 + (l & 3), iy = y0 + ((l >> 2) & 3), iz = z0 + (l >> 4);
    const bool valid = ix < P.n[0] && iy < P.n[1] && iz < P.n[2];
    const int64_t idx = valid ? ix + P.n[0] * (iy + P.n[1] * (int64_t)iz) : 0;
    double acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0.0;
    load_arc_table<kWave>(tab);
    wave_lds_order();
    const int kbeg = blockIdx.y * P.kchunk, kend = min(P.nk, kbeg + P.kchunk);
    const int S = P.step;
    const int64_t Mhi = P.Mlo + P.Mcount - 1;
    for (int kk = kbeg; kk < kend; ++kk) {
        const int k = P.kperm[kk];
        int wlo, whi;
        typename PairOf<SHAPE, Real, IL, kWave>::type pair;
        pair.bind(box, P.lut, tab, P.tr + k, ix, iy, iz);
        {
            const TrDev T = P.tr[k];
            double x[3];
            frame_coords(T, ix, iy, iz, x);
            int lo = 0x7fffffff, hi = -0x7fffffff - 1;
            if (valid) pair_range<SHAPE>(T, x, P.r0, lo, hi);
            wave_window(P, lo, hi, wlo, whi);
            if (wlo > whi) continue;   // no shell kept: a cylinder's set-up costs more than all else here
            pair.setup(T, x, P.r0);
            pair.agree(valid);
        }
        for (int plo = wlo; plo <= whi; plo += HB) {
            const int phi = min(whi, plo + HB - 1);
            const int wn = phi - plo + 1;
            wave_lds_order();
            // transpose of the even split: each shell gathers its fine bins (Remark 1)
            for (int i = l; i < wn; i += kWave)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const Real* Wk = W + ((int64_t)b * P.K + k) * P.Mcount;
                    double a = 0.0;
                    for (int t = 0; t < S; ++t) {
                        const int64_t m = (int64_t)(plo + i - 1) * S + 1 + t;
                        if (m >= P.Mlo && m <= Mhi) a += (double)Wk[m - P.Mlo];
                    }
                    Ws[b * HB + i] = (Real)(a * S);
                }
            wave_lds_order();
            if (valid) {
                Gather<NB, AT, Real> sink;
                sink.Ws = Ws;
                sink.stride = HB;
                sink.first = plo;
#pragma unroll
                for (int b = 0; b < NB; ++b) sink.part[b] = AT(0);
                pair.sweep(plo, phi, sink, P.r0);
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] += (double)sink.part[b];
            }
        }
    }
    if (!valid) return;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (direct) out[b * P.N + idx] = (Real)acc[b];
        else unsafeAtomicAdd(&z64[b * P.N + idx], acc[b]);
    }
}

// ---------------------------------------------------------------------------
// quadrature over surface points (Alg. 2 / Alg. 6)
// ---------------------------------------------------------------------------

// The surface points of a transducer are a tensor grid in its frame: rows of the
// first surface coordinate, each a point (X, Y) of two frame coordinates, times
// columns of the second one along the third, so that a point's squared distance is
// one FMA on top of its row's.
// (Read through the constant address space: the same for every lane, so a scalar load.)
typedef const __attribute__((address_space(4))) double ConstDouble;
struct QuadFrame {
    double p0, p1, pc;   // the voxel's coordinates against the rows and the columns
    __device__ __forceinline__ QuadFrame(const TrDev& T, int ix, int iy, int iz)
    {
        double x[3];
        frame_coords(T, ix, iy, iz, x);
        p0 = x[0];
        p1 = T.shape == 0 ? x[2] : x[1];
        pc = T.shape == 0 ? x[1] : x[2];
    }
    __device__ __forceinline__ double row2(const ConstDouble* w) const
    {
        const double a = p0 - w[0], b = p1 - w[1];
        return fma(a, a, b * b);
    }
};

// bin of the distance sqrt(r2): [r0 + m - 1, r0 + m), decided in FP64
__device__ __forceinline__ int point_bin(double r2, double r0)
{
    const int m = (int)floor(sqrt64(r2) - r0) + 1;
    double e = r0 + (double)(m - 1);
    if (r2 < e * e) return m - 1;
    e += 1.0;
    if (!(r2 < e * e)) return m + 1;
    return m;
}

// the inverse distance of the weights
template <class AT> __device__ __forceinline__ AT inv_dist(double r2, float inv);
template <> __device__ __forceinline__ float inv_dist<float>(double, float inv) { return inv; }
template <> __device__ __forceinline__ double inv_dist<double>(double r2, float) { return rsq64(r2); }

// Half a bin less the error of the FP32 estimate of a distance below rmax
// (2.8e-7 of it: conversions, v_rsq_f32, one FMA against the rounded r0)
__device__ __forceinline__ float sure_half(double rmax) { return (float)(0.5 - 3e-7 * rmax); }

// Bins and inverse distances of kQuadPoints points at squared distances row2 +
// (pc - col)^2.  The FP32 distance decides the bin unless it falls within its
// own error of an edge; then (in 6 % of the wave's steps at 2000 bins) the wave
// decides in FP64.
constexpr int kQuadPoints = 2;
template <class AT, int G>
__device__ __forceinline__ void quad_points(double row2, double pc, const ConstDouble* col, double r0,
                                            float r0f, float half, int (&m)[G], AT (&inv)[G])
{
    double r2[G];
    bool unsure = false;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const double d = pc - col[g];
        r2[g] = fma(d, d, row2);
        const float f = (float)r2[g], i = __builtin_amdgcn_rsqf(f);
        const float t = fmaf(f, i, -r0f), fl = floorf(t);
        m[g] = (int)fl + 1;
        unsure |= !(fabsf((t - fl) - 0.5f) < half);
        inv[g] = inv_dist<AT>(r2[g], i);
    }
    if (__any(unsure))
#pragma unroll
        for (int g = 0; g < G; ++g) m[g] = point_bin(r2[g], r0);
}

// Bound by VALU issue: per point two FP64 operations, one FP32 reciprocal root
// for bin and weight, and the sink's.  Before, each point took six FP64
// operations from its global coordinates and two FP64 comparisons of its bin.
// 128^3 voxels x 256 cylinders x 16 x 16 points, FP32: A 141 -> 108 ms, A^T 103 ->
// 63 ms; FP64: 159 -> 127, 140 -> 106; the same bins and weights bit for bit (97 and 60,
// 120 and 104 ms with the order and number of work-groups as they are now).  The
// forward is left with its runs: in nearly every step some lane's run ends and
// the wave steps through the flush.
template <class AT, int NB, class Real>
__global__ __launch_bounds__(kThreads) void k_fwd_quad(KParams P, const Real* __restrict__ coef,
                                                        double* __restrict__ f)
{
    constexpr int HB = kHistQuad;   // bins per pass
    extern __shared__ double hist[];
    Brick Bk;
    const unsigned line = blockIdx.x / (unsigned)P.nbx;   // row of bricks
    brick_setup(P, (int)(line * P.nbx + spread_column(blockIdx.x, line, P.nbx)), Bk);
    double p0[NB];
    bool nz = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        p0[b] = Bk.valid ? (double)coef[b * P.N + Bk.idx] : 0.0;
        nz |= p0[b] != 0.0;
    }
    if (!__syncthreads_or(nz)) return;
    const float r0f = (float)P.r0;
    const int kbeg = blockIdx.y * P.kchunk, kend = min(P.nk, kbeg + P.kchunk);
    for (int kk = kbeg; kk < kend; ++kk) {
        const int k = P.kperm[kk];
        const TrDev T = P.tr[k];
        const ConstDouble* row = (const ConstDouble*)(P.qrow + (int64_t)k * 2 * P.qn1);
        const ConstDouble* col = (const ConstDouble*)(P.qcol + (int64_t)k * P.qn2);
        const AT dA = (AT)P.qdA[k];
        const QuadFrame F(T, Bk.ix, Bk.iy, Bk.iz);
        int wlo, whi;
        brick_window(P, Bk, T, wlo, whi);
        const float half = sure_half(P.r0 + whi + 1);
        for (int plo = wlo; plo <= whi; plo += HB) {
            const int phi = min(whi, plo + HB - 1);
            const int wn = phi - plo + 1;
            for (int i = threadIdx.x; i < wn; i += kThreads)
#pragma unroll
                for (int b = 0; b < NB; ++b) hist[b * HB + i] = 0.0;
            __syncthreads();
            if (nz) {
                // consecutive points in one bin add up in a register
                int mcur = plo - 1;
                AT acc = AT(0);
                auto flush = [&]() {
                    if ((unsigned)(mcur - plo) < (unsigned)wn)
#pragma unroll
                        for (int b = 0; b < NB; ++b) atomicAdd(&hist[b * HB + (mcur - plo)], p0[b] * (double)acc);
                };
                auto add = [&](int m, AT cv) {
                    if (m != mcur) {
                        flush();
                        mcur = m;
                        acc = cv;
                    } else {
                        acc += cv;
                    }
                };
                for (int a = 0; a < P.qn1; ++a) {
                    const double r2 = F.row2(row + 2 * a);
                    int q = 0;
                    for (; q + kQuadPoints <= P.qn2; q += kQuadPoints) {
                        int m[kQuadPoints];
                        AT inv[kQuadPoints];
                        quad_points<AT>(r2, F.pc, col + q, P.r0, r0f, half, m, inv);
#pragma unroll
                        for (int g = 0; g < kQuadPoints; ++g) add(m[g], dA * inv[g]);
                    }
                    for (; q < P.qn2; ++q) {
                        int m[1];
                        AT inv[1];
                        quad_points<AT>(r2, F.pc, col + q, P.r0, r0f, half, m, inv);
                        add(m[0], dA * inv[0]);
                    }
                }
                flush();
            }
            __syncthreads();
            const int64_t fo = (plo - P.Mlo);
            for (int i = threadIdx.x; i < wn; i += kThreads)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    double v = hist[b * HB + i];
                    if (v != 0.0) unsafeAtomicAdd(&f[((int64_t)b * P.K + k) * P.Mcount + fo + i], v);
                }
            __syncthreads();
        }
    }
}

template <class AT, int NB, class Real>
__global__ __launch_bounds__(kThreads) void k_adj_quad(KParams P, const Real* __restrict__ W,
                                                        Real* __restrict__ out, double* __restrict__ z64,
                                                        int direct)
{
    constexpr int HB = kHistQuad;   // bins per pass
    extern __shared__ double smem_d[];
    Real* Ws = reinterpret_cast<Real*>(smem_d);
    Brick Bk;
    const unsigned line = blockIdx.x / (unsigned)P.nbx;   // row of bricks
    brick_setup(P, (int)(line * P.nbx + spread_column(blockIdx.x, line, P.nbx)), Bk);
    double acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0.0;
    const float r0f = (float)P.r0;
    const int kbeg = blockIdx.y * P.kchunk, kend = min(P.nk, kbeg + P.kchunk);
    for (int kk = kbeg; kk < kend; ++kk) {
        const int k = P.kperm[kk];
        const TrDev T = P.tr[k];
        const ConstDouble* row = (const ConstDouble*)(P.qrow + (int64_t)k * 2 * P.qn1);
        const ConstDouble* col = (const ConstDouble*)(P.qcol + (int64_t)k * P.qn2);
        const AT dA = (AT)P.qdA[k];
        const QuadFrame F(T, Bk.ix, Bk.iy, Bk.iz);
        int wlo, whi;
        brick_window(P, Bk, T, wlo, whi);
        const float half = sure_half(P.r0 + whi + 1);
        for (int plo = wlo; plo <= whi; plo += HB) {
            const int phi = min(whi, plo + HB - 1);
            const int wn = phi - plo + 1;
            __syncthreads();
            const int64_t fo = (plo - P.Mlo);
            for (int i = threadIdx.x; i < wn; i += kThreads)
#pragma unroll
                for (int b = 0; b < NB; ++b) Ws[b * HB + i] = W[((int64_t)b * P.K + k) * P.Mcount + fo + i];
            __syncthreads();
            if (Bk.valid) {
                AT part[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) part[b] = AT(0);
                auto add = [&](int m, AT cv) {
                    if ((unsigned)(m - plo) >= (unsigned)wn) return;
#pragma unroll
                    for (int b = 0; b < NB; ++b) part[b] = fma(cv, (AT)Ws[b * HB + (m - plo)], part[b]);
                };
                for (int a = 0; a < P.qn1; ++a) {
                    const double r2 = F.row2(row + 2 * a);
                    int q = 0;
                    for (; q + kQuadPoints <= P.qn2; q += kQuadPoints) {
                        int m[kQuadPoints];
                        AT inv[kQuadPoints];
                        quad_points<AT>(r2, F.pc, col + q, P.r0, r0f, half, m, inv);
#pragma unroll
                        for (int g = 0; g < kQuadPoints; ++g) add(m[g], dA * inv[g]);
                    }
                    for (; q < P.qn2; ++q) {
                        int m[1];
                        AT inv[1];
                        quad_points<AT>(r2, F.pc, col + q, P.r0, r0f, half, m, inv);
                        add(m[0], dA * inv[0]);
                    }
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[b] += (double)part[b];
            }
        }
    }
    if (!Bk.valid) return;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (direct) out[b * P.N + Bk.idx] = (Real)acc[b];
        else unsafeAtomicAdd(&z64[b * P.N + Bk.idx], acc[b]);
    }
}

// ---------------------------------------------------------------------------
// work count: area evaluations (closed form: one per quadrant and bin inside the
// kept range; quadrature: one per surface point) and voxel-transducer pairs
// ---------------------------------------------------------------------------

template <int SHAPE>
__global__ __launch_bounds__(kThreads) void k_count(KParams P, int quad, unsigned long long* __restrict__ out)
{
    __shared__ unsigned long long red[2];
    __shared__ double box[SHAPE == 1 ? kBoxSlots * kThreads : 1];
    __shared__ double tab[kArcTab];
    load_arc_table<kThreads>(tab);
    if (threadIdx.x < 2) red[threadIdx.x] = 0;
    __syncthreads();
    Brick Bk;
    brick_setup(P, blockIdx.x, Bk);
    unsigned long long evals = 0, pairs = 0;
    if (Bk.valid) {
        for (int kk = 0; kk < P.nk; ++kk) {
            const TrDev T = P.tr[P.kperm[kk]];
            if (quad) { evals += P.qn1 * P.qn2; pairs += 1; continue; }
            double x[3];
            frame_coords(T, Bk.ix, Bk.iy, Bk.iz, x);
            const int lo = (int)P.Jlo, hi = (int)P.Jhi;
            Count sink{0};
            typename PairOf<SHAPE, double, kIlExact>::type pair;
            pair.bind(box, nullptr, tab, P.tr + P.kperm[kk], Bk.ix, Bk.iy, Bk.iz);
            pair.setup(T, x, P.r0);
            pair.agree(true);
            pair.sweep(lo, hi, sink, P.r0);
            evals += sink.n;
            pairs += 1;
        }
    }
    atomicAdd(&red[0], evals);
    atomicAdd(&red[1], pairs);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&out[0], red[0]);
        atomicAdd(&out[1], red[1]);
    }
}

// ---------------------------------------------------------------------------
// support of the coefficients (the voxels the forward's sum over voxels needs)
// ---------------------------------------------------------------------------

template <class Real>
__device__ __forceinline__ bool voxel_nonzero(const KParams& P, const Brick& Bk, const Real* coef, int B)
{
    bool nz = false;
    if (Bk.valid)
        for (int b = 0; b < B; ++b) nz |= coef[b * P.N + Bk.idx] != Real(0);
    return nz;
}

// nonzero voxels per brick
template <class Real>
__global__ __launch_bounds__(kThreads) void k_support_count(KParams P, const Real* __restrict__ coef, int B,
                                                             const int32_t* __restrict__ order,
                                                             int32_t* __restrict__ cnt)
{
    Brick Bk;
    brick_setup(P, order[blockIdx.x], Bk);
    const int c = __syncthreads_count(voxel_nonzero(P, Bk, coef, B));
    if (threadIdx.x == 0) cnt[blockIdx.x] = c;
}

// inclusive prefix sum of v over the wave's lanes
__device__ __forceinline__ int wave_scan(int v)
{
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o);
        if (l >= o) v += t;
    }
    return v;
}

// exclusive prefix sums of the per-brick counts (one work-group); off[n] = total.
// Eight counts a thread and a scan within each wave, with one exchange between
// the waves per 2048 counts: 130 -> 36 us for 12500 bricks, where a scan over the
// work-group took sixteen barriers per 256 counts.
__global__ __launch_bounds__(kThreads) void k_support_scan(const int32_t* __restrict__ cnt, int n,
                                                            int32_t* __restrict__ off)
{
    constexpr int kEach = 8;
    __shared__ int wsum[2][kThreads / 64];
    const int w = threadIdx.x >> 6;
    int carry = 0, flip = 0;
    for (int base = 0; base < n; base += kThreads * kEach, flip ^= 1) {
        const int i0 = base + threadIdx.x * kEach;
        int v[kEach], sum = 0;
#pragma unroll
        for (int e = 0; e < kEach; ++e) {
            v[e] = i0 + e < n ? cnt[i0 + e] : 0;
            sum += v[e];
        }
        const int inc = wave_scan(sum);
        if ((threadIdx.x & 63) == 63) wsum[flip][w] = inc;
        __syncthreads();   // the other half of wsum is the previous trip's
        int at = carry + inc - sum;
#pragma unroll
        for (int u = 0; u < kThreads / 64; ++u) {
            if (u < w) at += wsum[flip][u];
            carry += wsum[flip][u];
        }
#pragma unroll
        for (int e = 0; e < kEach; ++e) {
            if (i0 + e < n) off[i0 + e] = at;
            at += v[e];
        }
    }
    if (threadIdx.x == 0) off[n] = carry;
}

// the nonzero voxels of each brick at the brick's offset, in thread order (the
// brick's four 4 x 4 x 4 cubes in turn); bricks in the order `order` (Morton
// order of the brick coordinates, so that consecutive entries lie in a compact
// cluster of bricks)
template <class Real>
__global__ __launch_bounds__(kThreads) void k_support_write(KParams P, const Real* __restrict__ coef, int B,
                                                             const int32_t* __restrict__ order,
                                                             const int32_t* __restrict__ off,
                                                             int32_t* __restrict__ list)
{
    __shared__ int wcount[kThreads / 64];
    Brick Bk;
    brick_setup(P, order[blockIdx.x], Bk);
    const bool nz = voxel_nonzero(P, Bk, coef, B);
    const unsigned long long m = __ballot(nz);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) wcount[w] = __popcll(m);
    __syncthreads();
    int base = off[blockIdx.x];
    for (int v = 0; v < w; ++v) base += wcount[v];
    if (nz) list[base + rank] = (int32_t)Bk.idx;
}

// ---------------------------------------------------------------------------
// temporal stage
// ---------------------------------------------------------------------------

// s_hat[b][k][l] = sum_j G[j] scale[m] f[b][k][m],  m = U l - (jlo + jj)  (0-based l).
// A work-group takes kFirL samples, four threads each, and stages scale f of their
// windows in LDS, as many taps at a time as fit: rows by m modulo U, so that the
// samples of one tap, U bins apart, are neighbours there.  What remains is one
// LDS read and one FMA per tap and sample.  Without it (each sample reading its
// bins with a stride of U through the caches) the stage took 930 us of a sparse
// forward with 64 x 2688 samples at U = 11 in FP64, and 10 us of latency at the
// smallest sizes: now 72 and 4.
constexpr int kFirL = 64;         // samples per work-group
constexpr int kFirTaps = 1024;    // taps staged at a time
constexpr int kFirMaxU = 48;      // up to here a window fits: kFirL U + kFirTaps + 2 U bins of 8 bytes
template <class Real>
__global__ __launch_bounds__(kThreads) void k_fir(const double* __restrict__ f, const double* __restrict__ scale,
                                                   const double* __restrict__ G, int jlo, int jcnt, int U, int L,
                                                   int K, int64_t Mlo, int64_t Mcount, Real* __restrict__ out)
{
    extern __shared__ double win[];
    __shared__ double red[kThreads];
    const int k = blockIdx.y, b = blockIdx.z, l0 = blockIdx.x * kFirL;
    const double* fk = f + ((int64_t)b * K + k) * Mcount;
    const int lt = threadIdx.x & (kFirL - 1), part = threadIdx.x / kFirL;
    // h sums to zero, so the samples are small differences of large terms:
    // accumulated in FP64
    double acc = 0.0;
    for (int jc = 0; jc < jcnt; jc += kFirTaps) {
        const int nj = min(kFirTaps, jcnt - jc);
        const int W = U * (kFirL - 1) + nj, row = kFirL + nj / U + 1;
        const int64_t m0 = (int64_t)U * l0 - jlo - (jc + nj - 1) - Mlo;   // first bin of the window
        __syncthreads();
        for (int i = threadIdx.x; i < W; i += kThreads) {
            const int64_t mi = m0 + i;
            const double v = mi >= 0 && mi < Mcount ? scale[mi] * fk[mi] : 0.0;
            const int q = U == 1 ? i : i / U;
            win[(i - q * U) * row + q] = v;
        }
        __syncthreads();
        // tap jc + nj - 1 - e of sample lt reads bin U lt + e of the window
        const int per = (nj + 3) / 4, e0 = part * per, e1 = min(nj, e0 + per);
        int q = U == 1 ? e0 : e0 / U, ph = e0 - q * U;
        const double* Ge = G + (jc + nj - 1);
#pragma unroll 4
        for (int e = e0; e < e1; ++e) {
            acc = fma(Ge[-e], win[ph * row + q + lt], acc);
            if (++ph == U) { ph = 0; ++q; }
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    const int l = l0 + lt;
    if (part == 0 && l < L)
        out[((int64_t)b * K + k) * L + l] = (Real)((red[lt] + red[lt + kFirL]) + (red[lt + 2 * kFirL] + red[lt + 3 * kFirL]));
}

// the same, one sample a thread, for up-sampling factors whose windows do not fit
// LDS: neighbouring threads' bins are then further apart than a cache line anyway
template <class Real>
__global__ void k_fir_wide(const double* __restrict__ f, const double* __restrict__ scale,
                           const double* __restrict__ G, int jlo, int jcnt, int U, int L, int K, int64_t Mlo,
                           int64_t Mcount, Real* __restrict__ out)
{
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y, b = blockIdx.z;
    if (l >= L) return;
    const double* fk = f + ((int64_t)b * K + k) * Mcount;
    double acc = 0.0;
    const int64_t top = (int64_t)U * l - jlo - Mlo;   // bin of tap 0
    const int j0 = (int)max((int64_t)0, top - (Mcount - 1)), j1 = (int)min((int64_t)jcnt - 1, top);
#pragma unroll 8
    for (int jj = j0; jj <= j1; ++jj) acc = fma(G[jj], scale[top - jj] * fk[top - jj], acc);
    out[((int64_t)b * K + k) * L + l] = (Real)acc;
}

// W[b][k][m] = scale[m] sum_l G[U l - m] y[b][k][l]; and z64 <- 0 (nz of them) for the sums
// that follow, in the same launch
template <class Real>
__global__ void k_adjw(const Real* __restrict__ y, const double* __restrict__ scale, const double* __restrict__ G,
                       int jlo, int jcnt, int U, int L, int K, int64_t Mlo, int64_t Mcount, Real* __restrict__ W,
                       double* __restrict__ z64, int64_t nz)
{
    const int64_t mi = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * gridDim.y * gridDim.z * blockDim.x;
    for (int64_t i = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x * blockDim.x + mi; i < nz; i += stride)
        z64[i] = 0.0;
    const int k = blockIdx.y, b = blockIdx.z;
    if (mi >= Mcount) return;
    const int m = (int)(Mlo + mi);
    const Real* yk = y + ((int64_t)b * K + k) * L;
    // U l - m = j in [jlo, jlo + jcnt - 1]
    int lmin = -floordiv(-(m + jlo), U);
    int lmax = floordiv(m + jlo + jcnt - 1, U);
    lmin = max(lmin, 0);
    lmax = min(lmax, L - 1);
    double acc = 0.0;
    const double* Gm = G - (m + jlo);
#pragma unroll 8
    for (int l = lmin; l <= lmax; ++l) acc = fma(Gm[U * l], (double)yk[l], acc);
    W[((int64_t)b * K + k) * Mcount + mi] = (Real)(scale[mi] * acc);
}

// ---------------------------------------------------------------------------
// E~ / F~ tables of the lookup-table I_l, one node per thread
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_lut_build(double2* __restrict__ T)
{
    const int id = blockIdx.x * 256 + threadIdx.x;
    if (id >= kLutN * kLutN) return;
    const double s = lut_node(id % kLutN), nu = lut_node(id / kLutN);
    double E = 0.0, F = 0.0;
    if (s > 0.0) {
        const double c = sqrt64<2>((1.0 - s) * (1.0 + s));   // cos(arcsin s)
        const double dl = sqrt64<2>(fma(-nu * s, s, 1.0));    // Delta(arcsin s)
        E = ellip_e_scd<2, true>(s, c, dl, nu, &F);
    }
    T[id] = make_double2(E, F);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

namespace {

template <int SHAPE, class AT, class Real, int IL>
hipError_t fwd_sparse_nb(int nb, dim3 grid, const KParams& P, const Real* coef, double* f, hipStream_t s)
{
    switch (nb) {
    case 1: k_fwd_sparse_wave<SHAPE, AT, 1, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    case 2: k_fwd_sparse_wave<SHAPE, AT, 2, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    case 4: k_fwd_sparse_wave<SHAPE, AT, 4, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    default: k_fwd_sparse_wave<SHAPE, AT, 8, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    }
    return hipGetLastError();
}

template <int SHAPE, class AT, class Real, int IL>
hipError_t fwd_wave_nb(int nb, dim3 grid, const KParams& P, const Real* coef, double* f, hipStream_t s)
{
    switch (nb) {
    case 1: k_fwd_wave<SHAPE, AT, 1, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    case 2: k_fwd_wave<SHAPE, AT, 2, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    case 4: k_fwd_wave<SHAPE, AT, 4, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    default: k_fwd_wave<SHAPE, AT, 8, Real, IL><<<grid, kWave, 0, s>>>(P, coef, f); break;
    }
    return hipGetLastError();
}

template <int SHAPE, class AT, class Real, int IL>
hipError_t adj_wave_nb(int nb, dim3 grid, const KParams& P, const Real* W, Real* out, double* z64, int direct,
                       hipStream_t s)
{
    switch (nb) {
    case 1: k_adj_wave<SHAPE, AT, 1, Real, IL><<<grid, kWave, 0, s>>>(P, W, out, z64, direct); break;
    case 2: k_adj_wave<SHAPE, AT, 2, Real, IL><<<grid, kWave, 0, s>>>(P, W, out, z64, direct); break;
    case 4: k_adj_wave<SHAPE, AT, 4, Real, IL><<<grid, kWave, 0, s>>>(P, W, out, z64, direct); break;
    default: k_adj_wave<SHAPE, AT, 8, Real, IL><<<grid, kWave, 0, s>>>(P, W, out, z64, direct); break;
    }
    return hipGetLastError();
}

template <int SHAPE, class AT, class Real, int IL>
hipError_t fwd_tile_nb(int nb, const KParams& P, const int32_t* items, int nitems, int tile, int ntiles,
                       int nbricks, const Real* coef, double* f, hipStream_t s)
{
    const size_t sh = (size_t)nb * tile * sizeof(double);
    switch (nb) {
    case 1: k_fwd_tile<SHAPE, AT, 1, Real, IL><<<nitems, kThreads, sh, s>>>(P, items, tile, ntiles, nbricks, coef, f); break;
    case 2: k_fwd_tile<SHAPE, AT, 2, Real, IL><<<nitems, kThreads, sh, s>>>(P, items, tile, ntiles, nbricks, coef, f); break;
    case 4: k_fwd_tile<SHAPE, AT, 4, Real, IL><<<nitems, kThreads, sh, s>>>(P, items, tile, ntiles, nbricks, coef, f); break;
    default: k_fwd_tile<SHAPE, AT, 8, Real, IL><<<nitems, kThreads, sh, s>>>(P, items, tile, ntiles, nbricks, coef, f); break;
    }
    return hipGetLastError();
}

template <class Real>
hipError_t fwd_tile_cyl(int mode, bool carlson, int nb, const KParams& P, const int32_t* items, int nitems, int tile, int ntiles,
                        int nbricks, const Real* coef, double* f, hipStream_t s)
{
    if (mode == 2)
        return fwd_tile_nb<1, double, Real, kIlTrapezoid>(nb, P, items, nitems, tile, ntiles, nbricks, coef, f, s);
    if (mode == 3)
        return fwd_tile_nb<1, double, Real, kIlTable>(nb, P, items, nitems, tile, ntiles, nbricks, coef, f, s);
    if (carlson) return fwd_tile_nb<1, double, Real, kIlCarlson>(nb, P, items, nitems, tile, ntiles, nbricks, coef, f, s);
    return fwd_tile_nb<1, double, Real, kIlExact>(nb, P, items, nitems, tile, ntiles, nbricks, coef, f, s);
}

// cylinder launches by I_l variant: area mode 0 exact, 2 trapezoid, 3 tables
template <class Real>
hipError_t fwd_sparse_cyl(int mode, bool carlson, int nb, dim3 grid, const KParams& P, const Real* coef, double* f, hipStream_t s)
{
    if (mode == 2) return fwd_sparse_nb<1, double, Real, kIlTrapezoid>(nb, grid, P, coef, f, s);
    if (mode == 3) return fwd_sparse_nb<1, double, Real, kIlTable>(nb, grid, P, coef, f, s);
    if (carlson) return fwd_sparse_nb<1, double, Real, kIlCarlson>(nb, grid, P, coef, f, s);
    return fwd_sparse_nb<1, double, Real, kIlExact>(nb, grid, P, coef, f, s);
}

template <class Real>
hipError_t fwd_wave_cyl(int mode, bool carlson, int nb, dim3 grid, const KParams& P, const Real* coef, double* f,
                        hipStream_t s)
{
    if (mode == 2) return fwd_wave_nb<1, double, Real, kIlTrapezoid>(nb, grid, P, coef, f, s);
    if (mode == 3) return fwd_wave_nb<1, double, Real, kIlTable>(nb, grid, P, coef, f, s);
    if (carlson) return fwd_wave_nb<1, double, Real, kIlCarlson>(nb, grid, P, coef, f, s);
    return fwd_wave_nb<1, double, Real, kIlExact>(nb, grid, P, coef, f, s);
}

template <class Real>
hipError_t adj_wave_cyl(int mode, bool carlson, int nb, dim3 grid, const KParams& P, const Real* W, Real* out,
                        double* z64, int direct, hipStream_t s)
{
    if (mode == 2) return adj_wave_nb<1, double, Real, kIlTrapezoid>(nb, grid, P, W, out, z64, direct, s);
    if (mode == 3) return adj_wave_nb<1, double, Real, kIlTable>(nb, grid, P, W, out, z64, direct, s);
    if (carlson) return adj_wave_nb<1, double, Real, kIlCarlson>(nb, grid, P, W, out, z64, direct, s);
    return adj_wave_nb<1, double, Real, kIlExact>(nb, grid, P, W, out, z64, direct, s);
}

template <class AT, class Real>
hipError_t fwd_quad_nb(int nb, dim3 grid, const KParams& P, const Real* coef, double* f, hipStream_t s)
{
    size_t sh = (size_t)nb * kHistQuad * sizeof(double);
    switch (nb) {
    case 1: k_fwd_quad<AT, 1, Real><<<grid, kThreads, sh, s>>>(P, coef, f); break;
    case 2: k_fwd_quad<AT, 2, Real><<<grid, kThreads, sh, s>>>(P, coef, f); break;
    case 4: k_fwd_quad<AT, 4, Real><<<grid, kThreads, sh, s>>>(P, coef, f); break;
    default: k_fwd_quad<AT, 8, Real><<<grid, kThreads, sh, s>>>(P, coef, f); break;
    }
    return hipGetLastError();
}

template <class AT, class Real>
hipError_t adj_quad_nb(int nb, dim3 grid, const KParams& P, const Real* W, Real* out, double* z64, int direct,
                       hipStream_t s)
{
    size_t sh = (size_t)nb * kHistQuad * sizeof(Real);
    switch (nb) {
    case 1: k_adj_quad<AT, 1, Real><<<grid, kThreads, sh, s>>>(P, W, out, z64, direct); break;
    case 2: k_adj_quad<AT, 2, Real><<<grid, kThreads, sh, s>>>(P, W, out, z64, direct); break;
    case 4: k_adj_quad<AT, 4, Real><<<grid, kThreads, sh, s>>>(P, W, out, z64, direct); break;
    default: k_adj_quad<AT, 8, Real><<<grid, kThreads, sh, s>>>(P, W, out, z64, direct); break;
    }
    return hipGetLastError();
}

int chunk_nb(int rem)
{
    return rem >= 8 ? 8 : rem >= 4 ? 4 : rem >= 2 ? 2 : 1;
}

int grid_fill_blocks(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

template <class Real>
hipError_t forward_t(const LaunchPlan& L, const Real* coef, Real* sig, int B, hipStream_t s, bool sparse)
{
    hipError_t e;
    // the (transducer, time tile) forward stores every fine bin of f itself
    const bool tiles = L.tile > 0 && !sparse && L.mode != 1;
    if (!tiles) {
        const int64_t nf = (int64_t)B * L.base.K * L.base.Mcount;
        k_fill<<<grid_fill_blocks(nf), 256, 0, s>>>(L.f, nf);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (sparse) {
        // support of the whole batch: the voxels with a nonzero coefficient in any volume
        k_support_count<Real><<<L.nbricks, kThreads, 0, s>>>(L.base, coef, B, L.sup_order, L.sup_cnt);
        k_support_scan<<<1, kThreads, 0, s>>>(L.sup_cnt, L.nbricks, L.sup_off);
        k_support_write<Real><<<L.nbricks, kThreads, 0, s>>>(L.base, coef, B, L.sup_order, L.sup_off, L.sup_list);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int b0 = 0; b0 < B;) {
        const int nb = chunk_nb(B - b0);
        for (int g = 0; g < L.ngroups; ++g) {
            const ShapeGroup& G = L.groups[g];
            KParams P = L.base;
            P.kperm = G.kperm;
            P.nk = G.nk;
            P.kchunk = G.kchunk_fwd;
            P.B = nb;
            dim3 grid(L.nbricks, (G.nk + G.kchunk_fwd - 1) / G.kchunk_fwd);
            const Real* cb = coef + (int64_t)b0 * P.N;
            double* fb = L.f + (int64_t)b0 * P.K * P.Mcount;
            if (sparse) {
                P.sup_list = L.sup_list;
                P.sup_total = L.sup_off + L.nbricks;
                P.kchunk = kSparseChunk;
                grid = dim3(kSparseGrid * (kThreads / kWave), 1);
            }
            if (L.mode == 1) e = fwd_quad_nb<Real, Real>(nb, grid, P, cb, fb, s);
            else if (tiles && G.shape == 0)
                e = fwd_tile_nb<0, Real, Real, kIlExact>(nb, P, G.items, G.nitems, L.tile, L.ntiles, L.nbricks, cb,
                                                         fb, s);
            else if (tiles)
                e = fwd_tile_cyl<Real>(L.mode, G.carlson, nb, P, G.items, G.nitems, L.tile, L.ntiles, L.nbricks, cb, fb, s);
            else if (sparse && G.shape == 0) e = fwd_sparse_nb<0, Real, Real, kIlExact>(nb, grid, P, cb, fb, s);
            else if (sparse) e = fwd_sparse_cyl<Real>(L.mode, G.carlson, nb, grid, P, cb, fb, s);
            else {
                const dim3 gw((unsigned)L.ncubes, (G.nk + G.kchunk_fwd - 1) / G.kchunk_fwd);
                if (G.shape == 0) e = fwd_wave_nb<0, Real, Real, kIlExact>(nb, gw, P, cb, fb, s);
                else e = fwd_wave_cyl<Real>(L.mode, G.carlson, nb, gw, P, cb, fb, s);
            }
            if (e != hipSuccess) return e;
        }
        b0 += nb;
    }
    if (L.U <= kFirMaxU) {
        const dim3 g2((L.L + kFirL - 1) / kFirL, L.base.K, B);
        const int nj = L.jcnt < kFirTaps ? L.jcnt : kFirTaps;
        const size_t sh = sizeof(double) * (size_t)L.U * (kFirL + nj / L.U + 1);
        k_fir<Real><<<g2, kThreads, sh, s>>>(L.f, L.scale, L.G, L.jlo, L.jcnt, L.U, L.L, L.base.K, L.base.Mlo,
                                             L.base.Mcount, sig);
    } else {
        const dim3 g2((L.L + 255) / 256, L.base.K, B);
        k_fir_wide<Real><<<g2, 256, 0, s>>>(L.f, L.scale, L.G, L.jlo, L.jcnt, L.U, L.L, L.base.K, L.base.Mlo,
                                            L.base.Mcount, sig);
    }
    return hipGetLastError();
}

template <class Real>
hipError_t adjoint_t(const LaunchPlan& L, const Real* sig, Real* coef, int B, hipStream_t s)
{
    hipError_t e;
    Real* W = (Real*)L.W;
    const bool direct = L.ngroups == 1 && L.groups[0].kchunk_adj >= L.groups[0].nk;
    const int64_t nz = (int64_t)B * L.base.N;
    const dim3 g1((unsigned)adjw_blocks(L.base.Mcount, (int64_t)L.base.K * B, direct ? 0 : nz), L.base.K, B);
    k_adjw<Real><<<g1, 256, 0, s>>>(sig, L.scale, L.G, L.jlo, L.jcnt, L.U, L.L, L.base.K, L.base.Mlo, L.base.Mcount,
                                    W, L.z64, direct ? 0 : nz);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int b0 = 0; b0 < B;) {
        const int nb = chunk_nb(B - b0);
        for (int g = 0; g < L.ngroups; ++g) {
            const ShapeGroup& G = L.groups[g];
            KParams P = L.base;
            P.kperm = G.kperm;
            P.nk = G.nk;
            P.kchunk = G.kchunk_adj;
            P.B = nb;
            dim3 grid(L.nbricks, (G.nk + G.kchunk_adj - 1) / G.kchunk_adj);
            const Real* Wb = W + (int64_t)b0 * P.K * P.Mcount;
            Real* ob = coef + (int64_t)b0 * P.N;
            double* zb = L.z64 + (int64_t)b0 * P.N;
            if (L.mode == 1) e = adj_quad_nb<Real, Real>(nb, grid, P, Wb, ob, zb, direct, s);
            else {
                const dim3 gw((unsigned)L.ncubes, (G.nk + G.kchunk_adj - 1) / G.kchunk_adj);
                if (G.shape == 0) e = adj_wave_nb<0, Real, Real, kIlExact>(nb, gw, P, Wb, ob, zb, direct, s);
                else e = adj_wave_cyl<Real>(L.mode, G.carlson, nb, gw, P, Wb, ob, zb, direct, s);
            }
            if (e != hipSuccess) return e;
        }
        b0 += nb;
    }
    if (!direct) {
        k_finish<Real><<<grid_fill_blocks(nz), 256, 0, s>>>(L.z64, coef, nz);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_count(const LaunchPlan& L, unsigned long long* out, hipStream_t s)
{
    for (int g = 0; g < L.ngroups; ++g) {
        KParams P = L.base;
        P.kperm = L.groups[g].kperm;
        P.nk = L.groups[g].nk;
        if (L.groups[g].shape == 0) k_count<0><<<L.nbricks, kThreads, 0, s>>>(P, L.mode == 1, out);
        else k_count<1><<<L.nbricks, kThreads, 0, s>>>(P, L.mode == 1, out);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_tile_cost(const KParams& P, int nbricks, int tile, int ntiles, double* cost, hipStream_t s)
{
    const int64_t n = (int64_t)nbricks * P.nk;
    k_tile_cost<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(P, nbricks, tile, ntiles, cost);
    return hipGetLastError();
}

hipError_t launch_forward(const LaunchPlan& L, const void* coef, void* sig, int B, hipStream_t s)
{
    if (L.fp64) return forward_t<double>(L, (const double*)coef, (double*)sig, B, s, false);
    return forward_t<float>(L, (const float*)coef, (float*)sig, B, s, false);
}

hipError_t launch_lut_build(double2* table, hipStream_t s)
{
    k_lut_build<<<(kLutN * kLutN + 255) / 256, 256, 0, s>>>(table);
    return hipGetLastError();
}

hipError_t launch_forward_sparse(const LaunchPlan& L, const void* coef, void* sig, int B, hipStream_t s)
{
    if (L.mode == 1) return hipErrorNotSupported;
    if (L.fp64) return forward_t<double>(L, (const double*)coef, (double*)sig, B, s, true);
    return forward_t<float>(L, (const float*)coef, (float*)sig, B, s, true);
}

hipError_t launch_adjoint(const LaunchPlan& L, const void* sig, void* coef, int B, hipStream_t s)
{
    if (L.fp64) return adjoint_t<double>(L, (const double*)sig, (double*)coef, B, s);
    return adjoint_t<float>(L, (const float*)sig, (float*)coef, B, s);
}

}  // namespace patop
