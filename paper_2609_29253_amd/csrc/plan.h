// Rules of the launch plan that follow from the geometry alone, on the host.
#pragma once

#include <algorithm>
#include <cmath>

#include "pairs.h"

namespace patop {

// Up to kSampled transducers of n, spread over them, stand for all: an array's
// elements are alike, and its set-up should not grow by a rule's cost (arc_share over all
// of 512 cylinders took 0.63 ms of 1.43, of 16384 20 of 43)
constexpr int kSampled = 32;
inline int sample_count(int n) { return std::min(n, kSampled); }
inline int sample_index(int i, int n) { return n <= kSampled ? i : (int)((int64_t)i * (n - 1) / (kSampled - 1)); }

// coordinate of the q-th of four sampled voxels along an axis of n
inline double sample_voxel(int64_t n, int q) { return (double)(n - 1) * (q + 0.5) / 4.0; }

// Work of a voxel-transducer pair, on average over 4 x 4 x 4 voxels of the grid and
// sampled transducers: shells of the distance window that are kept (P.r0, P.Jlo,
// P.Jhi), or the quadrature's points where any shell is.
inline double mean_shells(const TrDev* T, const int32_t* perm, int n, const KParams& P)
{
    double sum = 0.0;
    const int count = sample_count(n);
    for (int i = 0; i < count; ++i) {
        const TrDev& t = T[perm[sample_index(i, n)]];
        for (int v = 0; v < 64; ++v) {
            double d2 = 0.0;
            for (int a = 0; a < 3; ++a) {
                const double d = P.origin[a] + P.w * sample_voxel(P.n[a], (v >> (2 * a)) & 3) - t.cen[a];
                d2 += d * d;
            }
            const double d = std::sqrt(d2) - P.r0;
            const double lo = std::max(std::floor(d - t.rad), (double)P.Jlo), hi = std::min(std::ceil(d + t.rad), (double)P.Jhi);
            if (lo <= hi) sum += P.qn1 > 0 ? (double)P.qn1 * P.qn2 : hi - lo + 1.0;
        }
    }
    return sum / (64.0 * count);
}

// The share of the cylinders' pairs that the weighted areas serve (arc_fit), on the
// same voxels and transducers
template <int NW>
inline double arc_share(const TrDev* T, const int32_t* perm, int n, const KParams& P)
{
    int64_t fit = 0;
    const int count = sample_count(n);
    for (int i = 0; i < count; ++i) {
        const TrDev& t = T[perm[sample_index(i, n)]];
        for (int v = 0; v < 64; ++v) {
            double x[3];
            for (int a = 0; a < 3; ++a) {
                x[a] = t.base[a];
                for (int q = 0; q < 3; ++q) x[a] += t.g[a][q] * sample_voxel(P.n[q], (v >> (2 * q)) & 3);
            }
            const double rho = std::hypot(x[0], x[1]), ct = rho > 0.0 ? x[0] / rho : 1.0, st = rho > 0.0 ? std::fabs(x[1]) / rho : 0.0;
            const double cm = ct * t.cth + st * t.sth, sm = st * t.cth - ct * t.sth;
            const double cp = ct * t.cth - st * t.sth, sp = st * t.cth + ct * t.sth;
            const bool in0 = sm < 0.0, inpi = !in0 && sp < 0.0;
            fit += arc_fit<NW>(t.p[0], rho, in0 ? 1.0 : inpi ? cp : cm, in0 ? cm : inpi ? -1.0 : cp, cm, cp, true, in0 || inpi,
                               std::fabs(x[2]) + t.p[2], inpi)
                       .fits();
        }
    }
    return (double)fit / (64.0 * count);
}

// Whether a group of cylinders takes the kernels that evaluate every pair by Carlson's
// integral: waves that hold both kinds of pair step through both.  Below a share of
// 0.2 Carlson alone is faster (64 cylinders, A / A^T in ms, Carlson against mixed: FP32,
// 32^3 voxels near the axis, none served, 0.91 / 0.99 against 1.00 / 1.10, 48^3 at 0.09 4.70 /
// 5.05 against 4.98 / 5.45, 64^3 at 0.20 11.1 / 12.1 against 10.8 / 12.1, 0.39 6.48 / 7.19 against
// 5.89 / 6.79; FP64, 48^3, none served, 3.21 / 3.53 against 3.29 / 3.60, 96^3 at 0.24 24.7 / 25.6
// against 23.7 / 25.0).  A launch of few waves lasts as long as its slowest ones,
// which hold both kinds, so there every sampled pair has to be served (elements of
// a scan, us: FP32, 13824 waves, 0.93 served, 107 / 112 against 116 / 123, 21952 waves 171 / 191
// against 159 / 188; FP64, 21952 waves, 0.79 served, 189 / 210 against 212 / 242, 32768 waves
// 288 / 309 against 279 / 300).
inline bool carlson_only(double share, int64_t waves, bool fp64)
{
    return share < (waves < (fp64 ? 24576 : 16384) ? 1.0 : 0.2);
}

// Transducers per work-group of the adjoint: as many work-groups as 4096 of a brick's
// size, and two chunks where one work-group could see every transducer but the waves
// are few and the work is enough.  A voxel's sum has one order where at most two
// terms are added to the zero that it starts from, hence two, and only for an
// array of one shape (two shapes would make four).  Two chunks halve the last
// round (128^3 x 256 cylinders 67.5 -> 64.6 ms, quadrature 61.8 -> 59.5, 256 rectangles
// 10.6 -> 10.3, and more where the rounds are few: 100 x 98 x 110 x 5 elements of a scan 0.68 ->
// 0.56) at the cost of sums cleared, added and cast in memory.  Measured on 128^3
// voxels, W = shells per voxel: rectangles, one volume, 8 (W = 380) 0.347 -> 0.350 ms, 16
// (W = 770) 0.677 -> 0.669; eight volumes, 8 0.47 -> 0.54, 24 (W = 1150) 1.37 -> 1.39, 32
// (W = 1540) 1.83 -> 1.82; 32 with 128 samples kept 0.21 -> 0.42; cylinders, one volume,
// 2 (W = 450) 0.55 -> 0.56, 3 (W = 670) 0.81 -> 0.80, eight, 4 (W = 900) 1.29 -> 1.34, 8 (W =
// 1800) 2.60 -> 2.58; quadrature, one volume, 2 (W = 512) 0.495 -> 0.507, 3 (W = 770) 0.735 ->
// 0.728, eight, 6 (W = 1540) 2.42 -> 2.43, 8 (W = 2050) 3.23 -> 3.22.  So from W = 448 + 160 volumes on.
inline int adjoint_chunk(int nk, int64_t nbricks, bool one_shape, double shells, int volumes)
{
    const int64_t target = 4096;
    const int64_t nchunks = std::max<int64_t>(1, std::min<int64_t>(nk, (target + nbricks - 1) / nbricks));
    const int chunk = (int)((nk + nchunks - 1) / nchunks);
    if (one_shape && nbricks < 4 * target && nk * shells >= 448.0 + 160.0 * volumes) return std::min(chunk, (nk + 1) / 2);
    return chunk;
}

// Work-groups of 256 per transducer and volume of the launch that forms W and clears the
// adjoint's sums: what W's bins need, or, where the bins are few and the sums many (a
// short window over a large grid: 2 transducers x 256^3 voxels x 64 samples, 1.59 ms where a
// launch of its own to clear them took 0.56), what fills the device: 4096 in all.
inline int64_t adjw_blocks(int64_t bins, int64_t rows, int64_t sums)
{
    const int64_t fill = std::min<int64_t>(4096, (sums + 255) / 256);
    return std::max((bins + 255) / 256, (fill + rows - 1) / rows);
}

}  // namespace patop
