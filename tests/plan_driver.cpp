// The launch plan's rules on the host, for their CPU tests.
#include <hip/hip_runtime.h>

#include <vector>

// area.h writes two FMAs as instructions; here they are what they say
#define asm(...) r = fma(a, b, c)
#include "plan.h"
#undef asm

using namespace patop;

static std::vector<TrDev> table(const double* sphere, int nk, std::vector<int32_t>& perm)
{
    std::vector<TrDev> T(nk);
    for (int k = 0; k < nk; ++k) {
        std::memset(&T[k], 0, sizeof(TrDev));
        for (int a = 0; a < 3; ++a) T[k].cen[a] = sphere[4 * k + a];
        T[k].rad = sphere[4 * k + 3];
        perm.push_back(k);
    }
    return T;
}

// bounding spheres of nk transducers (in shells), a cube of n^3 voxels around 0
extern "C" int adjoint_chunk_of(const double* sphere, int nk, int n, double w, double r0, int jlo, int jhi, int points,
                                int one_shape, int volumes)
{
    std::vector<int32_t> perm;
    const auto T = table(sphere, nk, perm);
    KParams P;
    std::memset(&P, 0, sizeof P);
    for (int a = 0; a < 3; ++a) {
        P.n[a] = n;
        P.origin[a] = -0.5 * (n - 1) * w;
    }
    P.w = w;
    P.r0 = r0;
    P.Jlo = jlo;
    P.Jhi = jhi;
    P.qn1 = points;
    P.qn2 = points;
    const int64_t nbricks = (int64_t)((n + 7) / 8) * ((n + 7) / 8) * ((n + 3) / 4);
    return adjoint_chunk(nk, nbricks, one_shape, mean_shells(T.data(), perm.data(), nk, P), volumes);
}

extern "C" long adjw_blocks_of(long bins, long rows, long sums) { return adjw_blocks(bins, rows, sums); }

// cylinders (radius, theta_max, half length, frame coordinates of voxel 0), a cube of n^3
// voxels `w` apart along the frame's axes
extern "C" double arc_share_of(const double* cyl, int nk, int n, double w, int fp64)
{
    std::vector<TrDev> T(nk);
    std::vector<int32_t> perm;
    for (int k = 0; k < nk; ++k) {
        std::memset(&T[k], 0, sizeof(TrDev));
        for (int a = 0; a < 3; ++a) {
            T[k].p[a] = cyl[6 * k + a];
            T[k].base[a] = cyl[6 * k + 3 + a];
            T[k].g[a][a] = w;
        }
        T[k].cth = std::cos(T[k].p[1]);
        T[k].sth = std::sin(T[k].p[1]);
        perm.push_back(k);
    }
    KParams P;
    std::memset(&P, 0, sizeof P);
    for (int a = 0; a < 3; ++a) P.n[a] = n;
    return fp64 ? arc_share<2>(T.data(), perm.data(), nk, P) : arc_share<1>(T.data(), perm.data(), nk, P);
}

extern "C" int carlson_only_of(double share, long waves, int fp64) { return carlson_only(share, waves, fp64); }
