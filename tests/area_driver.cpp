// The kernels' pair sweeps on the host, for the CPU tests of their areas.
#include <hip/hip_runtime.h>

// area.h writes two FMAs as instructions; here they are what they say
#define asm(...) r = fma(a, b, c)
#include "pairs.h"
#undef asm

using namespace patop;

struct Sink {
    double* out;
    int lo;
    long n;
    int fetch(int) const { return 0; }
    void add(int m, double area, int)
    {
        out[m - lo] += area;
        ++n;
    }
    void operator()(int m, double area) { add(m, area, 0); }
    Sink give() const { return *this; }
    void take(const Sink& s) { n = s.n; }
};

template <class Pair>
static long sweep(const TrDev& T, const double* x, double r0, int lo, int hi, double* out)
{
    static double box[16];
    Sink sink{out, lo, 0};
    Pair p;
    p.bind(box, nullptr, kArcTable, &T, 0, 0, 0);
    p.setup(T, x, r0);
    p.sweep(lo, hi, sink, r0);
    return sink.n;
}

// areas of the bins lo .. hi of one pair; tr = shape and the three sizes, x the
// frame coordinates.  kind: 0 / 1 the kernels' sweep with FP32 / FP64 input and
// output, 2 / 3 a cylinder's by its elliptic integrals alone.  Returns the
// number of (quadrant, bin) areas.
extern "C" long pair_areas(const double* tr, const double* x, double r0, int lo, int hi, int kind, double* out)
{
    TrDev T;
    std::memset(&T, 0, sizeof T);
    T.shape = (int)tr[0];
    for (int i = 0; i < 3; ++i) {
        T.p[i] = tr[1 + i];
        T.base[i] = x[i];
    }
    if (T.shape == 0)
        return kind == 0 ? sweep<PairOf<0, float, kIlExact, 1>::type>(T, x, r0, lo, hi, out)
                         : sweep<PairOf<0, double, kIlExact, 1>::type>(T, x, r0, lo, hi, out);
    T.cth = std::cos(T.p[1]);
    T.sth = std::sin(T.p[1]);
    if (kind == 0) return sweep<PairOf<1, float, kIlExact, 1>::type>(T, x, r0, lo, hi, out);
    if (kind == 1) return sweep<PairOf<1, double, kIlExact, 1>::type>(T, x, r0, lo, hi, out);
    if (kind == 2) return sweep<CylinderPair<1, kIlExact, 1>>(T, x, r0, lo, hi, out);
    return sweep<CylinderPair<2, kIlExact, 1>>(T, x, r0, lo, hi, out);
}
