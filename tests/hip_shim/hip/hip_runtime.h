// Host stand-ins for the device names that the area headers use, so that their
// arithmetic compiles with a host compiler (one lane at a time).  The hardware
// seeds of reciprocals and roots are rounded to their own precision.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>

#define __device__
#define __host__
#define __forceinline__ inline

typedef int hipError_t;
typedef void* hipStream_t;
struct double2 {
    double x, y;
};
static struct {
    unsigned x;
} threadIdx;

using std::fma;
using std::fmax;
using std::fmin;
using std::max;
using std::min;

inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
inline float __builtin_amdgcn_rsqf(float x) { return 1.0f / std::sqrt(x); }
inline float __builtin_amdgcn_sqrtf(float x) { return std::sqrt(x); }
// v_rcp_f64 and v_rsq_f64 are good to about 2^-24
inline double short_mantissa(double x)
{
    uint64_t b;
    std::memcpy(&b, &x, 8);
    b &= ~((uint64_t(1) << 28) - 1);
    std::memcpy(&x, &b, 8);
    return x;
}
inline double __builtin_amdgcn_rcp(double x) { return short_mantissa(1.0 / x); }
inline double __builtin_amdgcn_rsq(double x) { return short_mantissa(1.0 / std::sqrt(x)); }
inline float __sinf(float x) { return std::sin(x); }
inline int __float_as_int(float f)
{
    int i;
    std::memcpy(&i, &f, 4);
    return i;
}
inline float __int_as_float(int i)
{
    float f;
    std::memcpy(&f, &i, 4);
    return f;
}
inline bool __any(bool b) { return b; }
inline bool __all(bool b) { return b; }
