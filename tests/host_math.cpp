// The arithmetic of dsve_math.hpp compiled for the host, for tests: the hardware estimates stand in as
// correctly rounded values, off by a relative error that the test chooses.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

static double off = 0.0;   // relative error of the estimates
static float __builtin_amdgcn_rcpf(float x) { return (float)((1.0 / x) * (1.0 + off)); }
static float __builtin_amdgcn_rsqf(float x) { return (float)((1.0 / sqrt((double)x)) * (1.0 + off)); }
static float __builtin_amdgcn_sqrtf(float x) { return (float)(sqrt((double)x) * (1.0 + off)); }
static float __builtin_amdgcn_exp2f(float x) { return (float)(exp2((double)x) * (1.0 + off)); }
static float __builtin_amdgcn_logf(float x) { return (float)log2((double)x); }
static double __builtin_amdgcn_rcp(double x) { return (double)(float)(1.0 / x) * (1.0 + off); }
static double __builtin_amdgcn_rsq(double x) { return (double)(float)(1.0 / sqrt(x)) * (1.0 + off); }
static uint64_t __builtin_amdgcn_ballot_w64(bool b) { return b; }   // a wave of one lane
static double __longlong_as_double(long long v) { double d; memcpy(&d, &v, 8); return d; }
static long long __double_as_longlong(double d) { long long v; memcpy(&v, &d, 8); return v; }

#include "dsve_math.hpp"

using namespace dsve;

#define EACH(NAME, EXPR) \
    void NAME(const double *in, double *out, long n, double err) \
    { \
        off = err; \
        for (long i = 0; i < n; ++i) { const double a = in[i]; out[i] = EXPR; } \
    }
extern "C" {
EACH(host_rcbrt, rcbrt_h(a))
EACH(host_pow_1p1, pow_1p1(a))
EACH(host_sqrt, m_sqrt(a))
// b at depth a and |Fr| = 1/2, laws of the Shields stress (K_s = 40, d50 = 0.3 mm, S_g = 2.6)
static Closure shields(double lp0, double lp1)
{
    Closure K{};
    K.lp0 = lp0;
    K.lp1 = lp1;
    return K;
}
EACH(host_mpm, (law_b<CL_MPM, double>(shields(1.3, 2e-4), a, 0.5 * sqrt(9.81 * a) * a, 1.0 / a)))
EACH(host_vanrijn, (law_b<CL_VANRIJN, double>(shields(26.0, 4e-6), a, 0.5 * sqrt(9.81 * a) * a, 1.0 / a)))
}
