// FP64 exponential and reciprocal square root for the kernels that are bound by
// them: N independent arguments are taken step by step together, so that their
// dependent chains overlap.
#pragma once
#include <hip/hip_runtime.h>

namespace pbm {

// 2^-r for 0 <= r < 2^30: r = n + f', |f'| <= 1/2, by adding 1.5 2^52 (the low word of
// the sum is then -n); 2^f as its degree-11 interpolation at the Chebyshev
// points of [-1/2, 1/2], relative error 2e-17 (coefficients from that
// interpolation in 50 digits).  15 instructions, 78 cycles per wavefront
// against 102 for the library's exp.
template <int N>
__device__ __forceinline__ void exp2neg_n(double (&x)[N])
{
    constexpr double c[12] = {1.0, 0.6931471805599453, 0.24022650695910158, 0.055504108664821625,
                              0.009618129107587256, 0.001333355814640647, 0.00015403530463724353,
                              1.5252733841556773e-05, 1.3215432535912375e-06, 1.0178057087733941e-07,
                              7.074194297288521e-09, 4.4558179083360645e-10};
    const double big = 6755399441055744.0;
    double p[N], f[N];
    int n[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const double t = big - x[i];
        n[i] = __double2loint(t);
        f[i] = (big - t) - x[i];
        p[i] = c[11];
    }
#pragma unroll
    for (int k = 10; k >= 0; --k)
#pragma unroll
        for (int i = 0; i < N; ++i) p[i] = fma(p[i], f[i], c[k]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = __builtin_amdgcn_ldexp(p[i], n[i]);
}

// 2^f for |f| <= 1/16: degree-7 interpolation at the Chebyshev points, relative
// error 6e-18.  With the triangles' centroids at distance r_0, the points of a
// triangle pair lie at r_0 + d, |d| at most the sum of the two triangles' largest
// offsets from their centroids, so where that sum is below 1/16 (in scaled
// coordinates; 0.05 at the benchmark's 10 vertices per square angstrom) one
// 2^-r_0 per triangle pair serves 36 point pairs and a pair's exponential takes 9
// instead of 15 instructions.
constexpr double kExpNear = 1.0 / 16.0;
template <int N>
__device__ __forceinline__ void exp2near_n(double (&x)[N])
{
    constexpr double c[8] = {1.0, 0.6931471805599453, 0.2402265069591204, 0.055504108664823096,
                             0.00961812908242099, 0.0013333558127014689, 0.00015404562882891175,
                             1.5253528985683798e-05};
    double p[N];
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = c[7];
#pragma unroll
    for (int k = 6; k >= 0; --k)
#pragma unroll
        for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], c[k]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = p[i];
}

// 1/sqrt(x): the hardware estimate (relative error 5.3e-8) and one third-order
// step, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2: error 1.4e-16, as after two
// Newton steps, in three instructions fewer
template <int N>
__device__ __forceinline__ void rsqrt3_n(const double (&x)[N], double (&y)[N])
{
    double e[N], h[N];
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = __builtin_amdgcn_rsq(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) h[i] = x[i] * y[i];
#pragma unroll
    for (int i = 0; i < N; ++i) e[i] = fma(-h[i], y[i], 1.0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        h[i] = y[i] * e[i];
        e[i] = fma(0.375, e[i], 0.5);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = fma(h[i], e[i], y[i]);
}

// 2^-x for 0 <= x <= 1/4: degree-8 interpolation at the Chebyshev points, relative
// error 1.3e-17
constexpr double kExpSmall = 0.25;
template <int N>
__device__ __forceinline__ void exp2small_n(double (&x)[N])
{
    constexpr double c[9] = {1.0, -0.6931471805599435, 0.24022650695891115, -0.05550410865702935,
                             0.009618128947059545, -0.0013333539542589711, 0.00015402262213827067,
                             -1.5202193099207678e-05, 1.2120929405791944e-06};
    double p[N];
#pragma unroll
    for (int i = 0; i < N; ++i) p[i] = c[8];
#pragma unroll
    for (int k = 7; k >= 0; --k)
#pragma unroll
        for (int i = 0; i < N; ++i) p[i] = fma(p[i], x[i], c[k]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = p[i];
}

}  // namespace pbm
