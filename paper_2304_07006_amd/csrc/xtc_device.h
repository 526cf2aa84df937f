// Device-side helpers shared by the xTC kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace xtc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int kPairTile = 128;   // pair-column padding unit (xtc_pair_ld)
constexpr int kGridPad = 128;    // grid-row padding unit of the prepared operands

// Jastrow parameters as kernels see them.  dcoef[k] = (k+1) coef[k], so the
// power-form derivative is a Horner polynomial in t = r/(1+r); entries beyond
// ncoef are zero, so all 16 terms are evaluated (leading zero terms leave the
// Horner value exactly unchanged) without a data-dependent loop.
struct JasDev {
    int32_t kind;    // 0 Pade, 1 power
    int32_t ncoef;
    double b;
    double dcoef[16];
    double d2coef[16];   // (k+2)(k+1) coef[k+1]: u''(t) as a Horner polynomial
    // the same parameters rounded to FP32 (reduced-precision forms; kernel
    // arguments, so they stay in scalar registers)
    float fb;
    float fdcoef[16];
    float fd2coef[16];
};

// 1/sqrt(x) and 1/x in FP64 from the hardware approximations (v_rsq_f64,
// v_rcp_f64, relative error e below 2^-22) and one third-order step each
// (1/sqrt(1-e) = 1 + e/2 + 3e^2/8 + O(e^3), 1/(1-e) = 1 + e + e^2 + O(e^3)),
// for x > 0 and finite: a few ulp, in fewer instructions than two Newton steps
// and than the correctly rounded sequences the compiler emits for sqrt and
// division.
__device__ __forceinline__ double rsq_f64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp_f64(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// scale u'(r)/r for the electron-electron Jastrow, from r^2 > 0.  For
// d^x = (x - x') u'(r)/r the caller adds kR2FloorF64 to r^2: the value stays
// finite at coincident points, where the difference vector it multiplies is
// exactly zero (the gradient of an isotropic function is taken as 0 there), and
// the floor is below the last bit of r^2 for every r above 1e-137.  `scale` is
// the reciprocal size of u' and multiplies it first: 1/r at the floor is 1e145,
// and scale / r by itself overflows for |u'| below 1e-157.
//   Pade : u = r/(2(1+br))      -> u'/r = 1 / (2 r (1+br)^2)
//   power: u = sum c_k t^k      -> u'/r = (sum k c_k t^(k-1)) / (r (1+r)^2)
constexpr double kR2FloorF64 = 1e-290;
template <int KIND>
__device__ __forceinline__ double du_over_r_nz_f64(double r2, const JasDev& J, double scale = 1.0) {
    const double s = rsq_f64(r2);                 // 1/r
    const double r = r2 * s;
    if constexpr (KIND == 0) {
        const double it = rcp_f64(fma(J.b, r, 1.0));
        return (0.5 * scale * s) * (it * it);
    } else {
        const double q = rcp_f64(1.0 + r);
        const double t = r * q;
        double p = J.dcoef[15];
#pragma unroll
        for (int k = 14; k >= 0; --k) p = fma(p, t, J.dcoef[k]);
        return ((p * scale) * s) * (q * q);
    }
}

// u'(r)/r for r^2 >= 0, exactly 0 at r^2 == 0, for any finite coefficients.
template <int KIND>
__device__ __forceinline__ double du_over_r_f64(double r2, const JasDev& J) {
    const double f = du_over_r_nz_f64<KIND>(r2, J);   // not finite at r2 == 0: selected away
    return r2 > 0.0 ? f : 0.0;
}

// Gradient epilogue of one Pi value: dL/dc_j gains j t^(j-1) q^2 / r times
// (r_g - r_g') . Pi(g,g') (power Jastrow, u' = sum_j j c_j t^(j-1) q^2 with
// t = r q, q = 1/(1+r)); FP64, nothing from coincident points.  gsum[j - 1]
// collects the terms without their factor j (pi_grad_factors).  Half of
// the epilogue's instructions were the correctly rounded square root and two
// divisions.
__device__ __forceinline__ void pi_grad_point(const d4& pi, const d4& pj, double px, double py, double pz,
                                              double (&gsum)[16]) {
    const double dx = pi.x - pj.x, dy = pi.y - pj.y, dz = pi.z - pj.z;
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    if (!(r2 > 0.0)) return;
    const double s = rsq_f64(r2);                 // 1/r
    const double r = r2 * s;
    const double q = rcp_f64(1.0 + r);
    const double t = r * q;
    double tp = fma(dx, px, fma(dy, py, dz * pz)) * (q * q) * s;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        gsum[j] += tp;
        tp *= t;
    }
}
__device__ __forceinline__ void pi_grad_factors(double (&gsum)[16]) {
#pragma unroll
    for (int j = 0; j < 16; ++j) gsum[j] *= (double)(j + 1);
}

__device__ __forceinline__ int pair_index(int p, int q, int N) {
    // p <= q
    return p * N - (p * (p - 1)) / 2 + (q - p);
}

__device__ __forceinline__ int pair_sym(int p, int q, int N) {
    return p <= q ? pair_index(p, q, N) : pair_index(q, p, N);
}

// The pair (p, q), p <= q < N, of packed index P: pair_index inverted, from the
// root of its quadratic in FP32 (exact integers below 2^24), corrected.
__device__ __forceinline__ void pair_split(int P, int N, int& p, int& q) {
    const float b = 2.0f * N + 1.0f;
    p = min(max((int)(0.5f * (b - sqrtf(fmaxf(b * b - 8.0f * P, 0.0f)))), 0), N - 1);
    while (p > 0 && pair_index(p, p, N) > P) --p;
    while (p + 1 < N && pair_index(p + 1, p + 1, N) <= P) ++p;
    q = p + P - pair_index(p, p, N);
}

}  // namespace xtc
