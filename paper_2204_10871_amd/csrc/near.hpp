// Terms of nearby lenses, shared by the level-3 ray kernels (k_interp.hip,
// k_learn.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace irs {

// Term of one nearby lens for a ray at (t1, t2): m (d1, d2)/(d1^2 + d2^2),
// d = theta - z, with d1 and d1s = d1^2 + kNearTiny taken once per lens for
// all rays of a column.  The quotient m/rr is the hardware reciprocal
// estimate v times m, corrected once (w = y + v (m - rr y)), which squares
// the estimate's relative error.  kNearTiny (far below the square of any
// lens-ray distance that occurs) keeps rr > 0 where a lens sits exactly on
// a ray, whose term is then exactly 0 because d = 0; it changes no other rr.
constexpr double kNearTiny = 1e-300;
// Largest level-1 cell side a plan may have: every nearby lens then lies
// within 3 sqrt(2) kMaxCell of a ray, so rr < 1e49 and a product of four
// rr stays below kGroupMax.
constexpr double kMaxCell = 1e24;

__device__ __forceinline__ void near_term(double d1, double d1s, double t2, double zy, double m,
                                          double &n1, double &n2)
{
    const double d2 = t2 - zy;
    const double rr = fma(d2, d2, d1s);
    const double v = __builtin_amdgcn_rcp(rr);
    const double y = m * v;
    const double w = fma(v, fma(-rr, y, m), y);
    n1 = fma(w, d1, n1);
    n2 = fma(w, d2, n2);
}

// The same for G rays of one column (rows t2s[0..G-1]): the G quotients
// m/rr_k come from one reciprocal of their product p = rr_0 ... rr_{G-1},
// corrected once as above (q = m/p), then back-substitution through the
// prefix products P_k = rr_0 ... rr_k: m/rr_k = q P_{k-1} for k = G-1 down to
// 1, q taking q rr_k = m/P_{k-1} after each step, and m/rr_0 = the last q.
// Each quotient carries at most about 2G + 4 units of rounding.  Where p lies
// at or below 1e-200 (a lens on or extremely close to a ray) the quotients are
// taken one by one, with kNearTiny added to each rr.  Cells no wider than
// kMaxCell keep p below 1e200, far from overflow, so p needs no upper test.
constexpr double kGroupMin = 1e-200;
// rows of a lane that share one reciprocal per lens: four keeps the group's
// products in few enough registers for five waves per SIMD
constexpr int kNearGroup = 4;

template <int G>
__device__ __forceinline__ void near_group_d2(double d1, double d1s, const double *d2, double m,
                                              double *n1s, double *n2s)
{
    // d1s = d1^2 here (no kNearTiny: that is added on the one-by-one path)
    double rr[G], pre[G], w[G];
#pragma unroll
    for (int k = 0; k < G; ++k) rr[k] = fma(d2[k], d2[k], d1s);
    pre[0] = rr[0];
#pragma unroll
    for (int k = 1; k < G; ++k) pre[k] = pre[k - 1] * rr[k];
    const double p = pre[G - 1];
    if (__builtin_expect(p > kGroupMin, 1)) {
        const double v = __builtin_amdgcn_rcp(p);
        const double y = m * v;
        double q = fma(v, fma(-p, y, m), y);          // m / p
#pragma unroll
        for (int k = G - 1; k >= 1; --k) {
            w[k] = q * pre[k - 1];
            q = q * rr[k];                            // m / P_{k-1}
        }
        w[0] = q;
    } else {
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const double r = rr[k] + kNearTiny;
            const double v = __builtin_amdgcn_rcp(r);
            const double y = m * v;
            w[k] = fma(v, fma(-r, y, m), y);
        }
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
        n1s[k] = fma(w[k], d1, n1s[k]);
        n2s[k] = fma(w[k], d2[k], n2s[k]);
    }
}

template <int G>
__device__ __forceinline__ void near_group(double d1, double d1s, const double *t2s, double zy,
                                           double m, double *n1s, double *n2s)
{
    double d2[G];
#pragma unroll
    for (int k = 0; k < G; ++k) d2[k] = t2s[k] - zy;
    near_group_d2<G>(d1, d1s, d2, m, n1s, n2s);
}

}  // namespace irs
