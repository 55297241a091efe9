// Direct ray shooting: every ray sums every lens (Eq. 6), then the macro term
// and the negative sheet (the rectangle's closed forms of Appendix A, or
// -kappa_* theta on a circular lens plane, Eq. 9), the mapping
// beta = theta - alpha (Eq. 4) and the source-pixel binning.  This is the
// ordinary IRS the paper compares against (Sec. 3.1), whose cost grows as
// N_rays * N_* (Eq. 12).
//
// Two kernels:
//   k_direct_f64  -- plain double precision, lens tiles in LDS: one ray per lane
//                    or, in plans of many rays (k_direct_f64_blocks), blocks of
//                    256 columns of a ray row, four rays per lane.
//   k_direct_f32  -- the FP32 VALU-bound form: each wave owns 64 columns of up
//                    to eight ray rows (four or sixteen in the other shapes);
//                    ray-lens offsets are rounded to FP32 once from their FP64
//                    values (d1 per column and lens, d2 per row and lens
//                    through LDS), the lane's rays share every d1, and each
//                    ray's sum is compensated: 32 lenses are summed plainly,
//                    then added with Kahan's correction.  The lenses
//                    of the 3 x 3 level-1 cells around the ray are then
//                    re-evaluated in FP64 and the difference to their FP32
//                    terms is added (FP32 quantisation of a lens at distance d
//                    errs by ~1e-7/d^2, which only matters close by).  The
//                    macro term, the sheet and beta are assembled in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "plan.hpp"

namespace irs {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;

// -------------------------------------------------------------------------
// Epilogue shared by both kernels: macro term + sheet + beta + pixel.
// -------------------------------------------------------------------------
// have: I1, I2 are the rectangle's sheet integrals.
__device__ __forceinline__ void assemble(const DevGeom &g, double t1, double t2, double s1,
                                         double s2, double &a1, double &a2, int32_t &pix,
                                         bool have = false, double I1 = 0.0, double I2 = 0.0)
{
    double h1 = 0.0, h2 = 0.0;
    if (g.sheet == 2) {                      // circular plane: -kappa_* theta (Eq. 9)
        h1 = -g.kappa_star * t1;
        h2 = -g.kappa_star * t2;
    } else if (g.sheet) {
        if (!have) sheet_unit(g, t1, t2, I1, I2);
        const double f = -g.kappa_star / M_PI;
        h1 = f * I1;
        h2 = f * I2;
    }
    a1 = g.kpg * t1 + s1 + h1;
    a2 = g.kmg * t2 + s2 + h2;
    pix = pixel_of(g, t1 - a1, t2 - a2);
}

// Per-ray output or binning, called by every lane: the wave's lanes hold rays in
// order, so runs of equal pixels are added once each (a pass over the wave's
// distinct pixels instead, up to 64 of them: 311 against 303 us for 2048^2 FP64
// rays, 1026 against 1010 for 1e6 FP32 rays of 4450 lenses).
__device__ __forceinline__ void emit(bool valid, int64_t out_idx, double a1, double a2,
                                     int32_t pix, double *a1o, double *a2o, int64_t *pixo,
                                     uint32_t *counts, unsigned long long *landed)
{
    if (counts) {
        const int32_t pv = valid ? pix : -1;
        bin_runs(counts, pv);
        const uint64_t got = __ballot(pv >= 0);
        if (__lane_id() == 0 && got) landed_add(landed, (unsigned long long)__popcll(got));
    } else if (valid) {
        if (a1o) a1o[out_idx] = a1;
        if (a2o) a2o[out_idx] = a2;
        if (pixo) pixo[out_idx] = pix;
    }
}

// -------------------------------------------------------------------------
// FP64
// -------------------------------------------------------------------------
constexpr int kLens64 = 256;
constexpr int kBlock = 4 * kWave;               // columns of a block (k_direct_f64_blocks)

// Below this |theta_2 - y_i| a term takes the IEEE division: r^2 may be 0,
// subnormal or too small for the refined reciprocals (a product of two r^2
// has to stay a normal number).
constexpr double kNear64 = 1e-35;

// One lens's term for one ray, any r^2 (0 on the ray).
__device__ __forceinline__ void term_any(double d1, double r2, double d2, double m, double &s1,
                                         double &s2)
{
    if (r2 > 0.0) {
        const double w = m / r2;
        s1 += w * d1;
        s2 += w * d2;
    }
}

// m / r2, r2 and m (or m = 0) far from the ends of the exponent range: the
// hardware estimate (2^-24) after one Newton step is within 2^-48 of 1/r2, and
// the quotient corrected once with its exact remainder is the rounded
// quotient, as the IEEE division's (which adds scaling and fix-up for the
// ends of the range): before its rounding it is within 2^-94, so the two
// differ for about one quotient in 2^41.
template <bool UNIT>
__device__ __forceinline__ double quotient(double m, double r2)
{
    double v = __builtin_amdgcn_rcp(r2);
    v = fma(v, fma(-r2, v, 1.0), v);
    const double q = UNIT ? v : m * v;
    return fma(v, fma(-r2, q, m), q);
}

// m / r2[k] for two r2: both estimates come from one reciprocal of their product
// (refined once, 2^-48); each is then corrected with its own remainder as in
// quotient(), so the quotients are rounded alike.  Groups of two, so that a wave
// of two rays a lane has them whole: four r2 a reciprocal take half a slot less a
// quotient and give 2048^2 rays and 105 lenses no less time (261 us against 260),
// but calls of 1e5 rays and 1e4 lenses 2.5 ms instead of 1.1.
template <bool UNIT>
__device__ __forceinline__ void quotient2(double m, const double *r2, double *w)
{
    const double p = r2[0] * r2[1];
    double v = __builtin_amdgcn_rcp(p);
    v = fma(v, fma(-p, v, 1.0), v);
    const double e[2] = {v * r2[1], v * r2[0]};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double q = UNIT ? e[k] : m * e[k];
        w[k] = fma(e[k], fma(-r2[k], q, m), q);
    }
}

// Lenses of a map staged in LDS, kLens64 at a time, by the whole workgroup.
template <bool UNIT>
struct Stage64 {
    double2 xy[kLens64];
    double m[UNIT ? 1 : kLens64];
};

// One lens for a lane's R rays of one row at d2 = theta_2 - y, |d2| >= kNear64;
// rays 2 h and 2 h + 1 share a reciprocal.
template <bool UNIT, int R>
__device__ __forceinline__ void row_lens_far(double x, double d2, double m, const double *t1,
                                             double *s1, double *s2)
{
    const double q2 = d2 * d2;
    double d1[R], r2[R], w[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        d1[k] = t1[k] - x;
        r2[k] = fma(d1[k], d1[k], q2);
    }
    if constexpr (R == 1) w[0] = quotient<UNIT>(m, r2[0]);
    else
#pragma unroll
        for (int k = 0; k < R; k += 2) quotient2<UNIT>(m, r2 + k, w + k);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        s1[k] = fma(w[k], d1[k], s1[k]);
        s2[k] = fma(w[k], d2, s2[k]);
    }
}

// The same for a staged lens at any distance from the row.
template <bool UNIT, int R>
__device__ __forceinline__ void row_lens(const Stage64<UNIT> &sm, int t, const double *t1,
                                         double t2, double *s1, double *s2)
{
    const double2 z = sm.xy[t];
    const double m = UNIT ? 1.0 : sm.m[t];
    const double d2 = t2 - z.y;
    if (fabs(d2) < kNear64) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const double d1 = t1[k] - z.x;
            term_any(d1, fma(d1, d1, d2 * d2), d2, m, s1[k], s2[k]);
        }
    } else {
        row_lens_far<UNIT, R>(z.x, d2, m, t1, s1, s2);
    }
}

// The staged lenses for a lane's R rays (1, or pairs) of the row t2, where the
// plan is tame (irs_plan_s::tame: lenses and masses allow quotient()):
// theta_2 - y_i and its square are taken once for the R rays.  Four lenses a step,
// against two: 1,000 to 65,000 rays and 1e4 lenses 750 against 1,020 us.
template <bool UNIT, int R>
__device__ __forceinline__ void row_lenses(const Stage64<UNIT> &sm, int cnt, const double *t1,
                                           double t2, double *s1, double *s2)
{
    constexpr int S = 4;
    int t = 0;
    for (; t + S <= cnt; t += S) {
        double2 z[S];
        double d[S], m[S], least = INFINITY;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            z[u] = sm.xy[t + u];
            m[u] = UNIT ? 1.0 : sm.m[t + u];
            d[u] = t2 - z[u].y;
            least = fmin(least, fabs(d[u]));
        }
        if (__builtin_expect(least < kNear64, 0)) {
#pragma unroll 1
            for (int u = 0; u < S; ++u) row_lens<UNIT, R>(sm, t + u, t1, t2, s1, s2);
        } else {
#pragma unroll
            for (int u = 0; u < S; ++u) row_lens_far<UNIT, R>(z[u].x, d[u], m[u], t1, s1, s2);
        }
    }
    for (; t < cnt; ++t) row_lens<UNIT, R>(sm, t, t1, t2, s1, s2);
}

// The staged lenses for the first n of a lane's R rays of the row t2, by the
// division: plans that are not tame.
template <bool UNIT, int R>
__device__ __forceinline__ void wild_lenses(const Stage64<UNIT> &sm, int cnt, int n,
                                            const double *t1, double t2, double *s1, double *s2)
{
    for (int t = 0; t < cnt; ++t) {
        const double2 z = sm.xy[t];
        const double m = UNIT ? 1.0 : sm.m[t];
        const double d2 = t2 - z.y;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (k >= n) break;
            const double d1 = t1[k] - z.x;
            term_any(d1, fma(d1, d1, d2 * d2), d2, m, s1[k], s2[k]);
        }
    }
}

// Every lens in packed order, kLens64 at a time through LDS: take(cnt) after
// each stage.  Called by the whole workgroup.
template <bool UNIT, class F>
__device__ __forceinline__ void lens_stages(Stage64<UNIT> &sm, const double *__restrict__ lx,
                                            const double *__restrict__ ly,
                                            const double *__restrict__ lm, int32_t nl, F take)
{
    const int tid = threadIdx.x;
    for (int32_t base = 0; base < nl; base += kLens64) {
        __syncthreads();
        if (base + tid < nl) {
            sm.xy[tid] = make_double2(lx[base + tid], ly[base + tid]);
            if (!UNIT) sm.m[tid] = lm[base + tid];
        }
        __syncthreads();
        take(min(kLens64, nl - base));
    }
}

// The rectangle's sheet integrals along a ray row, as a series about a point
// (x0, y) of it (T_0 in two parts, the larger at T[kSheetTerms]): with
// w = z - corner, S = I2 + i I1 has d^2 S/dx^2 = sum +-1/w and
// dS/dx = sum +-(ln|w| + i atan(v/u)) (signs and terms of sheet_unit), so
//     S(x0 + s d) = sum_n T_n d^n,   T_n = -s/(n (n-1)) sum +-(-s/w)^(n-1), n >= 2.
// Lane = 16 corner + m takes its corner's terms and the powers m, m + 16, m + 32.
// Returns the number of terms that leave less than 2^-57 of s (4 s rho^n with
// rho = s/(distance to the nearest corner)), 0 for rho > 0.4.  Called by whole
// waves; x0, y, s wave-uniform; T: the wave's LDS.
//
// The closed form (four logarithms and arctangents) is 560 of the 1940 VALU
// instructions of a ray in a map of 105 lenses; the series is about 150 where a
// wave takes a block of 256 rays.  2048^2 rays, 105 lenses: 303 -> 263 us.  The
// closed form's rounding (corner terms of 100 and more that cancel) is most of a
// deflection's error; T_0 carries its roundings along, so the error against 64
// more bits falls: mean 2.4e-14 -> 1.0e-14 (1.2e6 rays, 915 lenses).
constexpr int kSheetTerms = 48;

__device__ __forceinline__ double over_corners(double v)
{
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// a + b and what its rounding lost, added to lo
__device__ __forceinline__ double sum_err(double a, double b, double &lo)
{
    const double s = a + b, t = s - a;
    lo += (a - (s - t)) + (b - t);
    return s;
}

// (hi, lo) += a * b
__device__ __forceinline__ void add_product(double a, double b, double &hi, double &lo)
{
    const double p = a * b;
    lo += fma(a, b, -p);
    hi = sum_err(hi, p, lo);
}

// the corners' (hi, lo) summed
__device__ __forceinline__ void over_corners2(double &hi, double &lo)
{
#pragma unroll
    for (int b = 16; b <= 32; b *= 2) {
        const double h = __shfl_xor(hi, b), l = __shfl_xor(lo, b);
        lo += l;
        hi = sum_err(hi, h, lo);
    }
}

__device__ __forceinline__ int sheet_row_series(const DevGeom &g, double x0, double y, double s,
                                                double2 *T)
{
    const int lane = threadIdx.x % kWave, c = lane / 16, m = lane % 16;
    const double ca = (c == 0 || c == 3) ? g.a1 : g.a2, cb = c < 2 ? g.b1 : g.b2;
    const double sgn = (c == 0 || c == 2) ? 1.0 : -1.0;
    double ul = 0.0, vl = 0.0;
    const double u = sum_err(x0, -ca, ul), v = sum_err(y, -cb, vl);
    const double r2 = u * u + v * v, inv = 1.0 / r2;
    double rho2 = s * s * inv, big = r2;
    rho2 = fmax(rho2, __shfl_xor(rho2, 16));
    rho2 = fmax(rho2, __shfl_xor(rho2, 32));
    if (!(rho2 <= 0.16)) return 0;
    big = fmax(big, __shfl_xor(big, 16));
    big = fmax(big, __shfl_xor(big, 32));
    // T_0 and T_1 with what their roundings lose: the logarithms scaled by a
    // power of two (the same in all corners, which leaves the sums unchanged)
    const double l = 0.5 * sgn * log(ldexp(r2, -__builtin_amdgcn_frexp_exp(big)));
    const bool steep = fabs(u) < fabs(v);
    const double q = steep ? u / v : v / u, t = atan(q);
    double ol = copysign(kHalfPiLo, q);
    const double o = sum_err(copysign(M_PI_2, q), -t, ol);            // pi/2 - t
    const double tu = sgn * (steep ? o : t), tv = sgn * (steep ? t : o);    // atan(v/u), atan(u/v)
    double h1 = v * l, e1 = fma(v, l, -h1), h2 = u * l, e2 = fma(u, l, -h2);
    add_product(u, tu, h1, e1);
    add_product(v, tv, h2, e2);
    e1 += ul * tu + vl * (l + sgn) + (steep ? sgn * u * ol : 0.0);
    e2 += vl * tv + ul * (l + sgn) + (steep ? 0.0 : sgn * v * ol);
    over_corners2(h1, e1);
    over_corners2(h2, e2);
    const double g1 = over_corners(tu), g2 = over_corners(l);
    // (-s/w)^m, then steps of 16
    double qr = -s * u * inv, qi = s * v * inv, er = sgn, ei = 0.0;
#pragma unroll
    for (int b = 1; b < 16; b <<= 1) {
        const double tr = er * qr - ei * qi, ti = er * qi + ei * qr;
        er = (m & b) ? tr : er;
        ei = (m & b) ? ti : ei;
        const double sr = qr * qr - qi * qi;
        qi = 2.0 * qr * qi;
        qr = sr;
    }
#pragma unroll
    for (int h = 0; h < kSheetTerms / 16; ++h) {
        const int n = 16 * h + m + 1;
        const double sr = over_corners(er), si = over_corners(ei);
        const double f = -s / ((double)n * (double)(n - 1));
        double2 t = n == 1 ? make_double2(s * g2, s * g1) : make_double2(f * sr, f * si);
        if (c == 0 && n < kSheetTerms) T[n] = t;
        if (lane == 0 && h == 0) {
            T[0] = make_double2(e2, e1);
            T[kSheetTerms] = make_double2(h2, h1);
        }
        const double tr = er * qr - ei * qi;
        ei = er * qi + ei * qr;
        er = tr;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const float bits = -0.5f * __log2f((float)rho2);        // of one more term; >= 1.32
    return __builtin_amdgcn_readfirstlane(min(kSheetTerms, 2 + (int)ceilf(59.0f / fmaxf(bits, 1.0f))));
}

// The lens sums of a lane's ray (t1, t2), every lens in packed order; two lenses a
// step, whose chains overlap, where the wave's rays lie in one row.
template <bool UNIT>
__device__ __forceinline__ void lens_sums(Stage64<UNIT> &sm, const double *__restrict__ lx,
                                          const double *__restrict__ ly,
                                          const double *__restrict__ lm, int32_t nl, bool tame,
                                          const double *t1, const double *t2, bool one_row,
                                          double *s1, double *s2)
{
    const int tid = threadIdx.x;
    s1[0] = s2[0] = 0.0;
    for (int32_t base = 0; base < nl; base += kLens64) {
        __syncthreads();
        if (base + tid < nl) {
            sm.xy[tid] = make_double2(lx[base + tid], ly[base + tid]);
            if (!UNIT) sm.m[tid] = lm[base + tid];
        }
        __syncthreads();
        const int cnt = min(kLens64, nl - base);
        if (tame && one_row) {                               // wave-uniform
            int t = 0;
            for (; t + 1 < cnt; t += 2) {
                const double2 za = sm.xy[t], zb = sm.xy[t + 1];
                const double da = t2[0] - za.y, db = t2[0] - zb.y;
                if (__builtin_expect(fmin(fabs(da), fabs(db)) < kNear64, 0)) {
                    row_lens<UNIT, 1>(sm, t, t1, t2[0], s1, s2);
                    row_lens<UNIT, 1>(sm, t + 1, t1, t2[0], s1, s2);
                } else {
                    row_lens_far<UNIT, 1>(za.x, da, UNIT ? 1.0 : sm.m[t], t1, s1, s2);
                    row_lens_far<UNIT, 1>(zb.x, db, UNIT ? 1.0 : sm.m[t + 1], t1, s1, s2);
                }
            }
            if (t < cnt) row_lens<UNIT, 1>(sm, t, t1, t2[0], s1, s2);
        } else {
            for (int t = 0; t < cnt; ++t) {
                const double2 z = sm.xy[t];
                const double m = UNIT ? 1.0 : sm.m[t];
                const double d1 = t1[0] - z.x, d2 = t2[0] - z.y;
                const double r2 = fma(d1, d1, d2 * d2);
                if (__builtin_expect(tame && fabs(d2) >= kNear64, 1)) {
                    const double w = quotient<UNIT>(m, r2);
                    s1[0] = fma(w, d1, s1[0]);
                    s2[0] = fma(w, d2, s2[0]);
                } else {
                    term_any(d1, r2, d2, m, s1[0], s2[0]);
                }
            }
        }
    }
}

// One ray a lane, a workgroup's rays consecutive ones.  A ray's sums do not depend
// on which rays share its wave.  (Arrays of one ray: with scalars the compiler
// takes 74 registers instead of 65, six waves a SIMD instead of seven.)
template <bool UNIT>
__global__ __launch_bounds__(kThreads) void k_direct_f64(
    DevGeom g, const double *__restrict__ lx, const double *__restrict__ ly,
    const double *__restrict__ lm, int32_t nl, bool tame, int64_t r_begin, int64_t r_end,
    int64_t out_base, double *a1o, double *a2o, int64_t *pixo, uint32_t *counts,
    unsigned long long *landed)
{
    __shared__ Stage64<UNIT> sm;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t w0 = r_begin + ((int64_t)blockIdx.x * kWaves + wave) * kWave;
    double t1[1], t2[1], s1[1], s2[1];
    // the wave's first ray's row; most waves stay in it
    const int64_t j0 = w0 / g.nx, i0 = w0 - j0 * g.nx;
    const bool one_row = i0 + kWave <= g.nx;
#pragma unroll
    for (int k = 0; k < 1; ++k) {
        int64_t i = i0 + lane + kWave * k, j = j0;
        if (!one_row) {
            const int64_t r = min(w0 + lane + kWave * k, r_end - 1);
            j = r / g.nx;
            i = r - j * g.nx;
        }
        t1[k] = ray_x(g, i);
        t2[k] = ray_y(g, j);
    }
    lens_sums<UNIT>(sm, lx, ly, lm, nl, tame, t1, t2, one_row, s1, s2);
#pragma unroll
    for (int k = 0; k < 1; ++k) {
        const int64_t r = w0 + lane + kWave * k;
        double a1, a2;
        int32_t pix;
        assemble(g, t1[k], t2[k], s1[k], s2[k], a1, a2, pix);
        emit(r < r_end, r - out_base, a1, a2, pix, a1o, a2o, pixo, counts, landed);
    }
}

// Blocks: the kBlock columns from a multiple of kBlock of one ray row, in four
// groups of 64 (lane: columns lane + 64 k).  Rays of groups 0 and 1, and of 2 and
// 3, share a reciprocal where both groups hold columns of the grid, the others
// take their own, and all take the sheet as the series about the middle of the
// block's columns where sheet_row_series allows it, else in closed form.  Which of
// these a ray takes, and its partner, depend on the plan and the ray alone, so
// that maps, bands of rows, ranges of deflections and batches agree bit for bit
// (a call of a few rays pays 1 us for the series: 4 rays, 75 lenses 21.6 us
// against 20.7 with the closed form).
//
// A wave takes R of a block's groups: all four, or, for calls of few blocks
// (kFewBlocks), two.  Bound by FP64 issue: with four rays a lane, per ray and lens
// about 2.5 slots (a slot: one FMA) of offsets and r^2, 6.2 of the quotient and 2 of
// the sums, against about 24 with the IEEE division and one ray a lane.  2048^2
// rays, 105 lenses, whole call: 425 us with one ray a lane, the division and the
// sheet in closed form, 260 now; 275 with waves of 256 consecutive rays, of which
// those that pass a row's end do without the series and the shared distances.
struct BlockLds {
    double2 T[kWaves][kSheetTerms + 1];
};

// unit: the wave's, of those [.., u1) counted along the rows, 4/R a block; of its
// rays those in [r_begin, r_end) are put out
template <bool UNIT, int R>
__device__ __forceinline__ void direct_block(Stage64<UNIT> &sm, BlockLds &bl, const DevGeom &g,
                                             const double *__restrict__ lx,
                                             const double *__restrict__ ly,
                                             const double *__restrict__ lm, int32_t nl, bool tame,
                                             int64_t unit, int64_t u1, int64_t r_begin,
                                             int64_t r_end, int64_t out_base, double *a1o,
                                             double *a2o, int64_t *pixo, uint32_t *counts,
                                             unsigned long long *landed)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t blk = unit / (4 / R), nb = (g.nx + kBlock - 1) / kBlock;
    const int64_t j = blk / nb, b0 = (blk - j * nb) * kBlock;
    const int64_t c0 = b0 + unit % (4 / R) * (kWave * R);  // the wave's first column
    // the wave's groups that hold columns; wave-uniform (every wave meets the barriers)
    const int n = unit < u1 ? (int)max<int64_t>(0, min<int64_t>(R, (g.nx - c0 + kWave - 1) / kWave)) : 0;
    const double t2 = ray_y(g, j);
    double t1[R], s1[R], s2[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        t1[k] = ray_x(g, c0 + kWave * k + lane);
        s1[k] = s2[k] = 0.0;
    }
    lens_stages<UNIT>(sm, lx, ly, lm, nl, [&](int cnt) {
        if (!tame) {
            wild_lenses<UNIT, R>(sm, cnt, n, t1, t2, s1, s2);
        } else if (n == R) {
            row_lenses<UNIT, R>(sm, cnt, t1, t2, s1, s2);
        } else {
            if (R > 2 && n >= 2) row_lenses<UNIT, 2>(sm, cnt, t1, t2, s1, s2);
            if (n == 1) row_lenses<UNIT, 1>(sm, cnt, t1, t2, s1, s2);
            if (R > 2 && n == 3) row_lenses<UNIT, 1>(sm, cnt, t1 + R - 2, t2, s1 + R - 2, s2 + R - 2);
        }
    });
    if (n == 0) return;
    double I1[R] = {}, I2[R] = {};
    int terms = 0;                                         // wave-uniform
    if (g.sheet == 1) {
        // about the middle of the block's columns of the grid: past the rectangle's
        // edge the arctangents jump
        const int64_t half = min<int64_t>(kBlock, g.nx - b0) / 2;
        const double x0 = ray_x(g, b0 + half), s = (double)max<int64_t>(1, half) * g.ray_dx;
        double2 *T = bl.T[wave];
        terms = sheet_row_series(g, x0, t2, s, T);
        if (terms) {
            const double is = 1.0 / s;
            double d[R];
#pragma unroll
            for (int k = 0; k < R; ++k) d[k] = (t1[k] - x0) * is;
            for (int m = terms - 1; m >= 0; --m) {
                const double2 t = T[m];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    I1[k] = fma(I1[k], d[k], t.y);
                    I2[k] = fma(I2[k], d[k], t.x);
                }
            }
            const double2 t = T[kSheetTerms];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                I1[k] += t.y;
                I2[k] += t.x;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t c = c0 + kWave * k + lane, r = j * g.nx + c;
        double a1, a2;
        int32_t pix;
        assemble(g, t1[k], t2, s1[k], s2[k], a1, a2, pix, terms > 0, I1[k], I2[k]);
        emit(c < g.nx && r >= r_begin && r < r_end, r - out_base, a1, a2, pix, a1o, a2o, pixo,
             counts, landed);
    }
}

template <bool UNIT, int R>
__global__ __launch_bounds__(kThreads) void k_direct_f64_blocks(
    DevGeom g, const double *__restrict__ lx, const double *__restrict__ ly,
    const double *__restrict__ lm, int32_t nl, bool tame, int64_t u0, int64_t u1, int64_t r_begin,
    int64_t r_end, int64_t out_base, double *a1o, double *a2o, int64_t *pixo, uint32_t *counts,
    unsigned long long *landed)
{
    __shared__ Stage64<UNIT> sm;
    __shared__ BlockLds bl;
    const int64_t unit = u0 + (int64_t)blockIdx.x * kWaves +
                         __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    direct_block<UNIT, R>(sm, bl, g, lx, ly, lm, nl, tame, unit, u1, r_begin, r_end, out_base, a1o,
                          a2o, pixo, counts, landed);
}

// Persistent FP64 form for batches: item = four blocks, or 256 consecutive rays, of
// a map (direct_items).
template <bool UNIT>
__global__ __launch_bounds__(kThreads, 4) void k_direct_f64_queue(
    const DirectArgs *__restrict__ maps, const int64_t *__restrict__ item_start, int32_t nmaps,
    unsigned long long *cursor)
{
    __shared__ Stage64<UNIT> sm;
    __shared__ BlockLds bl;
    __shared__ long long s_item;
    const int tid = threadIdx.x;
    const int64_t total = item_start[nmaps];
    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = (long long)atomicAdd(cursor, 1ull);
        __syncthreads();
        const int64_t item = s_item;
        if (item >= total) break;                    // every workgroup reaches this
        int lo = 0, hi = nmaps - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (item_start[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        const DirectArgs &a = maps[lo];
        const int64_t n = item - item_start[lo];
        if (a.blocks) {
            direct_block<UNIT, 4>(sm, bl, a.g, a.lx, a.ly, a.lm, a.nl, a.tame != 0,
                                  n * kWaves + __builtin_amdgcn_readfirstlane(tid / kWave),
                                  a.blocks, a.ray_first, a.ray_last, 0, nullptr, nullptr,
                                  nullptr, a.counts, a.landed);
        } else {
            const DevGeom &g = a.g;
            const int64_t r = n * kThreads + tid;
            const bool valid = r < a.ray_last;
            const int64_t rr = valid ? r : 0;
            const double t1 = ray_x(g, rr % g.nx), t2 = ray_y(g, rr / g.nx);
            double s1, s2;
            lens_sums<UNIT>(sm, a.lx, a.ly, a.lm, a.nl, a.tame != 0, &t1, &t2, false, &s1, &s2);
            double a1, a2;
            int32_t pix;
            assemble(g, t1, t2, s1, s2, a1, a2, pix);
            emit(valid, 0, a1, a2, pix, nullptr, nullptr, nullptr, a.counts, a.landed);
        }
    }
}

// Blocks of the whole map, for plans of 2^20 rays and more in rows of more than 192
// rays; 0: one ray a lane.  A property of the plan, so that every call on it and
// every batch with it takes a ray in one way.  With fewer rays four a lane
// would be under four waves a SIMD, and a row of 193 rays is the shortest that
// fills four groups: blocks then leave at most a third of their lanes idle.
int64_t direct_blocks(const irs_plan_s *p)
{
    const DevGeom &g = p->dg;
    if (p->params.precision != IRS_FP64 || g.nx <= 3 * kWave || g.nx * g.ny < ((int64_t)1 << 20))
        return 0;
    return (g.nx + kBlock - 1) / kBlock * g.ny;
}

// Calls of at most this many blocks (four waves a SIMD) take two of a block's groups
// a wave: 4e5 rays (1,600 blocks) and 1e4 lenses 2.05 against 2.21 ms, 1.3e6 rays of a
// map of 262 rows (5,240) 1137 lenses 643 against 688 us, but 4e6 rays (16,800),
// 105 lenses 275 against 260.
constexpr int64_t kFewBlocks = 4096;

// -------------------------------------------------------------------------
// FP32 with compensation
//
// Offsets are formed in FP64 and rounded to FP32 once: d1 = RN(theta1 - x_i)
// per (column, lens), shared by the lane's 8 rays; d2 = RN(theta2 - y_i) per
// (row, lens), computed once per workgroup into LDS and read by all 64
// columns as broadcasts.  A single rounding of the exact offset is unbiased;
// a tile-local frame (d1 = RN(xr - RN(x_i - o))) is not: its second rounding
// carries the ray's offset identically into every lens of a binade, which
// adds up coherently over 1e6 lenses.
// -------------------------------------------------------------------------
constexpr int kTX = kWave;            // ray columns per tile: one per lane
constexpr int kChunk = 32;            // lenses per uncompensated partial sum
constexpr float kTiny = 1e-30f;       // keeps 1/r^2 finite for a lens on a ray

// 1/r^2 from d1^2 (+ kTiny, precomputed) and d2: hardware reciprocal refined
// by one Newton step, so the result is correctly rounded and unbiased.  A
// lens on the ray gives r^2 = kTiny and a zero term (its offsets are 0).
__device__ __forceinline__ float inv_r2(float d1sq, float d2)
{
    const float r2 = fmaf(d2, d2, d1sq);
    const float v = __builtin_amdgcn_rcpf(r2);
    const float e = fmaf(-r2, v, 1.0f);
    return fmaf(v, e, v);
}

__device__ __forceinline__ void kahan_add(float &s, float &c, float x)
{
    const float y = x - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

}  // namespace

// The FP32 tile, bound by its arithmetic (five FMAs and a reciprocal per ray and
// lens, 29 cycles a wave; 4e6 rays and 1e5 lenses: 74.7 ms, 74.3 by that count
// at 2.4 GHz).  A wave takes up to RPT ray rows of 64 columns, a workgroup's
// four waves share stages of LT lenses in LDS.  Every shape and every number of
// rows computes each ray with the same operations in the same order (LT is a
// multiple of kChunk), so all of them give identical bits.
template <bool UNIT, int RPT, int LT>
struct DirectTile {
    static constexpr int TY = RPT * kWaves;
    // row counts the lens loop is compiled for: 1 to RPT, in steps for RPT > 8
    static constexpr int STEP = RPT > 8 ? RPT / 8 : 1;
    struct Smem {
        double X[LT], Y[LT];
        float4 m4[UNIT ? 1 : LT / 4];
        float4 d24[TY][LT / 4];          // d2 per (row, lens), each wave its own RPT rows
    };
    struct Acc {
        float in1[RPT], in2[RPT], s1[RPT], c1[RPT], s2[RPT], c2[RPT];
    };

    // one stage's lenses into R rows
    template <int R>
    __device__ __forceinline__ static void stage(const Smem &sm, const float4 (*d24)[LT / 4],
                                                 double t1, int cnt, Acc &A)
    {
        const float *s_m = reinterpret_cast<const float *>(sm.m4);
        const int full = cnt - cnt % kChunk;
        for (int c = 0; c < full; c += kChunk) {
#pragma unroll 2
            for (int t = 0; t < kChunk; t += 4) {
                float d1[4], d1sq[4], ms[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    d1[u] = (float)(t1 - sm.X[c + t + u]);
                    d1sq[u] = fmaf(d1[u], d1[u], kTiny);
                    ms[u] = UNIT ? 1.0f : s_m[c + t + u];
                }
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const float4 D = d24[k][(c + t) / 4];
                    const float d2s[4] = {D.x, D.y, D.z, D.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        float w = inv_r2(d1sq[u], d2s[u]);
                        if (!UNIT) w = ms[u] * w;
                        A.in1[k] = fmaf(d1[u], w, A.in1[k]);
                        A.in2[k] = fmaf(d2s[u], w, A.in2[k]);
                    }
                }
            }
            fold<R>(A);
        }
        if (full < cnt) {
            for (int t = full; t < cnt; ++t) {
                const float d1 = (float)(t1 - sm.X[t]);
                const float d1sq = fmaf(d1, d1, kTiny);
                const float m = UNIT ? 1.0f : s_m[t];
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const float d2 = reinterpret_cast<const float *>(d24[k])[t];
                    float w = inv_r2(d1sq, d2);
                    if (!UNIT) w = m * w;
                    A.in1[k] = fmaf(d1, w, A.in1[k]);
                    A.in2[k] = fmaf(d2, w, A.in2[k]);
                }
            }
            fold<R>(A);
        }
    }

    template <int R>
    __device__ __forceinline__ static void fold(Acc &A)
    {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            kahan_add(A.s1[k], A.c1[k], A.in1[k]);
            kahan_add(A.s2[k], A.c2[k], A.in2[k]);
            A.in1[k] = A.in2[k] = 0.0f;
        }
    }

    // the smallest compiled count that holds nr rows (nr is the wave's)
    template <int R>
    __device__ __forceinline__ static void stage_rows(int nr, const Smem &sm,
                                                      const float4 (*d24)[LT / 4], double t1,
                                                      int cnt, Acc &A)
    {
        if constexpr (R > STEP) {
            if (nr <= R - STEP) {
                stage_rows<R - STEP>(nr, sm, d24, t1, cnt, A);
                return;
            }
        }
        stage<R>(sm, d24, t1, cnt, A);
    }

    // rays of columns 64 tx .. and rows j0 .. j0 + nr - 1, tx, j0 and nr <= RPT
    // the calling wave's own; all waves of the workgroup call it
    __device__ static void run(Smem &sm, const DirectArgs &a, int64_t tx, int64_t j0, int nr)
    {
        const DevGeom &g = a.g;
        float *s_m = reinterpret_cast<float *>(sm.m4);
        const int tid = threadIdx.x;
        const int lane = tid % kWave, wave = tid / kWave;
        const int64_t i = tx * kTX + lane;
        const double t1 = ray_x(g, i);
        const int32_t nl = a.nl;
        float4(*d24)[LT / 4] = sm.d24 + wave * RPT;

        Acc A;
#pragma unroll
        for (int k = 0; k < RPT; ++k)
            A.in1[k] = A.in2[k] = A.s1[k] = A.c1[k] = A.s2[k] = A.c2[k] = 0.0f;

        for (int32_t base = 0; base < nl; base += LT) {
            __syncthreads();
            for (int t = tid; t < LT; t += kThreads) {
                const int32_t li = base + t;
                if (li < nl) {
                    sm.X[t] = a.lx[li];
                    sm.Y[t] = a.ly[li];
                    if (!UNIT) s_m[t] = (float)a.lm[li];
                }
            }
            __syncthreads();
            const int cnt = min(LT, nl - base);
            for (int k = 0; k < nr; ++k) {
                const double t2r = ray_y(g, j0 + k);
                for (int t = lane; t < cnt; t += kWave)
                    reinterpret_cast<float *>(d24[k])[t] = (float)(t2r - sm.Y[t]);
            }
            // the wave's own rows: its LDS writes before its reads
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (nr > 0) stage_rows<RPT>(nr, sm, d24, t1, cnt, A);
        }

        // FP64 near-lens residual, assembly and output, ray by ray; one body,
        // with the next row's sums moved to index 0 after each
        const int64_t cx = ((2 * i + 1) * (int64_t)g.n1x) / (2 * g.nx);
        const int64_t cxl = cx > 0 ? cx - 1 : 0;
        const int64_t cxh = cx < g.n1x - 1 ? cx + 1 : g.n1x - 1;
#pragma unroll 1
        for (int k = 0; k < nr; ++k) {
            const int64_t j = j0 + k;
            const int64_t r = j * g.nx + i;
            const bool valid = i < g.nx && j >= a.row0 && j < a.row1 && r >= a.ray_first &&
                               r < a.ray_last;
            const double t2 = ray_y(g, j);
            double sum1 = (double)A.s1[0] - (double)A.c1[0];
            double sum2 = (double)A.s2[0] - (double)A.c2[0];
            if (valid) {
                const int64_t cy = ((2 * j + 1) * (int64_t)g.n1y) / (2 * g.ny);
                const int64_t cyl = cy > 0 ? cy - 1 : 0;
                const int64_t cyh = cy < g.n1y - 1 ? cy + 1 : g.n1y - 1;
                double r1 = 0.0, r2s = 0.0;
                for (int64_t row = cyl; row <= cyh; ++row) {
                    const int32_t pb = a.cell_start[row * g.n1x + cxl];
                    const int32_t pe = a.cell_start[row * g.n1x + cxh + 1];
                    for (int32_t pl = pb; pl < pe; ++pl) {
                        const double X = a.lx[pl], Y = a.ly[pl];
                        const double m64 = UNIT ? 1.0 : a.lm[pl];
                        // the FP32 term exactly as the main loop formed it
                        const float d1f = (float)(t1 - X);
                        const float d2f = (float)(t2 - Y);
                        float w = inv_r2(fmaf(d1f, d1f, kTiny), d2f);
                        if (!UNIT) w = (float)m64 * w;
                        // the FP64 term
                        const double e1 = t1 - X, e2 = t2 - Y;
                        const double rr2 = e1 * e1 + e2 * e2;
                        const double w64 = rr2 > 0.0 ? m64 / rr2 : 0.0;
                        r1 += w64 * e1 - (double)d1f * (double)w;
                        r2s += w64 * e2 - (double)d2f * (double)w;
                    }
                }
                sum1 += r1;
                sum2 += r2s;
            }
            double a1, a2;
            int32_t pix;
            assemble(g, t1, t2, sum1, sum2, a1, a2, pix);
            emit(valid, r - a.ray_first, a1, a2, pix, a.a1o, a.a2o, a.pixo, a.counts, a.landed);
#pragma unroll
            for (int h = 0; h + 1 < RPT; ++h) {
                A.s1[h] = A.s1[h + 1];
                A.c1[h] = A.c1[h + 1];
                A.s2[h] = A.s2[h + 1];
                A.c2[h] = A.c2[h + 1];
            }
        }
    }
};

// One launch's rays as pieces, one per wave: tile columns of 64 rays, `split`
// of them cut into p + 1 runs of rows and the others into p, each column as
// evenly as its rows allow, so the runs of a column differ by one row at most.
// The longer runs come first, which leaves the SIMDs that get the grid's waves
// in turn about equally loaded.
struct DirectSplit {
    int64_t tx0, ntx;                    // tile columns
    int64_t j0;                          // first row
    int32_t rows;
    int32_t p;
    int64_t split;
    int64_t end[4];                      // ends of the classes: long runs of the columns
                                         // with p and p + 1, then their short runs
};

namespace {

// waves per SIMD of a tile with RPT rows a wave: what its registers and LDS allow
constexpr int direct_waves(int64_t rpt) { return rpt == 8 ? 4 : rpt < 8 ? 3 : 2; }
// Pieces per SIMD and round, on 1024 SIMDs.  Whole tiles of 32 rows leave a last
// round nearly empty (1067 workgroups of three a compute unit: 53.2 ms for 2e6
// rays and 1e5 lenses; 39.6 ms in equal pieces; 560: 1575 against 1033 us for
// 1e6 rays and 4450 lenses).  Six a SIMD where four are resident: the pieces
// that start later keep the SIMD busy while the first ones stage and end
// (four: 40.6 ms and 1130 us; 1e6 rays, 1e5 lenses: 20.9 against 22.0 ms).
constexpr int64_t direct_round(int64_t rpt) { return 1024 * (rpt == 8 ? 6 : rpt < 8 ? 3 : 2); }

DirectSplit direct_split(int64_t tx0, int64_t ntx, int64_t j0, int64_t rows, int64_t rpt)
{
    const int64_t round = direct_round(rpt);
    // the least number of pieces in whole rounds, of one row at least
    const int64_t need = ntx * ((rows + rpt - 1) / rpt);
    int64_t total = (need + round - 1) / round * round;
    total = std::min(total, ntx * rows);
    DirectSplit d{};
    d.tx0 = tx0;
    d.ntx = ntx;
    d.j0 = j0;
    d.rows = (int32_t)rows;
    d.p = (int32_t)(total / ntx);
    d.split = d.p < rows ? total % ntx : 0;
    const int64_t np[2] = {d.p, d.p + 1}, nc[2] = {ntx - d.split, d.split};
    int64_t e = 0;
    for (int c = 0; c < 2; ++c) d.end[c] = e += nc[c] * (rows % np[c]);
    for (int c = 0; c < 2; ++c) d.end[2 + c] = e += nc[c] * (np[c] - rows % np[c]);
    return d;
}

template <bool UNIT, int RPT, int LT>
__global__ __launch_bounds__(kThreads, direct_waves(RPT)) void k_direct_f32(DirectArgs a, DirectSplit d)
{
    using T = DirectTile<UNIT, RPT, LT>;
    __shared__ typename T::Smem sm;
    const int64_t w = (int64_t)blockIdx.x * kWaves +
                      __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int64_t tx = d.tx0, j0 = d.j0;
    int nr = 0;
    if (w < d.end[3]) {
        const int c = w < d.end[0] ? 0 : w < d.end[1] ? 1 : w < d.end[2] ? 2 : 3;
        const int32_t np = d.p + (c & 1);
        const int32_t len = d.rows / np, nlong = d.rows % np;
        const uint32_t v = (uint32_t)(w - (c ? d.end[c - 1] : 0));
        const uint32_t per = (uint32_t)(c < 2 ? nlong : np - nlong);
        const uint32_t col = v / per, q = v - col * per;
        tx += col + ((c & 1) ? 0 : d.split);
        nr = len + (c < 2);
        j0 += c < 2 ? (int64_t)q * nr : (int64_t)nlong * (len + 1) + (int64_t)q * len;
    }
    T::run(sm, a, tx, j0, nr);
}

// Persistent form for batches: workgroups pull (map, tile) items from a
// device queue until it is empty.  Items are numbered map by map in the
// order the host chose (longest-processing-time first); item_start[m] is the
// first item of map m and item_start[nmaps] the total.
template <bool UNIT, int RPT, int LT>
__global__ __launch_bounds__(kThreads, direct_waves(RPT)) void k_direct_f32_queue(
    const DirectArgs *__restrict__ maps, const int64_t *__restrict__ item_start, int32_t nmaps,
    unsigned long long *cursor)
{
    using T = DirectTile<UNIT, RPT, LT>;
    __shared__ typename T::Smem sm;
    __shared__ long long s_item;
    const int64_t total = item_start[nmaps];
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = (long long)atomicAdd(cursor, 1ull);
        __syncthreads();
        const int64_t item = s_item;
        if (item >= total) break;                    // every workgroup reaches this
        int lo = 0, hi = nmaps - 1;                  // map m with item_start[m] <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (item_start[mid] <= item) lo = mid;
            else hi = mid - 1;
        }
        const DirectArgs &a = maps[lo];
        const int64_t t = item - item_start[lo];
        const int64_t j0 = (t / a.ntx) * T::TY +
                           RPT * __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
        T::run(sm, a, t % a.ntx, j0,
               (int)max((int64_t)0, min((int64_t)RPT, a.row1 - j0)));
    }
}

}  // namespace

irs_status launch_direct(irs_plan_s *p, const RaySel &sel)
{
    const DevGeom &g = p->dg;
    const int32_t nl = (int32_t)p->n_lens;
    hipStream_t s = p->stream;
    const bool unit = p->unit_mass;
    if (sel.row1 <= sel.row0) return IRS_OK;

    if (p->params.precision == IRS_FP64) {
        const int64_t rb = std::max(sel.row0 * g.nx, sel.ray_first);
        const int64_t re = std::min(sel.row1 * g.nx, sel.ray_last);
        if (sel.stats) sel.stats->direct_pairs += std::max<int64_t>(0, re - rb) * (int64_t)nl;
        if (re <= rb) return IRS_OK;
        const bool tame = p->tame;
        // the call's units: blocks, half blocks or rays
        const bool blocks = direct_blocks(p) > 0;
        const int64_t nb = (g.nx + kBlock - 1) / kBlock;
        int64_t u0 = rb, u1 = re;
        bool few = false;
        if (blocks) {
            u0 = rb / g.nx * nb + rb % g.nx / kBlock;
            u1 = (re - 1) / g.nx * nb + (re - 1) % g.nx / kBlock + 1;
            few = u1 - u0 <= kFewBlocks;
            if (few) {
                u0 *= 2;
                u1 *= 2;
            }
        }
        const int64_t chunk = (int64_t)1 << (blocks ? 22 : 30);      // units a launch
        const int64_t per = blocks ? kWaves : kThreads;              // ... a workgroup
        for (int64_t c0 = u0; c0 < u1; c0 += chunk) {
            const int64_t c1 = std::min(u1, c0 + chunk);
            const unsigned grid = (unsigned)((c1 - c0 + per - 1) / per);
            if (sel.stats) {
                irs_status st = sel.stats->begin(s, 1);
                if (st != IRS_OK) return st;
                sel.stats->n_rays++;
            }
#define IRS_OUT sel.ray_first, sel.alpha1, sel.alpha2, sel.pixel, sel.counts, sel.landed
#define IRS_D64(U)                                                                             \
    do {                                                                                       \
        if (few)                                                                               \
            hipLaunchKernelGGL((k_direct_f64_blocks<U, 2>), dim3(grid), dim3(kThreads), 0, s, \
                               g, p->d_x, p->d_y, p->d_m, nl, tame, c0, c1, rb, re, IRS_OUT);  \
        else if (blocks)                                                                       \
            hipLaunchKernelGGL((k_direct_f64_blocks<U, 4>), dim3(grid), dim3(kThreads), 0, s, \
                               g, p->d_x, p->d_y, p->d_m, nl, tame, c0, c1, rb, re, IRS_OUT);  \
        else                                                                                   \
            hipLaunchKernelGGL(k_direct_f64<U>, dim3(grid), dim3(kThreads), 0, s, g, p->d_x,   \
                               p->d_y, p->d_m, nl, tame, c0, c1, IRS_OUT);                     \
    } while (0)
            if (unit) IRS_D64(true);
            else IRS_D64(false);
#undef IRS_D64
#undef IRS_OUT
            IRS_HIP(hipGetLastError());
            if (sel.stats) {
                irs_status st = sel.stats->end(s);
                if (st != IRS_OK) return st;
            }
        }
        return IRS_OK;
    }

    const int v = p->direct_variant;
    const int64_t rpt = direct_variant_rows(v) / kWaves;
    // rows that hold rays asked for, and the columns if it is one row
    const int64_t jA = std::max(sel.row0, sel.ray_first / g.nx);
    const int64_t jB = std::min(sel.row1, (sel.ray_last + g.nx - 1) / g.nx);
    if (jB <= jA || sel.ray_last <= sel.ray_first) return IRS_OK;
    int64_t tx0 = 0, tx1 = (g.nx + kTX - 1) / kTX;
    if (jB - jA == 1) {
        tx0 = std::max<int64_t>(0, sel.ray_first - jA * g.nx) / kTX;
        tx1 = (std::min(g.nx, sel.ray_last - jA * g.nx) + kTX - 1) / kTX;
    }
    const int64_t ntx = tx1 - tx0;
    const int64_t max_rows = std::max<int64_t>(1, ((int64_t)1 << 22) / ntx) * rpt * kWaves;
    if (sel.stats) {
        const int64_t r0 = std::max(sel.row0 * g.nx, sel.ray_first);
        const int64_t r1 = std::min(sel.row1 * g.nx, sel.ray_last);
        sel.stats->direct_pairs += std::max<int64_t>(0, r1 - r0) * (int64_t)nl;
    }
    DirectArgs a{};
    a.g = g;
    a.lx = p->d_x;
    a.ly = p->d_y;
    a.lm = p->d_m;
    a.cell_start = p->d_cell_start;
    a.nl = nl;
    a.ntx = ntx;
    a.row0 = sel.row0;
    a.row1 = sel.row1;
    a.ray_first = sel.ray_first;
    a.ray_last = sel.ray_last;
    a.a1o = sel.alpha1;
    a.a2o = sel.alpha2;
    a.pixo = sel.pixel;
    a.counts = sel.counts;
    a.landed = sel.landed;
    for (int64_t j0 = jA; j0 < jB; j0 += max_rows) {
        const DirectSplit d = direct_split(tx0, ntx, j0, std::min(max_rows, jB - j0), rpt);
        const unsigned nb = (unsigned)((d.end[3] + kWaves - 1) / kWaves);
        if (sel.stats) {
            irs_status st = sel.stats->begin(s, 1);
            if (st != IRS_OK) return st;
            sel.stats->n_rays++;
        }
#define IRS_DF32(U, R, L) hipLaunchKernelGGL((k_direct_f32<U, R, L>), dim3(nb), dim3(kThreads), 0, s, a, d)
        if (unit) {
            if (v == 0) IRS_DF32(true, 4, 512);
            else if (v == 1) IRS_DF32(true, 8, 256);
            else IRS_DF32(true, 16, 128);
        } else {
            if (v == 0) IRS_DF32(false, 4, 512);
            else if (v == 1) IRS_DF32(false, 8, 256);
            else IRS_DF32(false, 16, 128);
        }
#undef IRS_DF32
        IRS_HIP(hipGetLastError());
        if (sel.stats) {
            irs_status st = sel.stats->end(s);
            if (st != IRS_OK) return st;
        }
    }
    return IRS_OK;
}

int direct_variant_rows(int v) { return (v == 0 ? 4 : v == 1 ? 8 : 16) * kWaves; }

const char *direct_variant_name(int v)
{
    return v == 0 ? "rpt4_lt512" : v == 1 ? "rpt8_lt256" : "rpt16_lt128";
}

int64_t direct_items(const irs_plan_s *p, int variant)
{
    const DevGeom &g = p->dg;
    if (p->params.precision == IRS_FP64) {
        const int64_t nb = direct_blocks(p);
        return nb > 0 ? (nb + kWaves - 1) / kWaves : (g.nx * g.ny + kThreads - 1) / kThreads;
    }
    const int64_t TY = direct_variant_rows(variant);
    return ((g.nx + kTX - 1) / kTX) * ((g.ny + TY - 1) / TY);
}

DirectArgs direct_args_full(const irs_plan_s *p, int variant, uint32_t *counts,
                            unsigned long long *landed)
{
    DirectArgs a{};
    a.g = p->dg;
    a.lx = p->d_x;
    a.ly = p->d_y;
    a.lm = p->d_m;
    a.cell_start = p->d_cell_start;
    a.nl = (int32_t)p->n_lens;
    a.tame = p->tame ? 1 : 0;
    a.ntx = (p->dg.nx + kTX - 1) / kTX;
    a.blocks = direct_blocks(p);
    a.row0 = 0;
    a.row1 = p->dg.ny;
    a.ray_first = 0;
    a.ray_last = p->dg.nx * p->dg.ny;
    a.counts = counts;
    a.landed = landed;
    (void)variant;
    return a;
}

irs_status launch_direct_queue(hipStream_t s, int precision, bool unit, int v,
                               const DirectArgs *maps, const int64_t *item_start,
                               int32_t nmaps, unsigned long long *cursor, int blocks)
{
    if (precision == IRS_FP64) {
        if (unit)
            hipLaunchKernelGGL(k_direct_f64_queue<true>, dim3(blocks), dim3(kThreads), 0, s,
                               maps, item_start, nmaps, cursor);
        else
            hipLaunchKernelGGL(k_direct_f64_queue<false>, dim3(blocks), dim3(kThreads), 0, s,
                               maps, item_start, nmaps, cursor);
    } else {
#define IRS_DQ(U, R, L) hipLaunchKernelGGL((k_direct_f32_queue<U, R, L>), dim3(blocks), dim3(kThreads), 0, s, maps, item_start, nmaps, cursor)
        if (unit) {
            if (v == 0) IRS_DQ(true, 4, 512);
            else if (v == 1) IRS_DQ(true, 8, 256);
            else IRS_DQ(true, 16, 128);
        } else {
            if (v == 0) IRS_DQ(false, 4, 512);
            else if (v == 1) IRS_DQ(false, 8, 256);
            else IRS_DQ(false, 16, 128);
        }
#undef IRS_DQ
    }
    IRS_HIP(hipGetLastError());
    return IRS_OK;
}

namespace {
__global__ void k_zero(uint32_t *__restrict__ p, size_t n, uint32_t *__restrict__ p2, size_t m)
{
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < m; i += step) p2[i] = 0u;
    // 16 bytes a store where p allows it
    const size_t head = min(n, (size_t)(-(intptr_t)p & 15) / 4), quads = (n - head) / 4;
    uint4 *q = (uint4 *)(p + head);
    for (size_t i = i0; i < quads; i += step) q[i] = make_uint4(0u, 0u, 0u, 0u);
    if (i0 < head) p[i0] = 0u;
    if (i0 < n - head - 4 * quads) p[head + 4 * quads + i0] = 0u;
}
}  // namespace

irs_status launch_zero(hipStream_t s, void *ptr, size_t n_words, void *ptr2, size_t m_words)
{
    if (n_words + m_words == 0) return IRS_OK;
    const size_t blocks = std::min<size_t>((std::max(n_words / 4, m_words) + 255) / 256 + 1, 4096);
    hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t *)ptr, n_words,
                       (uint32_t *)ptr2, m_words);
    IRS_HIP(hipGetLastError());
    return IRS_OK;
}

}  // namespace irs
