// lens_device.h -- per-sub-pixel physics of the forward model, gfx950.
//
// Cao et al. (2025), Sec. 2.1 (Eqs. 1-2) and Sec. 2.4 (Eqs. 8-10, 12-14).
// Every function here runs E times per proposal (E = sub-pixels in the
// mask's PSF-dilated footprint).
//
// Precision.  beta = theta - alpha is a difference of arcsecond-sized
// numbers, and a Sersic profile with n > 1 has an infinitely steep cusp at
// its centre: an FP32 ray trace (absolute error ~4e-7 arcsec) gives 1e-5
// brightness errors next to a cusp.  Likewise b_n (R/R_e)^(1/n) amplifies the
// relative error of (R/R_e)^(1/n) by up to ~30.  So the ray trace and the
// profiles run in FP64 -- FP64 FMAs issue at the FP32 rate on CDNA4 -- with
// FP32 hardware only where its error is not amplified: the reciprocal and
// reciprocal-square-root seeds (refined by a Newton step) and log2 of the
// elliptical radius, whose error reaches the exponent scaled by
// b_n/(2n ln 2) ~ 1.  The binned pixel is rounded to FP32 once.
#pragma once

#include <hip/hip_runtime.h>

#include "lens_approx.h"
#include "lens_internal.h"

namespace lensk {

__device__ __forceinline__ float hw_log2(float x) { return __builtin_amdgcn_logf(x); }

// 1/sqrt(x) and 1/x for x in the normal FP32 range: FP32 hardware seed and
// one FP64 Newton step (relative error ~1e-14).
__device__ __forceinline__ double rsq_nr(double x)
{
    const double r = (double)__builtin_amdgcn_rsqf((float)x);
    return fma(0.5 * r, fma(-(x * r), r, 1.0), r);
}

__device__ __forceinline__ double rcp_nr(double x)
{
    const double r = (double)__builtin_amdgcn_rcpf((float)x);
    return fma(r, fma(-x, r, 1.0), r);
}

// 1/sqrt(x) for any x > 0: FP64 hardware seed and two Newton steps.
__device__ __forceinline__ double rsq64(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    r = fma(0.5 * r, fma(-(x * r), r, 1.0), r);
    return fma(0.5 * r, fma(-(x * r), r, 1.0), r);
}

// 1/psi from psi2 = psi^2 >= 0, and 0 at psi = 0: rsq_nr where psi2 lies in
// FP32's normal range, else rsq64.  The test is wave-uniform and laid out
// for its usual outcome (no lane of the wave at the mass centre), which then
// runs without a taken branch; each lane's result is the same either way.
__device__ __forceinline__ double rsq_psi(double psi2)
{
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psi2 >= 1e-30)) == 0, 1)) return rsq_nr(psi2);
    // a copy the compiler cannot see through, so that this path's per-lane
    // test stays inside it instead of being computed on the common path too
    double p = psi2;
    asm volatile("" : "+v"(p));
    return p >= 1e-30 ? rsq_nr(p) : p > 0.0 ? rsq64(p) : 0.0;
}

// a b + c as one VOP3 v_fma_f64 with c taken from an SGPR pair; c must be
// wave-uniform (here: a polynomial coefficient).  Written out because the
// compiler otherwise keeps FP64 coefficients in VGPRs and emits v_fmac_f64,
// whose tied addend costs a v_mov_b64 per step and ~40 VGPRs for the tables.
__device__ __forceinline__ double fma_c(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// sum_i c[i] w^i; `lead` holds c[N - 1] (a caller may pass it in a VGPR
// loaded once outside its loop, which saves a v_mov_b64 per evaluation).
template <int N>
__device__ __forceinline__ double horner(const double (&c)[N], double w, double lead)
{
    double p = lead;
#pragma unroll
    for (int i = N - 2; i >= 0; --i) p = fma_c(p, w, c[i]);
    return p;
}

template <int N>
__device__ __forceinline__ double horner(const double (&c)[N], double w)
{
    return horner(c, w, c[N - 1]);
}

template <int N>
__device__ __forceinline__ constexpr double leading(const double (&c)[N])
{
    return c[N - 1];
}

// Adding 1.5 * 2^52 rounds a double below 2^51 in magnitude to an integer, and
// leaves that integer in the sum's low word.
constexpr double kRound = 6755399441055744.0;

// 2^(e l) for e l in [-1022, 1023]: 2^round(e l) times a polynomial in the
// remainder.  `round` holds kRound and `lead` c[N - 1] (a caller may pass them
// in VGPRs loaded once outside its loop: an instruction takes one scalar
// operand).  Rounding by addition saves the conversion of the integer.
template <int N>
__device__ __forceinline__ double exp2_64(const double (&c)[N], double e, double l, double lead, double round)
{
    const double m = fma(e, l, round), k = m - round;
    return ldexp(horner(c, fma(e, l, -k), lead), __double2loint(m));
}

template <int N>
__device__ __forceinline__ double exp2_64(const double (&c)[N], double e, double l)
{
    return exp2_64(c, e, l, c[N - 1], kRound);
}

constexpr double kPi2 = 1.5707963267948966;
constexpr double kAtanh075 = 0.97295507452765665255;   // atanh(3/4)

// theta_E sqrt(q) atan(c u1)/c (the SIE deflection along the major axis).
// |c u1| <= 1: polynomial in (c u1)^2; else atan t = pi/2 - atan(1/t).
// |c u1| > 1 needs q < 1/sqrt(2) and a cone around the major axis, so most
// waves have no such lane: they skip the reduction on a wave-uniform branch
// (a divergent one would still issue it, with the lanes masked off).  Each
// lane's arithmetic is the same on either path.
__device__ __forceinline__ double sie_a1(double u1, double ce, double bsie, double bsc)
{
    const double t = ce * u1;
    const double z = fabs(t);
    const bool big = z > 1.0;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(big) != 0, 0)) {
        const double zi = big ? rcp_nr(z) : z;
        const double p = horner(kAtanOverT64, zi * zi);
        return big ? copysign(bsc * fma(-zi, p, kPi2), t) : bsie * u1 * p;
    }
    return bsie * u1 * horner(kAtanOverT64, z * z);
}

// theta_E sqrt(q) atanh(c u2)/c (along the minor axis).  |t| <= 1/2:
// polynomial in t^2; 1/2 < |t| <= 0.9: atanh z = atanh(3/4) + atanh((z - 3/4)/(1 - 3z/4)),
// whose second argument lies in [-0.4, 0.47]; |t| > 0.9 (axis ratios below
// 0.44 only): the logarithm.
__device__ __forceinline__ double sie_a2(double u2, double ce, double bsie, double bsc)
{
    const double t = ce * u2;
    const double z = fabs(t);
    if (z <= 0.9) {
        const bool red = z > 0.5;
        // the reduction on a wave-uniform branch, as in sie_a1
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(red) != 0, 0)) {
            const double zr = red ? (z - 0.75) * rcp_nr(fma(-0.75, z, 1.0)) : z;
            const double p = horner(kAtanhOverT64, zr * zr);
            return red ? copysign(bsc * fma_c(zr, p, kAtanh075), t) : bsie * u2 * p;
        }
        return bsie * u2 * horner(kAtanhOverT64, z * z);
    }
    // atanh z = (ln 2 / 2) log2 y with y = (1 + z)/(1 - z) > 19:
    // FP32 log2 seed l0 (absolute error ~1e-6), then one Newton step on 2^l = y,
    // l1 = l0 + (y 2^-l0 - 1) log2 e: quadratic in the seed's error (~1e-13), plus the
    // 2^x polynomial's 1.9e-9, i.e. < 1e-9 relative in atanh z (log2 y > 4.2).
    const double y = (1.0 + z) * rcp_nr(1.0 - z);
    const double l0 = (double)hw_log2((float)y);
    const double l1 = fma(fma(y, exp2_64(kExp2_64, -1.0, l0), -1.0), 1.4426950408889634, l0);
    return copysign(bsc * 0.34657359027997264 * l1, t);
}

// Elliptical Sersic (Eqs. 8, 10) without its amplitude, from r2 = (R/R_e)^2:
//   exp(-b ((R/R_e)^(1/n) - 1)) = 2^(B (1 - t)),  t = r2^(1/(2n)),  B = b log2 e.
// log2 r2 = (binary exponent of r2) + log2(mantissa in [1/2, 1)), the FP32
// hardware log2 seeing only the mantissa and the sum taken in FP64: an absolute
// error of ~1e-7 at any magnitude.  (An FP32 log2 of r2 itself is good to one
// ulp of its result, ~1e-6 absolute once |log2 r2| nears 20, i.e. next to a
// steep Sersic centre, and the exponent carries that error into the
// brightness.)  The mantissa's log2 is clamped below at -2048, so the centre
// (r2 = 0) gives t = 2^-(2048 e) ~ 0 rather than NaN; a radius whose t
// overflows gives B (1 - t) = -inf, whose power of two exp2_hw makes 0.
// lead: the leading coefficient of kExp2_64 (see horner).
__device__ __forceinline__ double log2_r2(double r2)
{
    const float lm = __builtin_amdgcn_fmed3f(hw_log2((float)__builtin_amdgcn_frexp_mant(r2)), -2048.0f, 0.0f);
    return (double)__builtin_amdgcn_frexp_exp(r2) + (double)lm;
}

// log2 r2 for a Sersic exponent.  For a profile with n >= 1/2 (e <= 1),
// where every lane of the wave has log2 r2 >= -2 (R >= R_e / 2),
// it is the FP32 hardware log2 of r2 itself: an absolute error within an ulp
// of a result of that size (1.2e-7 for |l| < 2, 2.4e-7 for |l| < 4) plus
// 8.6e-8 from rounding r2 to FP32.  It reaches the brightness scaled by
// ln2^2 B e t (t = 2^(e l)): with one-ulp errors of this log2 and of exp2_hw
// aligned, at most 8.8e-7 of the local brightness wherever that is above 1/8
// of its value at R_e, against 1.1e-6 for the exponent split over the whole
// index domain (whose worst case is at n = 0.1, where this form would reach
// 1.7e-6: hence the gate on e).  A wave with a lane nearer a centre (where t
// is small and the cusp steep, and where r2 = 0 gives -inf) takes log2_r2.
// A radius whose FP32 value overflows gives l = +inf, t = NaN and, through
// exp2_hw, 0, as log2_r2's large finite value does.
// thr (uniform): -2 where the FP32 form is allowed, +inf where it is not (a
// threshold rather than a flag keeps the sub-pixel loop's code the same).
// The test is laid out for the FP32 form, which then runs without a taken
// branch (most waves take it; two taken branches per Sersic cost 2%).
__device__ __forceinline__ double log2_r2_sersic(double r2, float thr)
{
    const float l = hw_log2((float)r2);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(l >= thr)) != 0, 0)) return log2_r2(r2);
    return (double)l;
}

// 2^y for y <= 1023, -inf and NaN included, for the brightness 2^(B (1 - t)), whose
// relative error is that of this function alone: nothing amplifies it.  The
// FP32 hardware 2^x is good to about one FP32 ulp of its result.
// - Where every lane of the wave has y <= 2, it is that 2^x of y rounded to
//   FP32.  The rounding adds at most ln2 2^-24 = 4.1e-8 relative for y in
//   [-2, 2], 8.3e-8 down to y = -4 (a sixteenth of the brightness at R_e),
//   and grows with |y| below, where the brightness shrinks faster.  Below
//   y = -126 the result is an FP32 subnormal or 0, under 1.2e-38 of the
//   brightness at R_e, and -inf gives 0.
// - Otherwise it is 2^round(y) times the 2^x of the remainder f in
//   [-1/2, 1/2] (f rounded to FP32: 1e-8 relative), as the centre of a steep
//   profile needs: there y reaches B, up to 57 at n = 20.  Here y is first
//   raised to -2000 (2^-2000 is 0 in FP64), which also maps NaN to 0: a NaN
//   lane fails the test above and lands here.
// The test is laid out for the first form, the common one.
__device__ __forceinline__ double exp2_hw(double y)
{
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(y <= 2.0)) == 0, 1)) return (double)__builtin_amdgcn_exp2f((float)y);
    y = fmax(y, -2000.0);
    const double k = rint(y);
    return ldexp((double)__builtin_amdgcn_exp2f((float)(y - k)), (int)k);
}

// 2^(B (1 - t)) with t = 2^(e lgd), lgd = log2 of (R/R_e)^2 (as above).  t's
// relative error is amplified by ln2 B t in the exponent, so it takes the FP64
// polynomial; the outer power's is not.
__device__ __forceinline__ double sersic_lg(double lgd, double e, double B, double lead, double round)
{
    const double t = exp2_64(kExp2_64, e, lgd, lead, round);
    return exp2_hw(fma(-B, t, B));
}

// The source's (R/R_e)^2 from the scaled offsets W1, W2 (PropBlock::src).
__device__ __forceinline__ double source_r2(double W1, double W2, const LightK &L)
{
    const double a = fma(L.S, W2, W1);
    return fma(a, a, W2 * W2);
}

// Source-plane position beta = theta - alpha - alpha_shear (Eqs. 1-2) as the
// scaled offsets W1, W2 of PropBlock, given (X1, X2) = (q x1, x2), the
// sub-pixel's coordinates in the frame of the mass ellipse, and the part
// linear in theta, (U1, U2).  With R = sqrt(X1^2 + X2^2) and (c, s) = (X1, X2) / R:
// SIE (kappa = theta_E / (2 R_p)): c_e = sqrt(1 - q^2),
// alpha = theta_E sqrt(q) / c_e (atan(c_e x1/R), atanh(c_e x2/R)) in the mass
// frame; alpha = 0 at the centre.  Shear (inside U): alpha = -(g1 x + g2 y, g2 x - g1 y).
// iq = 1 / q.
__device__ __forceinline__ void ray_trace(double X1, double X2, double U1, double U2, const PropBlock &P, double iq,
                                          double &W1, double &W2)
{
    const double ir = rsq_psi(fma(X1, X1, X2 * X2));
    const double a1 = sie_a1(X1 * ir * iq, P.ce, P.bsie, P.bsc);
    const double a2 = sie_a2(X2 * ir, P.ce, P.bsie, P.bsc);
    W1 = fma(-P.src.P, a1, U1);
    W2 = fma(-P.src.Q, a2, U2);
}

// The deflection from a per-proposal table.  c^2 + s^2 = 1, so the SIE's
// deflection is a function of the direction (c, s) alone, odd in each of its
// components: (p1 alpha1, q2 alpha2) = (c T1(u), s T2(u)) with u = |c| in
// [0, 1].  So is the power law's, times R^(1 - t) (see ray_trace_epl).  T1 and
// T2 are analytic except at u = +-i q / c_e (for the power law the branch
// point of its series, |e^(2 i phi)| = 1/f, is the same point); on each of
// the intervals of u the table holds the polynomial through their values at the
// interval's Chebyshev nodes (from sie_a1 and sie_a2, or the series).  With 32
// intervals and degree 5 that reproduces the SIE's to 1.3e-12 (q = 0.5) and
// 4e-11 (q = 0.3) relative, against 4e-10 and 1.3e-9 of the polynomials behind
// sie_a1 and sie_a2 (16 intervals at degree 6 are as accurate at two more FMAs
// per sub-pixel).  A sub-pixel then takes one interval lookup and two Horner
// sums instead of both deflection functions and, in most waves, a range
// reduction; or instead of the series, 20 terms of four FMAs each on average.  Below q = 0.3 the singularities come
// too close and the direct functions are used.
constexpr double kSieTabQ2 = 0.09;   // q^2 from which the table is used
constexpr double kTiny = 1e-37;      // above FP32's smallest normal number
// The power law's table replaces a series that is good to the rounding of FP64,
// and where a sub-pixel happens to land within ~1e-9 arcsec of a steep source's
// centre, a deflection off by 1e-12 already shows in lnL (5e-8 of it, once in
// 8,685 proposals).  Hence 64 intervals at degree 7: interpolation errors up to
// 1.0e-15 relative over every accepted slope (q = 0.3, t = 1.95; 3e-16 at t = 1.4,
// 1e-17 at q = 0.5), where degree 5 gave 6.6e-12 there and 1.8e-13 at q = 0.5, and
// degree 6 7.5e-14.  The monomial coefficients come from differences to a node's
// value: from the values themselves the rounding of their sums alone, amplified
// by the interpolation matrix, was 1e-14.  Evaluated in FP64 the table is then
// within 1.6e-15 of the series at 64 bits, the series itself within 5e-16.
template <bool EPL>
struct TabShape;
template <>
struct TabShape<false> {
    static constexpr int NI = kSieIntervals, DEG = kSieDeg, ENTRY = kSieEntry;
    __device__ static double node(int k) { return kSieNode[k]; }
    __device__ static constexpr double interp(int i, int k) { return kSieInterp[i][k]; }
};
template <>
struct TabShape<true> {
    static constexpr int NI = kEplIntervals, DEG = kEplDeg, ENTRY = kEplEntry;
    __device__ static double node(int k) { return kEplNode[k]; }
    __device__ static constexpr double interp(int i, int k) { return kEplInterp[i][k]; }
};
static_assert(kSieEntry >= 2 * kSieDeg + 2 && kEplEntry >= 2 * kEplDeg + 2, "deflection table entry");

// The SIE's table is static LDS, the power law's two tables lie behind the ring:
// together they are as large as some 50 ring columns of the widest images, which
// are then served without them (LensGeom::tab_off).
template <bool EPL>
__device__ __forceinline__ double *sie_table(const LensGeom &g)
{
    if constexpr (EPL) {
        extern __shared__ float4 lds4[];
        // in units of 16 bytes, so that the entries are known to be aligned and
        // read by 128-bit loads (in pairs of 64 bits the fused kernels took 20 %
        // longer)
        return reinterpret_cast<double *>(lds4 + (g.tab_off >> 4));
    } else {
        __shared__ __attribute__((aligned(16))) double t[(kSieIntervals + 1) * kSieEntry];
        return t;
    }
}

// Uniform over the workgroup.
template <bool EPL>
__device__ __forceinline__ bool sie_use_table(const LensGeom &g, const PropBlock &P)
{
    return (!EPL || g.tab_off >= 0) && P.q * P.q >= kSieTabQ2;
}

// Elliptical power law (Sec. 2.4: kappa = (3 - gamma)/2 (theta_E / R_p)^(gamma - 1)
// on the SIE's elliptical radius R_p, so gamma = 2 is the SIE).  In the frame
// of the mass ellipse, with R e^(i phi) = q x1 + i x2, t = gamma - 1,
// b = theta_E sqrt(q) and f = (1 - q)/(1 + q), the deflection is (Tessore &
// Metcalf 2015, the hypergeometric function written as its series)
//   alpha1 + i alpha2 = 2 b^t / (1 + q) R^(1 - t) e^(i phi) sum_n a_n e^(2 i n phi),
//   a_0 = 1,  a_n = -f (2n - 2 + t) / (2n + 2 - t) a_(n-1),  |a_n| <= f^n.
// The sum is taken by Horner in w = e^(2 i phi) with the proposal's
// coefficients from LDS (epl_setup): per node of the table, or per sub-pixel
// where the table is not used.
__device__ __forceinline__ double *epl_coefs()
{
    __shared__ double c[kEplMaxTerms];
    return c;
}
__device__ __forceinline__ int *epl_nterms()
{
    __shared__ int n;
    return &n;
}

// The series coefficients of proposal P into LDS, by thread 0, with the number
// of terms that brings the tail f^N / (1 - f) below 1e-16 (at most
// kEplMaxTerms: axis ratios below 0.15 then keep a tail above 1e-16), rounded up
// to whole groups of kEplGroup by zeros.  The caller's next barrier publishes
// them.
__device__ inline void epl_setup(const PropBlock &P)
{
    if (threadIdx.x != 0) return;
    const double f = -P.epl_mf, t = 1.0 - 2.0 * P.epl_h;
    int N = 1;
    if (f > 0.0) N = (int)ceil(log(1e-16 * (1.0 - f)) / log(f));
    N = N < 1 ? 1 : N > kEplMaxTerms ? kEplMaxTerms : N;
    double *c = epl_coefs();
    double a = 1.0;
    c[0] = 1.0;
    for (int n = 1; n < N; ++n) {
        a *= P.epl_mf * (2.0 * n - 2.0 + t) / (2.0 * n + 2.0 - t);
        c[n] = a;
    }
    for (; N % kEplGroup; ++N) c[N] = 0.0;
    *epl_nterms() = N;
}

// e^(i phi) sum_n a_n e^(2 i n phi) at e^(i phi) = c + i s.  By groups of terms: one
// at a time, each waited for its coefficient's way from LDS, which few waves do
// not hide (4,096 proposals of 128x128 px at axis ratios 0.15 to 0.29, 90 terms on
// average: split launches 20.8 -> 16.3 ms, the fused kernels 24 -> 17.5; 17 and 18.9
// in groups of two).
__device__ __forceinline__ void epl_angle(double c, double s, double &re, double &im)
{
    const double wr = fma(c, c, -(s * s)), wi = 2.0 * c * s;     // e^(2 i phi)
    const double *a = epl_coefs();
    const int N = __builtin_amdgcn_readfirstlane(*epl_nterms());
    double sr = 0.0, si = 0.0;
#pragma unroll 1
    for (int n = N - kEplGroup; n >= 0; n -= kEplGroup) {
        double an[kEplGroup];
#pragma unroll
        for (int j = 0; j < kEplGroup; ++j) an[j] = a[n + j];
#pragma unroll
        for (int j = kEplGroup - 1; j >= 0; --j) {
            const double tr = fma(sr, wr, fma(-si, wi, an[j]));
            si = fma(sr, wi, si * wr);
            sr = tr;
        }
    }
    re = fma(c, sr, -(s * si));
    im = fma(c, si, s * sr);
}

// R^(1 - t) = 2^(h log2 R^2) for R^2 >= 1e-30, with log2 R^2 refined by one
// Newton step on 2^l = R^2 and both powers of two at degree 11 (4e-16): good
// to ~1e-14 relative.
__device__ __forceinline__ double epl_power(double R2, double h)
{
    const double l0 = log2_r2(R2);
    const double l1 = fma(fma(R2, exp2_64(kExp2Hi64, -1.0, l0), -1.0), 1.4426950408889634, l0);
    return exp2_64(kExp2Hi64, h, l1);
}

// The same from a per-proposal table: R^2 = m 2^E, m in [1/2, 1); kPowMant
// entries hold (1/m_j, m_j^h) at the centres m_j of as many intervals of m,
// kPowExp more the powers 2^(E h) from E = kPowE0 on (R from 1e-15 to 2.3e4
// arcsec), and (m/m_j)^h is the binomial series to fifth order in m/m_j - 1,
// |.| <= 1/256: 8e-16 relative at worst (t = 1.95).
constexpr int kPowE0 = -98;
__device__ __forceinline__ double *pow_table(const LensGeom &g)
{
    return sie_table<true>(g) + (kEplIntervals + 1) * kEplEntry;
}

// The tables of proposal P by the threads [0, nt) of the workgroup; the caller
// publishes them with a barrier, and epl_setup's coefficients are published.
// Entry j of the deflection table of NI intervals: the coefficients of T1
// (from v^0 up), then those of T2, v = u NI - j in [0, 1]; one more entry holds
// the values at u = 1.
template <bool EPL>
__device__ __forceinline__ double table_node(const PropBlock &P, int comp, double u)
{
    const double s = sqrt((1.0 - u) * (1.0 + u));
    if constexpr (EPL) {
        double re, im;
        epl_angle(u, s, re, im);
        return comp == 0 ? P.src.P * P.epl_pref * re / u : P.src.Q * P.epl_pref * im / s;
    } else {
        return comp == 0 ? P.src.P * sie_a1(u / P.q, P.ce, P.bsie, P.bsc) / u
                         : P.src.Q * sie_a2(s, P.ce, P.bsie, P.bsc) / s;
    }
}

// The polynomial through the node values f (interp: in t = v - 1/2), in v.  The
// power law's from the differences to a middle node's value (see TabShape).
template <bool EPL>
__device__ __forceinline__ void table_poly(const double (&f)[TabShape<EPL>::DEG + 1],
                                           double (&c)[TabShape<EPL>::DEG + 1])
{
    constexpr int NN = TabShape<EPL>::DEG + 1;
    const double ref = EPL ? f[NN / 2] : 0.0;
#pragma unroll
    for (int i = 0; i < NN; ++i) c[i] = 0.0;
#pragma unroll
    for (int k = 0; k < NN; ++k) {
        if (EPL && k == NN / 2) continue;
        const double d = EPL ? f[k] - ref : f[k];
#pragma unroll
        for (int i = 0; i < NN; ++i) c[i] = fma(TabShape<EPL>::interp(i, k), d, c[i]);
    }
    if (EPL) c[0] += ref;
    // p(v - 1/2): synthetic division by the shift
#pragma unroll
    for (int i = 0; i < NN - 1; ++i)
#pragma unroll
        for (int k = NN - 2; k >= i; --k) c[k] = fma(-0.5, c[k + 1], c[k]);
}

// Writes one component of entry j, and of the entry past the last interval.
template <bool EPL>
__device__ __forceinline__ void table_write(const LensGeom &g, int j, int comp,
                                            const double (&c)[TabShape<EPL>::DEG + 1])
{
    constexpr int NN = TabShape<EPL>::DEG + 1;
    double *e = sie_table<EPL>(g) + j * TabShape<EPL>::ENTRY + comp * NN;
    double end = 0.0;
#pragma unroll
    for (int i = 0; i < NN; ++i) {
        e[i] = c[i];
        end += c[i];
    }
    if (j == TabShape<EPL>::NI - 1) {
        e += TabShape<EPL>::ENTRY;
#pragma unroll
        for (int i = 0; i < NN; ++i) e[i] = i == 0 ? end : 0.0;
    }
}

__device__ __forceinline__ void pow_setup(const LensGeom &g, const PropBlock &P, int tid, int nt)
{
    double *t = pow_table(g);
    for (int i = tid; i < kPowMant + kPowExp; i += nt) {
        if (i < kPowMant) {
            const double m = 0.5 + (i + 0.5) / (2 * kPowMant);
            t[2 * i] = 1.0 / m;
            t[2 * i + 1] = epl_power(m, P.epl_h);
        } else {
            t[kPowMant + i] = exp2_64(kExp2Hi64, P.epl_h, (double)(kPowE0 + i - kPowMant));
        }
    }
}

// The first threads write one interval and one component each.
template <bool EPL>
__device__ inline void sie_setup(const LensGeom &g, const PropBlock &P)
{
    if (!sie_use_table<EPL>(g, P)) return;
    constexpr int NI = TabShape<EPL>::NI, NN = TabShape<EPL>::DEG + 1;
    static_assert(2 * NI <= 256, "one thread per interval and component");
    if (EPL) pow_setup(g, P, threadIdx.x, blockDim.x);
    if (threadIdx.x >= 2 * NI) return;
    const int j = threadIdx.x >> 1, comp = threadIdx.x & 1;
    double f[NN], c[NN];
    double *e = sie_table<EPL>(g) + j * TabShape<EPL>::ENTRY + comp * NN;
    // one node at a time, through LDS (the kernels' register budget is set by
    // their busiest point, and all the nodes' deflections in flight would be it)
#pragma unroll 1
    for (int k = 0; k < NN; ++k) e[k] = table_node<EPL>(P, comp, (j + 0.5 + TabShape<EPL>::node(k)) * (1.0 / NI));
#pragma unroll
    for (int k = 0; k < NN; ++k) f[k] = e[k];
    table_poly<EPL>(f, c);
    table_write<EPL>(g, j, comp, c);
}

// The same tables by all NT threads of a workgroup that has little else to do
// before its first pixel (the split kernels): first one deflection per thread
// (every interval, component and node, left in the slot of the coefficient of
// the same number), then one polynomial per thread, in place.  The last barrier
// is the caller's.  The same operations in the same order as sie_setup.  (In the
// persistent kernels this form spilled 60 more scalar registers.)
template <int NT, bool EPL>
__device__ __forceinline__ void sie_setup_wide(const LensGeom &g, const PropBlock &P)
{
    if (!sie_use_table<EPL>(g, P)) return;   // uniform
    constexpr int NI = TabShape<EPL>::NI, NN = TabShape<EPL>::DEG + 1, NV = NI * NN, ENTRY = TabShape<EPL>::ENTRY;
    if (EPL) pow_setup(g, P, threadIdx.x, NT);
    // components by halves of the index range, so that most waves hold one
#pragma unroll 1
    for (int i = threadIdx.x; i < 2 * NV; i += NT) {
        const int comp = i >= NV, ii = comp ? i - NV : i, j = ii / NN, k = ii - j * NN;
        sie_table<EPL>(g)[j * ENTRY + comp * NN + k] =
            table_node<EPL>(P, comp, (j + 0.5 + TabShape<EPL>::node(k)) * (1.0 / NI));
    }
    __syncthreads();
    if (threadIdx.x < 2 * NI) {
        const int j = threadIdx.x >> 1, comp = threadIdx.x & 1;
        double f[NN], c[NN];
        const double *e = sie_table<EPL>(g) + j * ENTRY + comp * NN;
#pragma unroll
        for (int k = 0; k < NN; ++k) f[k] = e[k];
        table_poly<EPL>(f, c);
        table_write<EPL>(g, j, comp, c);
    }
}

// ray_trace with the deflection from the table.
template <bool EPL>
__device__ __forceinline__ void ray_trace_tab(const LensGeom &g, double X1, double X2, double U1, double U2,
                                              const PropBlock &P, double &W1, double &W2)
{
    // kTiny: at the mass centre c = s = 0, with no test for it; a relative change
    // of 1e-9 at R = 1e-14 arcsec
    const double R2 = fma(X1, X1, fma_c(X2, X2, kTiny));
    const double ir = rsq_nr(R2);
    double c = X1 * ir, s = X2 * ir;
    constexpr int DEG = TabShape<EPL>::DEG;
    // |c| <= 1 to a few roundings: rsq_nr's error is the Newton step's, which only
    // falls short
    const double un = fabs(c) * TabShape<EPL>::NI;
    // the entry's byte offset by a 24-bit multiply (full rate; j <= NI)
    const unsigned j = (unsigned)un;
    const double *e = reinterpret_cast<const double *>(reinterpret_cast<const char *>(sie_table<EPL>(g)) +
                                                       __umul24(j, (unsigned)(TabShape<EPL>::ENTRY * sizeof(double))));
    const double v = __builtin_amdgcn_fract(un);
    if constexpr (EPL) {
        const int hi = __double2hiint(R2), E = (hi >> 20) - (1022 + kPowE0);
        double mag;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64((unsigned)E >= (unsigned)kPowExp) == 0, 1)) {
            const double *t = pow_table(g), *m = t + 2 * ((hi >> (20 - kPowMantBits)) & (kPowMant - 1));
            const double h = P.epl_h, b2 = 0.5 * h * (h - 1.0), b3 = b2 * (h - 2.0) * (1.0 / 3.0),
                         b4 = b3 * (h - 3.0) * 0.25, b5 = b4 * (h - 4.0) * 0.2;
            const double x = fma(__builtin_amdgcn_frexp_mant(R2), m[0], -1.0);
            const double pw = fma(fma(fma(fma(fma(b5, x, b4), x, b3), x, b2), x, h), x, 1.0);
            mag = pw * m[1] * t[2 * kPowMant + E];
        } else {
            mag = R2 >= 1e-30 ? epl_power(R2, P.epl_h) : 0.0;
        }
        c *= mag;
        s *= mag;
    }
    double h1 = e[DEG];
#pragma unroll
    for (int i = DEG - 1; i >= 0; --i) h1 = fma(h1, v, e[i]);
    // the second set of coefficients is read after the first sum: 12 fewer
    // registers live at once (other waves hide the LDS latency)
    asm volatile("" ::: "memory");
    double h2 = e[2 * DEG + 1];
#pragma unroll
    for (int i = DEG - 1; i >= 0; --i) h2 = fma(h2, v, e[DEG + 1 + i]);
    W1 = fma(-c, h1, U1);
    W2 = fma(-s, h2, U2);
}

// The power law by its series; alpha = 0 for R^2 < 1e-30 (a sub-pixel within
// 1e-15 arcsec of the mass centre).
__device__ __forceinline__ void ray_trace_epl(double X1, double X2, double U1, double U2, const PropBlock &P,
                                              double &W1, double &W2)
{
    const double R2 = fma(X1, X1, X2 * X2);
    W1 = U1;
    W2 = U2;
    if (R2 >= 1e-30) {
        const double ir = rsq_nr(R2);
        double re, im;
        epl_angle(X1 * ir, X2 * ir, re, im);
        const double mag = P.epl_pref * epl_power(R2, P.epl_h);
        W1 = fma(-P.src.P, mag * re, U1);
        W2 = fma(-P.src.Q, mag * im, U2);
    }
}

// Sub-pixel sums of pixel (y, x), whose binned value is their mean over the
// s x s sub-pixel centres (Sec. 2.1).  Fine-grid index fx = x s + u maps to position (fx - (nx s - 1)/2) * pixel_scale / s.
// The offsets (dx, dy) from the mass centre step by pixel_scale / s (at most 7
// FP64 additions each, ~1e-15 arcsec from the direct product), and everything
// else linear in them is one FMA in dx with per-row constants: the mass-frame
// coordinates, U (PropBlock) and the lens light's (R/R_e)^2 (a quadratic in dx).  Lens and source light
// are summed apart (al, as: sums over the sub-pixels at unit amplitude).
template <int LM>
struct LightChannels {
    static constexpr int N = LM == LIGHT_BOTH ? 2 : LM == LIGHT_DOUBLE ? 4 : 1;
};

// Sub-pixel sums of pixel (y, x) of every light component at unit amplitude,
// in the order: lens (a, b), source (a, b).  Lens light only skips the ray
// trace; two components per galaxy share the elliptical radius of their side,
// whose second component differs only in R_e: log2 (R/R_b)^2 = log2 (R/R_a)^2
// + 2 log2(R_a/R_b).
template <int LM, bool EPL = false, bool TAB = false>
__device__ __forceinline__ void binned_channels(const LensGeom &g, const PropBlock &P, int y, int x,
                                                double (&acc)[LightChannels<LM>::N])
{
    constexpr bool LENS = LM != LIGHT_SRC, SRC = LM != LIGHT_LENS, DBL = LM == LIGHT_DOUBLE;
    constexpr int IS = DBL ? 2 : LENS ? 1 : 0;   // index of the (first) source channel
    constexpr int N = LightChannels<LM>::N;
    const int s = g.s;
    const double x0 = ((double)(x * s) - g.cfx) * g.sd;
    const double dx0 = x0 - P.xm;
    double dy = ((double)(y * s) - g.cfy) * g.sd - P.ym;
    // the step, the 2^x table's leading coefficient and the rounding constant
    // live in VGPRs: as SGPR pairs they are spilled or rematerialised on every
    // sub-pixel
    double h = g.sd, lead = leading(kExp2_64), rnd = kRound;
    asm("" : "+v"(h), "+v"(lead), "+v"(rnd));
    const double iq = !TAB && !EPL && SRC ? 1.0 / P.q : 0.0;
#pragma unroll
    for (int c = 0; c < N; ++c) acc[c] = 0.0;
    const double el = DBL ? g.fix_e[0] : P.lens.e, Bl = DBL ? g.fix_B[0] : P.lens.B;
    const double es = DBL ? g.fix_e[2] : P.src.e, Bs = DBL ? g.fix_B[2] : P.src.B;
    // the FP32 log2 of the Sersic radii only for indices >= 1/2
    // (log2_r2_sersic), and not for two components per galaxy: the second
    // one's exponent takes the first one's log2 shifted by 2 log2(R_a/R_b),
    // so an ulp of a large first log2 can land where the second profile is
    // still bright
    float thr_l = !DBL && el <= 1.0 ? -2.0f : __builtin_inff();
    float thr_s = !DBL && es <= 1.0 ? -2.0f : __builtin_inff();
    // in VGPRs too: the kernels have no scalar registers to spare
    asm("" : "+v"(thr_l), "+v"(thr_s));
    for (int v = 0; v < s; ++v, dy += h) {
        // values at dx = 0 of X1 = q (cm dx + sm dy), X2 = cm dy - sm dx and of U
        const double c1 = P.sq * dy, c2 = P.cm * dy;
        const double cu1 = fma(P.bu1, dy, P.au1), cu2 = fma(P.bu2, dy, P.au2);
        const double rs = P.lens.S * dy, rq = P.lens.Q * (dy * dy);
        // the channel values of the sub-pixel at offset dx
        auto sub = [&](double dx, double (&val)[N]) {
            if constexpr (SRC) {
                const double X1 = fma(P.cq, dx, c1), X2 = fma(-P.sm, dx, c2);
                const double U1 = fma(P.ku1, dx, cu1), U2 = fma(P.ku2, dx, cu2);
                double W1, W2;
                if constexpr (TAB) ray_trace_tab<EPL>(g, X1, X2, U1, U2, P, W1, W2);
                else if constexpr (EPL) ray_trace_epl(X1, X2, U1, U2, P, W1, W2);
                else ray_trace(X1, X2, U1, U2, P, iq, W1, W2);
                const double r2s = source_r2(W1, W2, P.src);
                if constexpr (LENS && !DBL) {
                    val[0] = sersic_lg(log2_r2_sersic(fma(fma(P.lens.P, dx, rs), dx, rq), thr_l), el, Bl, lead, rnd);
                    val[1] = sersic_lg(log2_r2_sersic(r2s, thr_s), es, Bs, lead, rnd);
                } else {
                    const double lgs = log2_r2_sersic(r2s, thr_s);
                    val[IS] = sersic_lg(lgs, es, Bs, lead, rnd);
                    if constexpr (DBL) val[IS + 1] = sersic_lg(lgs + P.dlg_s, g.fix_e[3], g.fix_B[3], lead, rnd);
                }
            }
            if constexpr (LENS && (DBL || !SRC)) {
                const double lgl = log2_r2_sersic(fma(fma(P.lens.P, dx, rs), dx, rq), thr_l);
                val[0] = sersic_lg(lgl, el, Bl, lead, rnd);
                if constexpr (DBL) val[1] = sersic_lg(lgl + P.dlg_l, g.fix_e[1], g.fix_B[1], lead, rnd);
            }
        };
        double dx = dx0;
        int u = 0;
        // two sub-pixels per step (one-component and two-channel models, direct
        // deflection), with the positions and the order of the additions of one
        // at a time: measured +2% on the survey-scale lens (four channels would
        // spill; with the deflection table it measured 1.6% and 4% slower on the
        // batched and survey-scale lenses)
        for (; !DBL && !TAB && u + 2 <= s; u += 2) {
            const double dxb = dx + h;
            double va[N], vb[N];
            sub(dx, va);
            sub(dxb, vb);
#pragma unroll
            for (int c = 0; c < N; ++c) acc[c] += va[c];
#pragma unroll
            for (int c = 0; c < N; ++c) acc[c] += vb[c];
            dx = dxb + h;
        }
        for (; u < s; ++u) {
            double va[N];
            sub(dx, va);
#pragma unroll
            for (int c = 0; c < N; ++c) acc[c] += va[c];
            dx += h;
        }
    }
}

template <bool EPL = false, bool TAB = false>
__device__ __forceinline__ void binned_sums(const LensGeom &g, const PropBlock &P, int y, int x, double &al_out,
                                            double &as_out)
{
    double acc[2];
    binned_channels<LIGHT_BOTH, EPL, TAB>(g, P, y, x, acc);
    al_out = acc[0];
    as_out = acc[1];
}

template <bool EPL = false, bool TAB = false>
__device__ __forceinline__ float binned_pixel(const LensGeom &g, const PropBlock &P, int y, int x)
{
    double al, as;
    binned_sums<EPL, TAB>(g, P, y, x, al, as);
    return (float)(fma(P.lens.I, al, P.src.I * as) * g.inv_s2);
}

// The unit-amplitude channels of pixel (y, x) (binned values, FP32), for
// amplitudes solved by non-negative least squares (Sec. 2.3).
template <int LM, bool EPL = false, bool TAB = false>
__device__ __forceinline__ void binned_pixel_channels(const LensGeom &g, const PropBlock &P, int y, int x,
                                                      float (&ch)[LightChannels<LM>::N])
{
    double acc[LightChannels<LM>::N];
    binned_channels<LM, EPL, TAB>(g, P, y, x, acc);
#pragma unroll
    for (int c = 0; c < LightChannels<LM>::N; ++c) ch[c] = (float)(acc[c] * g.inv_s2);
}

// Sersic b_n: root of P(2n, b) = 1/2 (Eq. 9), FP64 Newton safeguarded by
// bisection on [0, 2n + 1].  P by its power series, which converges for every
// b in the bracket; the median of Gamma(2n) lies below 2n.  Host only (the
// fixed indices of two-component light); the device uses sersic_bn_fit.
__host__ inline double sersic_bn(double n)
{
    const double a = 2.0 * n;
    const double lga1 = lgamma(a + 1.0);
    double lo = 0.0, hi = a + 1.0;
    double x = a - 1.0 / 3.0 + 4.0 / (405.0 * n);
    if (!(x > lo && x < hi)) x = 0.5 * a;
    for (int it = 0; it < 200; ++it) {
        double term = 1.0, sum = 1.0, ap = a;
        for (int k = 0; k < 4000; ++k) {
            ap += 1.0;
            term *= x / ap;
            sum += term;
            if (term < sum * 1e-17) break;
        }
        const double pref = exp(a * log(x) - x - lga1);
        const double f = pref * sum - 0.5;
        if (f < 0.0) lo = x; else hi = x;
        const double dens = pref * a / x;  // d/dx P(a, x) = x^(a-1) e^-x / Gamma(a)
        double xn = x - f / dens;
        if (!(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
        const double dx = fabs(xn - x);
        x = xn;
        // Newton converges quadratically: after a step below 1e-9 relative the new
        // iterate is exact to rounding (~1e-15 from the series and exp); waiting for
        // a step below 4e-16 instead runs up to 11 iterations bouncing at the last ulp
        if (dx <= 1e-9 * x || hi - lo <= 4e-16 * x) break;
    }
    return x;
}

// b_n of Eq. 9 from the piecewise fit (lens_approx.h): the quarter-octave
// interval of n from an FP32 log2 (each interval's fit covers a rounding across
// its edges), then one degree-10 Horner pass in FP64; within 5e-15 relative of
// the root for n in [kNMin, kNMax], where the iteration above needs an
// incomplete-gamma series with a division per term at every Newton step.
__device__ __forceinline__ double sersic_bn_fit(double n)
{
    int j = (int)__builtin_floorf((float)kBnPerOctave * hw_log2((float)(n * (1.0 / kBnLo))));
    j = j < 0 ? 0 : j > kBnIntervals - 1 ? kBnIntervals - 1 : j;
    const double u = (n - kBnMid[j]) * kBnInvHalf[j];
    const double *c = kBnCoef[j];
    double r = c[kBnDeg];
#pragma unroll
    for (int i = kBnDeg - 1; i >= 0; --i) r = fma(r, u, c[i]);
    return r;
}

}  // namespace lensk
