// lens_strip.h -- device pieces shared by the likelihood kernels (gfx950): the LDS
// ring of binned rows, the strip sweep, the PSF convolutions over a strip and the
// amplitude solve.
//
// Forward model: Cao et al. (2025), Sec. 2.1 (Eqs. 1-3), Sec. 2.2 (Eq. 5), Sec. 2.3.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "lens_device.h"
#include "lens_internal.h"

namespace lensk {

// ---------------------------------------------------------------------------
// fused likelihood: shared pieces
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
// the matrix-core A operands in the global address space: their loads then
// count on vmcnt alone, and an LDS wait does not also wait for them
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4 *gptr4;
// and the B operands' LDS ring, kept in the LDS address space through arrays
typedef const __attribute__((address_space(3))) uint16_t *lptr16;
typedef const __attribute__((address_space(3))) u32x4 *lptr4;
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// round-to-nearest-even FP32 -> BF16 (finite inputs)
__device__ __forceinline__ uint16_t bf16_rn(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// How a binned value is kept in the LDS ring: FP32, or NPL BF16 planes whose
// sum is the value (hi, hi + lo, hi + mid + lo).  The FP16 split first keeps
// the FP32 value's upper and lower 16 bits in its two planes; once the row is
// complete, convert_rows_f16 turns them into half planes at the row's scale.
template <int MODE>
struct RingStore {
    static constexpr int NPL = mode_planes(MODE);
    __device__ static void put(void *ring, int plane, int idx, float v)
    {
        if (MODE == MODE_FP32) {
            static_cast<float *>(ring)[idx] = v;
        } else if (MODE == MODE_SPLIT) {
            uint16_t *b = static_cast<uint16_t *>(ring);
            const uint32_t u = __float_as_uint(v);
            b[idx] = (uint16_t)(u >> 16);
            b[plane + idx] = (uint16_t)u;
        } else {
            uint16_t *b = static_cast<uint16_t *>(ring);
            const uint16_t h = bf16_rn(v);
            b[idx] = h;
            if (NPL >= 2) {
                const float r1 = v - bf16_f(h);
                const uint16_t m = bf16_rn(r1);
                b[plane + idx] = m;
                if (NPL >= 3) b[2 * plane + idx] = bf16_rn(r1 - bf16_f(m));
            }
        }
    }
    __device__ static void zero(void *ring, int plane, int idx)
    {
        if (MODE == MODE_FP32) {
            static_cast<float *>(ring)[idx] = 0.0f;
        } else {
            uint16_t *b = static_cast<uint16_t *>(ring);
#pragma unroll
            for (int p = 0; p < NPL; ++p) b[p * plane + idx] = 0;
        }
    }
};

// Solved amplitudes: the ring holds one FP32 plane per unit-amplitude channel.
template <int NCH>
struct RingStoreN {
    __device__ static void put(void *ring, int plane, int idx, const float (&v)[NCH])
    {
#pragma unroll
        for (int c = 0; c < NCH; ++c) static_cast<float *>(ring)[c * plane + idx] = v[c];
    }
    __device__ static void zero(void *ring, int plane, int idx)
    {
#pragma unroll
        for (int c = 0; c < NCH; ++c) static_cast<float *>(ring)[c * plane + idx] = 0.0f;
    }
};
template <> struct RingStore<MODE_FP32N> : RingStoreN<2> {};
template <> struct RingStore<MODE_FP32N_LENS> : RingStoreN<1> {};
template <> struct RingStore<MODE_FP32N_SRC> : RingStoreN<1> {};
template <> struct RingStore<MODE_FP32N_DBL> : RingStoreN<4> {};
// the mass model does not change the ring
template <int MODE> struct RingStoreM : RingStore<mode_base(MODE)> {};

// FP16 split: per ring slot, the largest |value| of the row being filled (FP32
// bits, by atomic max) and, once converted, the factor 2^-j that undoes the
// row's scale.
__device__ __forceinline__ uint32_t *f16_rowmax()
{
    __shared__ uint32_t m[kRingRowsMax];
    return m;
}
__device__ __forceinline__ float *f16_rowscale()
{
    __shared__ float sc[kRingRowsMax];
    return sc;
}

// The power of two that brings a row whose largest |value| is m into
// [2^13, 2^14), and (inv) the one that undoes it.
__device__ __forceinline__ float f16_row_scale(float m, float &inv)
{
    int e = 0;
    (void)frexpf(m, &e);                       // m < 2^e
    e = m > 0.0f ? max(e, -100) : 14;          // tiny rows: the scale stays finite
    inv = ldexpf(1.0f, e - 14);
    return ldexpf(1.0f, 14 - e);
}

// The nearest half to v sc, and the nearest half to the remainder.
__device__ __forceinline__ void f16_halves(float v, float sc, uint16_t &hi, uint16_t &lo)
{
    v *= sc;
    const _Float16 h = (_Float16)v;
    const _Float16 l = (_Float16)(v - (float)h);
    hi = __builtin_bit_cast(uint16_t, h);
    lo = __builtin_bit_cast(uint16_t, l);
}

// Binned rows [ya, yb) of the FP16 split, complete in the ring as FP32 bits:
// each row scaled by the power of two 2^j that brings its largest |value|
// into [2^13, 2^14), and split into the nearest half h and the nearest half to
// the remainder.  The pair keeps 22 significant bits of every value from
// 2^-3 of the row's largest up; below, the remainder is subnormal and the
// absolute error stays under 2^-39 of the row's largest value.  One wave per
// row; the row's maximum is cleared for the slot's next row after the next
// barrier (clear_rowmax_f16).
template <int NT>
__device__ __forceinline__ void convert_rows_f16(const LensGeom &g, uint16_t *ring, int ya, int yb)
{
    const int W = g.ring_w, RB = g.ring_rows, lane = threadIdx.x & 63;
    for (int y = ya + (int)(threadIdx.x >> 6); y < yb; y += NT / 64) {
        const int slot = (y + g.r) % RB;
        const float m = __uint_as_float(f16_rowmax()[slot]);
        float inv;
        const float sc = f16_row_scale(m, inv);
        if (lane == 0) f16_rowscale()[slot] = inv;
        uint16_t *hi = ring + slot * W, *lo = hi + g.plane;
        for (int x = lane; x < W; x += 64) {
            f16_halves(__uint_as_float(((uint32_t)hi[x] << 16) | lo[x]), sc, hi[x], lo[x]);
        }
    }
}

template <int NT>
__device__ __forceinline__ void clear_rowmax_f16(const LensGeom &g, int ya, int yb)
{
    for (int y = ya + (int)threadIdx.x; y < yb; y += NT) f16_rowmax()[(y + g.r) % g.ring_rows] = 0u;
}

// Modes whose ray trace takes the deflection table (where q allows): all with
// a lensed source.
template <int MODE>
__host__ __device__ constexpr bool sie_tab()
{
    return mode_light(MODE) != LIGHT_LENS;
}

// Per-proposal tables into LDS, published by strip_sweep's first barrier.
template <int MODE>
__device__ __forceinline__ void tables_setup(const LensGeom &g, const PropBlock &P)
{
    if constexpr (sie_tab<MODE>()) {
        if constexpr (mode_epl(MODE)) {
            epl_setup(P);
            __syncthreads();
        }
        sie_setup<mode_epl(MODE)>(g, P);
    }
}

// Binned rows [ya, yb) (all < ny) into their ring slots: every pixel in the
// row's needed range is evaluated; the rest of the row is cleared when the
// slot is being reused (clear = true).  Ring column of image column x is
// x + r - xoff; columns outside the image are never written and stay zero.
template <int MODE, int NT>
__device__ __forceinline__ void fill_rows(const LensGeom &g, const PropBlock &P, void *ring,
                                          const uint32_t *__restrict__ evl, const int *__restrict__ evpre,
                                          const int2 *__restrict__ evr, int ya, int yb, bool clear)
{
    const int W = g.ring_w, RB = g.ring_rows, r = g.r, c0 = r - g.xoff;
    const int slot_a = (ya + r) % RB;  // rows [ya, yb) occupy consecutive slots modulo RB
    if (clear) {
        const int xa = max(0, -c0), xb = min(g.nx, W - c0);   // image columns that have ring columns
        for (int y = ya; y < yb; ++y) {
            int slot = slot_a + (y - ya);
            if (slot >= RB) slot -= RB;
            const int2 lr = evr[y];
            for (int x = xa + threadIdx.x; x < xb; x += NT)
                if (x < lr.x || x >= lr.y) RingStoreM<MODE>::zero(ring, g.plane, slot * W + c0 + x);
        }
    }
    const int fb = evpre[yb];
    // TAB: the SIE deflection from the proposal's table (a uniform branch)
    auto pixels = [&](auto tab) {
        constexpr bool TAB = decltype(tab)::value;
        for (int f = evpre[ya] + threadIdx.x; f < fb; f += NT) {
            const uint32_t e = evl[f];
            const int y = (int)(e >> 16), x = (int)(e & 0xffffu);
            int slot = slot_a + (y - ya);
            if (slot >= RB) slot -= RB;
            if constexpr (mode_solved(MODE)) {
                constexpr int NCH = mode_channels(MODE);
                float ch[NCH];
                binned_pixel_channels<mode_light(MODE), mode_epl(MODE), TAB>(g, P, y, x, ch);
                RingStoreM<MODE>::put(ring, g.plane, slot * W + c0 + x, ch);
            } else {
                const float v = binned_pixel<mode_epl(MODE), TAB>(g, P, y, x);
                RingStoreM<MODE>::put(ring, g.plane, slot * W + c0 + x, v);
                if constexpr (mode_base(MODE) == MODE_SPLIT) atomicMax(&f16_rowmax()[slot], __float_as_uint(fabsf(v)));
            }
        }
    };
    if (sie_tab<MODE>() && sie_use_table<mode_epl(MODE)>(g, P)) pixels(std::true_type{});
    else pixels(std::false_type{});
}

// The strip sweep of the fused kernels: binned rows enter the ring strip by
// strip, each binned row is computed once, and conv(y0, y1) takes the sums of
// output rows [y0, y1).
template <int MODE, int NT, typename Conv>
__device__ __forceinline__ void strip_sweep(const LensGeom &g, const PropBlock &P, void *ring,
                                            const uint32_t *__restrict__ evl, const int *__restrict__ evpre,
                                            const int2 *__restrict__ evr, Conv conv)
{
    const int ny = g.ny, r = g.r, H = g.strip_h, RB = g.ring_rows;
    const int nwords = (mode_base(MODE) == MODE_FP32 ? RB * g.ring_w
                        : mode_solved(MODE)            ? mode_channels(MODE) * RB * g.ring_w
                                                       : RB * g.ring_w * mode_planes(MODE) / 2) / 4;
    constexpr bool F16 = mode_base(MODE) == MODE_SPLIT;
    float4 *r4 = static_cast<float4 *>(ring);
    for (int i = threadIdx.x; i < nwords; i += NT) r4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (F16) {
        for (int i = threadIdx.x; i < RB; i += NT) {
            f16_rowmax()[i] = 0u;
            f16_rowscale()[i] = 1.0f;   // rows above the image stay zero at scale 1
        }
    }
    __syncthreads();
    // binned rows [0, r) precede the first strip
    fill_rows<MODE, NT>(g, P, ring, evl, evpre, evr, 0, min(r, ny), false);
    for (int y0 = 0; y0 < ny; y0 += H) {
        __syncthreads();  // the previous strip is done reading the slots reused below
        const int ya = y0 + r, yb = y0 + H + r;  // new binned rows
        if (y0 > 0) {
            const int c0 = r - g.xoff, xa = max(0, -c0), xb = min(g.nx, g.ring_w - c0);
            for (int y = max(ya, ny); y < yb; ++y) {  // rows past the image: clear reused slots
                const int slot = (y + r) % RB;
                for (int x = xa + threadIdx.x; x < xb; x += NT)
                    RingStoreM<MODE>::zero(ring, g.plane, slot * g.ring_w + c0 + x);
            }
        }
        if (ya < ny) fill_rows<MODE, NT>(g, P, ring, evl, evpre, evr, ya, min(yb, ny), y0 > 0);
        __syncthreads();
        if constexpr (F16) {
            // the rows that entered the ring since the last conversion, as halves
            const int ca = y0 == 0 ? 0 : ya;
            convert_rows_f16<NT>(g, static_cast<uint16_t *>(ring), ca, yb);
            __syncthreads();
            clear_rowmax_f16<NT>(g, ca, yb);   // read for the last time above
        }
        conv(y0, min(y0 + H, ny));
    }
}

// The sums of a proposal (chi-square, or the NNLS moments) in one order
// everywhere: each strip's per-thread sums through the wave64 shuffle tree,
// added strip by strip to the wave's sum (from zero), the waves' sums added in
// order at the end.  The split kernels keep the per-strip wave sums apart and
// add them in the same order, so that both give the same bits.
//
// Explicit amplitudes: lnL = C - chi^2 / 2.
template <int MODE, int NT, typename Conv>
__device__ __forceinline__ void strip_loop(const LensGeom &g, const PropBlock &P, void *ring,
                                           const uint32_t *__restrict__ evl, const int *__restrict__ evpre,
                                           const int2 *__restrict__ evr, double *__restrict__ out,
                                           int64_t p, Conv conv)
{
    __shared__ double red[NT / 64];
    tables_setup<MODE>(g, P);
    double tot = 0.0;
    strip_sweep<MODE, NT>(g, P, ring, evl, evpre, evr, [&](int y0, int y1) { tot += wave_sum(conv(y0, y1)); });
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < NT / 64; ++w) s += red[w];
        out[p] = g.norm - 0.5 * s;
    }
}

// Moments of the amplitude solve (Sec. 2.3) over the masked pixels, with the
// columns c_a of M (each light component at unit amplitude), the data d and
// the weights w = mask/sigma: F_ab = sum (w c_a)(w c_b) (upper triangle, row by
// row) and g_a = sum (w c_a)(w d).  FP64 sums of products of FP32 values.
template <int NCH>
struct MomN {
    static constexpr int NF = NCH * (NCH + 1) / 2, NM = NF + NCH;
    double m[NM];
    __device__ void add(const double (&c)[NCH], float d, float w)
    {
        double wc[NCH];
        const double wd = (double)w * (double)d;
#pragma unroll
        for (int a = 0; a < NCH; ++a) wc[a] = (double)w * c[a];
        int i = 0;
#pragma unroll
        for (int a = 0; a < NCH; ++a)
#pragma unroll
            for (int b = a; b < NCH; ++b, ++i) m[i] = fma(wc[a], wc[b], m[i]);
#pragma unroll
        for (int a = 0; a < NCH; ++a) m[NF + a] = fma(wc[a], wd, m[NF + a]);
    }
};

// Non-negative least squares in NCH <= 4 variables (Sec. 2.3): the minimiser of
// chi^2(s) = D - 2 s.g + s.F s over s >= 0 is the least-squares solution on one
// of the 2^NCH supports that is feasible and has the smallest chi^2; on a
// support S the optimum has F_S s_S = g_S, so chi^2 = D - s_S.g_S.  Each
// support's system is solved by Gaussian elimination with partial pivoting
// and skipped when singular (a pivot below 1e-13 of the largest diagonal
// entry).  nnls_support: chi^2 and the amplitudes (0 off the support) of the
// support S >= 1, or infinity where it is singular or infeasible.  (Its small
// arrays are indexed by the support's members, in scratch memory: with constant
// indices, in registers, the four-component kernel took 174 VGPRs and half its
// waves.)
template <int NCH>
__device__ inline double nnls_support(const MomN<NCH> &mo, double D, int S, double (&s)[NCH])
{
    constexpr int NF = MomN<NCH>::NF;
    double F[NCH][NCH];
    int i = 0;
    for (int a = 0; a < NCH; ++a)
        for (int b = a; b < NCH; ++b) F[a][b] = F[b][a] = mo.m[i++];
    double dmax = 0.0;
    for (int a = 0; a < NCH; ++a) dmax = fmax(dmax, fabs(F[a][a]));
    int idx[NCH], m = 0;
    for (int a = 0; a < NCH; ++a)
        if (S & (1 << a)) idx[m++] = a;
    double A[NCH][NCH], b[NCH], x[NCH];
    for (int r = 0; r < m; ++r) {
        b[r] = mo.m[NF + idx[r]];
        for (int c = 0; c < m; ++c) A[r][c] = F[idx[r]][idx[c]];
    }
    bool ok = dmax > 0.0;
    for (int col = 0; col < m && ok; ++col) {
        int piv = col;
        for (int r = col + 1; r < m; ++r)
            if (fabs(A[r][col]) > fabs(A[piv][col])) piv = r;
        if (!(fabs(A[piv][col]) > 1e-13 * dmax)) {
            ok = false;
            break;
        }
        if (piv != col) {
            for (int c = 0; c < m; ++c) {
                const double t = A[col][c];
                A[col][c] = A[piv][c];
                A[piv][c] = t;
            }
            const double t = b[col];
            b[col] = b[piv];
            b[piv] = t;
        }
        for (int r = col + 1; r < m; ++r) {
            const double f = A[r][col] / A[col][col];
            for (int c = col; c < m; ++c) A[r][c] -= f * A[col][c];
            b[r] -= f * b[col];
        }
    }
    if (!ok) return INFINITY;
    for (int r = m - 1; r >= 0; --r) {
        double acc = b[r];
        for (int c = r + 1; c < m; ++c) acc -= A[r][c] * x[c];
        x[r] = acc / A[r][r];
    }
    double sg = 0.0;
    for (int r = 0; r < m; ++r) {
        ok = ok && x[r] >= 0.0;
        sg += x[r] * mo.m[NF + idx[r]];
    }
    for (int a = 0; a < NCH; ++a) s[a] = 0.0;
    for (int r = 0; r < m; ++r) s[idx[r]] = x[r];
    return ok ? D - sg : INFINITY;
}

// The best support, one support per lane of a wave (all lanes hold the same
// moments): chi^2 (>= 0) and its amplitudes in every lane.  D = sum (wd)^2 is
// chi^2 of no light at all.  Of equal chi^2 the lowest support is taken.  One
// thread trying the 15 supports of four components in turn took 57 us.
template <int NCH>
__device__ __forceinline__ double nnls_wave(const MomN<NCH> &mo, double D, double (&best_s)[NCH])
{
    const int lane = threadIdx.x & 63;
    double s[NCH] = {}, c2 = INFINITY;
    int S = lane;
    if (lane >= 1 && lane < (1 << NCH)) c2 = nnls_support<NCH>(mo, D, lane, s);
    if (lane == 0 || !(c2 < D)) {   // no light; also where chi^2 is NaN or the support is out
        c2 = D;
        S = 0;
    }
    double best = c2;
#pragma unroll
    for (int off = 1; off < (1 << NCH); off <<= 1) {
        const double o = __shfl_xor(best, off, 64);
        const int so = __shfl_xor(S, off, 64);
        if (o < best || (o == best && so < S)) {
            best = o;
            S = so;
        }
    }
    best = __shfl(best, 0, 64);
    S = __shfl(S, 0, 64);
#pragma unroll
    for (int a = 0; a < NCH; ++a) best_s[a] = S ? __shfl(s[a], S, 64) : 0.0;
    return fmax(best, 0.0);
}

// Solved amplitudes: the moments reduced like the chi-square, then one wave
// solves and writes lnL = C - chi^2 / 2 (and, if amp is not null, the NCH
// amplitudes of proposal p at amp[NCH p ...]).
template <int MODE, int NT, typename Conv>
__device__ __forceinline__ void strip_loop_solved(const LensGeom &g, const PropBlock &P, void *ring,
                                                  const uint32_t *__restrict__ evl, const int *__restrict__ evpre,
                                                  const int2 *__restrict__ evr, double *__restrict__ out,
                                                  double *__restrict__ amp, int64_t p, Conv conv)
{
    constexpr int NCH = mode_channels(MODE), NM = MomN<NCH>::NM;
    __shared__ double red[NM][NT / 64];
    tables_setup<MODE>(g, P);
    if ((threadIdx.x & 63) == 0)
        for (int i = 0; i < NM; ++i) red[i][threadIdx.x >> 6] = 0.0;
    strip_sweep<MODE, NT>(g, P, ring, evl, evpre, evr, [&](int y0, int y1) {
        MomN<NCH> mo = conv(y0, y1);
#pragma unroll
        for (int i = 0; i < NM; ++i) mo.m[i] = wave_sum(mo.m[i]);
        if ((threadIdx.x & 63) == 0)
            for (int i = 0; i < NM; ++i) red[i][threadIdx.x >> 6] += mo.m[i];
    });
    __syncthreads();
    if (threadIdx.x < 64) {
        MomN<NCH> t{};
        for (int w = 0; w < NT / 64; ++w)
            for (int i = 0; i < NM; ++i) t.m[i] += red[i][w];
        double s[NCH];
        const double chi2 = nnls_wave<NCH>(t, g.dd, s);
        if (threadIdx.x == 0) {
            out[p] = g.norm - 0.5 * chi2;
            if (amp)
                for (int a = 0; a < NCH; ++a) amp[NCH * p + a] = s[a];
        }
    }
}

// ---------------------------------------------------------------------------
// FP32 PSF convolution on the vector ALU
// ---------------------------------------------------------------------------
// Four taps w on the outputs whose windows start at v.x .. v.w (u: the next
// four columns), in ascending order per output.
__device__ __forceinline__ void taps4(float (&p)[4], const float *w, const float4 &v, const float4 &u)
{
    p[0] = fmaf(w[0], v.x, p[0]); p[1] = fmaf(w[0], v.y, p[1]); p[2] = fmaf(w[0], v.z, p[2]); p[3] = fmaf(w[0], v.w, p[3]);
    p[0] = fmaf(w[1], v.y, p[0]); p[1] = fmaf(w[1], v.z, p[1]); p[2] = fmaf(w[1], v.w, p[2]); p[3] = fmaf(w[1], u.x, p[3]);
    p[0] = fmaf(w[2], v.z, p[0]); p[1] = fmaf(w[2], v.w, p[1]); p[2] = fmaf(w[2], u.x, p[2]); p[3] = fmaf(w[2], u.y, p[3]);
    p[0] = fmaf(w[3], v.w, p[0]); p[1] = fmaf(w[3], u.x, p[1]); p[2] = fmaf(w[3], u.y, p[2]); p[3] = fmaf(w[3], u.z, p[3]);
}

// The four horizontally adjacent convolved outputs x0 .. x0 + 3 of row y from
// one FP32 plane of the ring, PSF row by PSF row: each row's partial sum in
// FP32 (blocked summation), the partials added in FP64.  The window comes from
// LDS as aligned float4s, the weights through the scalar cache.  K: the PSF
// side, or 0 for the lens's own at run time; per output the same fmaf sequence
// either way, so that single-lens and multi-lens results agree bit for bit.
template <int K, typename Psf>
__device__ __forceinline__ void conv_window(const LensGeom &g, const float *ring, Psf psf, int y, int x0,
                                            double (&o)[4])
{
    const int k = K ? K : g.k, W4 = g.ring_w >> 2, RB = g.ring_rows;
    int slot = y % RB;   // ring slot of binned row y - r + a at a = 0
    const float4 *row = reinterpret_cast<const float4 *>(ring + slot * g.ring_w + x0 - g.xoff);
    int left = RB - slot;   // rows until the ring wraps
    o[0] = o[1] = o[2] = o[3] = 0.0;
#pragma unroll 1
    for (int a = 0; a < k; ++a) {
        const Psf kr = psf + a * k;
        float p[4] = {};
        if constexpr (K != 0) {
            constexpr int KC = (K + 6) / 4;
            // from the slot each time: a pointer that steps cost the fused kernels
            // their fifth wave
            row = reinterpret_cast<const float4 *>(ring + slot * g.ring_w + x0 - g.xoff);
            slot = slot + 1 == RB ? 0 : slot + 1;
            float win[4 * KC];
#pragma unroll
            for (int i = 0; i < KC; ++i) {
                const float4 t = row[i];
                win[4 * i + 0] = t.x;
                win[4 * i + 1] = t.y;
                win[4 * i + 2] = t.z;
                win[4 * i + 3] = t.w;
            }
#pragma unroll
            for (int b = 0; b < K; ++b) {
                const float w = kr[b];
#pragma unroll
                for (int j = 0; j < 4; ++j) p[j] = fmaf(w, win[b + j], p[j]);
            }
        } else {
            const float4 *q = row;
            float4 v = *q++;
            int b = 0;
            for (; b + 8 <= k; b += 8, q += 2) {
                const float4 u = q[0], t = q[1];
                const float w[8] = {kr[b], kr[b + 1], kr[b + 2], kr[b + 3], kr[b + 4], kr[b + 5], kr[b + 6], kr[b + 7]};
                taps4(p, w, v, u);
                taps4(p, w + 4, u, t);
                v = t;
            }
            if (b + 4 <= k) {
                const float4 u = *q++;
                const float w[4] = {kr[b], kr[b + 1], kr[b + 2], kr[b + 3]};
                taps4(p, w, v, u);
                v = u;
                b += 4;
            }
            // k is odd: one or three taps are left
            {
                const float w = kr[b];
                p[0] = fmaf(w, v.x, p[0]); p[1] = fmaf(w, v.y, p[1]); p[2] = fmaf(w, v.z, p[2]); p[3] = fmaf(w, v.w, p[3]);
            }
            if (b + 1 < k) {
                const float w1 = kr[b + 1], w2 = kr[b + 2];
                const float4 u = *q;
                p[0] = fmaf(w1, v.y, p[0]); p[1] = fmaf(w1, v.z, p[1]); p[2] = fmaf(w1, v.w, p[2]); p[3] = fmaf(w1, u.x, p[3]);
                p[0] = fmaf(w2, v.z, p[0]); p[1] = fmaf(w2, v.w, p[1]); p[2] = fmaf(w2, u.x, p[2]); p[3] = fmaf(w2, u.y, p[3]);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] += (double)p[j];
        if constexpr (K == 0) {
            row += W4;
            if (--left == 0) {
                row -= RB * W4;
                left = RB;
            }
        }
    }
}

// Chi-square contribution of output rows [ya, yb), four outputs per thread.
// tid: the thread's place among the NT that share the strip.
// K as for conv_window.
template <int K, int NT, typename Psf>
__device__ __forceinline__ double conv_rows(const LensGeom &g, const float *ring, Psf psf,
                                            const uint32_t *__restrict__ cvl, const int *__restrict__ cvpre,
                                            const float *__restrict__ data, const float *__restrict__ wgt,
                                            int ya, int yb, int tid)
{
    double acc = 0.0;
    const int gb = cvpre[yb];
    for (int gi = cvpre[ya] + tid; gi < gb; gi += NT) {
        const uint32_t e = cvl[gi];
        const int y = (int)(e >> 16), x0 = (int)(e & 0xffffu);
        double o[4];
        conv_window<K>(g, ring, psf, y, x0, o);
        const float4 d = *reinterpret_cast<const float4 *>(data + (size_t)y * g.pitch + x0);
        const float4 w = *reinterpret_cast<const float4 *>(wgt + (size_t)y * g.pitch + x0);
        const double r0 = ((double)d.x - o[0]) * (double)w.x;
        const double r1 = ((double)d.y - o[1]) * (double)w.y;
        const double r2 = ((double)d.z - o[2]) * (double)w.z;
        const double r3 = ((double)d.w - o[3]) * (double)w.w;
        acc = fma(r0, r0, acc);
        acc = fma(r1, r1, acc);
        acc = fma(r2, r2, acc);
        acc = fma(r3, r3, acc);
    }
    return acc;
}

// Solved amplitudes: the channels convolved one after another (their window
// reads stay free of bank conflicts, and the registers of one channel serve
// all), and the moments of the amplitude solve accumulated in FP64 from the
// FP32 columns, data and weights.
template <int MODE, int NT, int K, typename Psf>
__device__ __forceinline__ MomN<mode_channels(MODE)> conv_rows_solved(const LensGeom &g, const float *ring, Psf psf,
                                                                      int ya, int yb, int tid)
{
    constexpr int NCH = mode_channels(MODE);
    MomN<NCH> mo{};
    const int gb = g.cvpre[yb];
    for (int gi = g.cvpre[ya] + tid; gi < gb; gi += NT) {
        const uint32_t e = g.cvl[gi];
        const int y = (int)(e >> 16), x0 = (int)(e & 0xffffu);
        double o[4][NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            double oc[4];
            conv_window<K>(g, ring + c * g.plane, psf, y, x0, oc);
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j][c] = oc[j];
        }
        const float4 d = *reinterpret_cast<const float4 *>(g.data + (size_t)y * g.pitch + x0);
        const float4 w = *reinterpret_cast<const float4 *>(g.wgt + (size_t)y * g.pitch + x0);
        mo.add(o[0], d.x, w.x);
        mo.add(o[1], d.y, w.y);
        mo.add(o[2], d.z, w.z);
        mo.add(o[3], d.w, w.w);
    }
    return mo;
}

// ---------------------------------------------------------------------------
// PSF convolution as a matrix-core contraction
// ---------------------------------------------------------------------------
// For a segment of 16 outputs x0..x0+15 of row y,
//   out[x0 + j] = sum_{a, i} T_a[j, i] w_a[i],  T_a[j, i] = Kf[a][i - j] (0 <= i - j < k),
//   w_a[i] = binned[y - r + a][x0 - r + i],  i < L (window_len: 16 + k - 1 rounded up),
// i.e. C = A B with A the banded Toeplitz expansion of the flipped PSF
// (16 x kL, built once per lens) and the B column of a segment its stacked
// PSF-row windows.  One v_mfma_f32_16x16x32_{bf16,f16} takes 32 of the kL
// products for 16 segments at once.  Operand layout (wave64): lane l holds A
// row l%16, B column l%16, K elements 8(l/16)..8(l/16)+7 of the 32; D rows
// 4(l/16)..+3 of column l%16.  The BF16 split3 forms the six products of three
// planes that reach 2^-24; the FP16 split is RowsF16.
template <int MODE>
__device__ __forceinline__ f32x4 mfma_products(const bf16x8 (&a)[3], const bf16x8 (&b)[3], f32x4 c)
{
    if (mode_base(MODE) == MODE_SPLIT3) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], c, 0, 0, 0);
    }
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], c, 0, 0, 0);
}

// The FP32 accumulator of the contraction is added into FP64 sums every
// kFlushChunks K-chunks: summed over all k L products in FP32, an output
// collects a rounding error at every accumulate step relative to its whole
// running sum, which reached ~5e-7 of the lnL error metric on the 200x200 /
// 41x41 workload; flushed, each FP32 partial is a short sum.
constexpr int kFlushChunks = 2;

// NTL tiles of 16 segments starting at segment t (tile j: t + 16 j ..), with
// one load of each A chunk shared by the tiles: per output the same products
// in the same order as a tile alone.  Lanes past the strip's last segment s1
// compute a discarded column.  Returns this lane's chi-square contribution.
template <int MODE, int NTL>
__device__ __forceinline__ double conv_tiles(const LensGeom &g, const uint16_t *ring, const uint4 *__restrict__ aop,
                                             const uint32_t *__restrict__ seg, const float *__restrict__ data,
                                             const float *__restrict__ wgt, int t, int s0, int s1)
{
    constexpr int NPL = mode_planes(MODE);
    const int lane = threadIdx.x & 63, n = lane & 15, kb = lane >> 4;
    const int W = g.ring_w, RB = g.ring_rows, L = g.L, nch = g.nchunks, plane = g.plane;
    int i = 8 * kb, adv = 0;     // window offset of this lane's K elements (K = 8 kb), and the rows it skips
    while (i >= L) {             // (only for L < 32)
        i -= L;
        ++adv;
    }
    bool dummy[NTL];
    int y[NTL], x0[NTL], slot[NTL];
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
        dummy[j] = t + 16 * j + n >= s1;
        const uint32_t e = dummy[j] ? seg[s0] : seg[t + 16 * j + n];
        y[j] = (int)(e >> 16);
        x0[j] = (int)(e & 0xffffu);
        slot[j] = (y[j] % RB + adv) % RB;   // ring slot of binned row y - r + a
    }
    double o[NTL][4] = {};       // outputs 4 kb .. 4 kb + 3 of column n, FP64
    gptr4 ap = (gptr4)aop + lane;
    for (int ch0 = 0; ch0 < nch; ch0 += kFlushChunks) {
        f32x4 c[NTL];
#pragma unroll
        for (int j = 0; j < NTL; ++j) c[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int ch1 = min(ch0 + kFlushChunks, nch);
        for (int ch = ch0; ch < ch1; ++ch) {
            bf16x8 av[3];
#pragma unroll
            for (int q = 0; q < NPL; ++q) av[q] = __builtin_bit_cast(bf16x8, ap[q * 64]);
#pragma unroll
            for (int j = 0; j < NTL; ++j) {
                bf16x8 bv[3];
                const uint16_t *bp = ring + (x0[j] - g.xoff) + slot[j] * W + i;
#pragma unroll
                for (int q = 0; q < NPL; ++q)
                    bv[q] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(bp + q * plane));
                c[j] = mfma_products<MODE>(av, bv, c[j]);
            }
            ap += NPL * 64;
            i += 32;
            while (i >= L) {
                i -= L;
#pragma unroll
                for (int j = 0; j < NTL; ++j) slot[j] = slot[j] + 1 == RB ? 0 : slot[j] + 1;
            }
        }
#pragma unroll
        for (int j = 0; j < NTL; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) o[j][v] += (double)c[j][v];
    }
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
        if (dummy[j]) continue;
        const int xo = x0[j] + 4 * kb;
        const float4 d = *reinterpret_cast<const float4 *>(data + (size_t)y[j] * g.pitch + xo);
        const float4 w = *reinterpret_cast<const float4 *>(wgt + (size_t)y[j] * g.pitch + xo);
        const double r0 = ((double)d.x - o[j][0]) * (double)w.x;
        const double r1 = ((double)d.y - o[j][1]) * (double)w.y;
        const double r2 = ((double)d.z - o[j][2]) * (double)w.z;
        const double r3 = ((double)d.w - o[j][3]) * (double)w.w;
        acc = fma(r0, r0, acc);
        acc = fma(r1, r1, acc);
        acc = fma(r2, r2, acc);
        acc = fma(r3, r3, acc);
    }
    return acc;
}

// The FP16 split: the PSF (scaled by 2^j, conv_scale = 2^-j) and each ring row
// (at its own scale) as hi + lo halves, three products a_hi b_lo + a_lo b_hi +
// a_hi b_hi per tap (the dropped a_lo b_lo and both truncations are each below
// 2^-22 of the tap's product).  A PSF row's window is CPR = L / 32 whole
// K-chunks of one ring row, so the FP32 partial of each PSF row is flushed to
// the FP64 output times the two scales, exactly (powers of two).
//
// A tile is 16 segments of kRowGroup = 4 output rows y .. y + 3 (column n of the
// tile: segment t + n of the list).  Ring row y - r + a meets PSF row a - j for
// output row y + j, so rows of a tile share the B operands read from LDS, and
// each PSF row's A operands, loaded once, serve all of them.  The split kernels
// take the four rows at once; the fused kernels, whose ray trace leaves no
// registers for several sets of A operands (with two sets the multi-lens kernel
// took 176 VGPRs and half its waves), take pairs of rows, which also spreads a
// strip over all their waves.  With two tiles of one row each (the A operands
// shared, B read for every row) the LDS reads of B were the bound of the split
// kernel: 0.73 of 0.75 ms for 2,048 proposals of 200x200 px, 41x41 PSF; with
// pairs of rows, the loads of A from the L1, 0.50 of 0.54 ms; with four rows it
// takes 0.41 ms.  Lanes past the strip's last segment s1 compute a discarded
// column.  Same operand layout and output mapping as conv_tiles.
template <int CPR>
struct RowsF16 {
    const LensGeom &g;
    gptr4 ap;
    lptr16 bp;
    int slot, y, x0;
    bool dummy;

    // from output row j of the tile at segment t
    __device__ __forceinline__ RowsF16(const LensGeom &g, const uint16_t *ring, const uint4 *__restrict__ aop,
                                       const uint32_t *__restrict__ seg, int t, int s0, int s1, int j)
        : g(g), ap((gptr4)aop + (threadIdx.x & 63))
    {
        const int lane = threadIdx.x & 63, n = lane & 15, kb = lane >> 4;
        dummy = t + n >= s1;
        const uint32_t e = seg[dummy ? s0 : t + n];
        y = (int)(e >> 16) + j;
        x0 = (int)(e & 0xffffu);
        slot = y % g.ring_rows;   // ring slot of binned row y - r
        bp = (lptr16)ring + slot * g.ring_w + (x0 - g.xoff) + 8 * kb;
    }
    // the next ring row's B operands; returns its scale
    __device__ __forceinline__ double load_b(f16x8 (&b)[2 * CPR])
    {
#pragma unroll
        for (int h = 0; h < CPR; ++h) {
            b[2 * h] = __builtin_bit_cast(f16x8, *(lptr4)(bp + 32 * h));
            b[2 * h + 1] = __builtin_bit_cast(f16x8, *(lptr4)(bp + 32 * h + g.plane));
        }
        const double sc = (double)f16_rowscale()[slot] * g.conv_scale;
        bp += g.ring_w;
        if (++slot == g.ring_rows) {
            slot = 0;
            bp -= g.ring_rows * g.ring_w;
        }
        return sc;
    }
    // the next PSF row's A operands
    __device__ __forceinline__ void load_a(f16x8 (&a)[2 * CPR])
    {
#pragma unroll
        for (int h = 0; h < 2 * CPR; ++h) a[h] = __builtin_bit_cast(f16x8, ap[h * 64]);
        ap += 2 * CPR * 64;
    }
    static __device__ __forceinline__ void row(const f16x8 (&a)[2 * CPR], const f16x8 (&b)[2 * CPR], double sc,
                                               double (&out)[4])
    {
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int h = 0; h < CPR; ++h) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[2 * h], b[2 * h + 1], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[2 * h + 1], b[2 * h], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[2 * h], b[2 * h], c, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) out[v] = fma((double)c[v], sc, out[v]);
    }
    // chi-square of output row y + j: outputs 4 kb .. 4 kb + 3 of column n
    __device__ __forceinline__ double residual(const float *__restrict__ data, const float *__restrict__ wgt, int j,
                                               int yb, const double (&o)[4], double acc) const
    {
        if (dummy || y + j >= yb) return acc;
        const size_t at = (size_t)(y + j) * g.pitch + x0 + 4 * ((threadIdx.x & 63) >> 4);
        const float4 d = *reinterpret_cast<const float4 *>(data + at);
        const float4 w = *reinterpret_cast<const float4 *>(wgt + at);
        const double r0 = ((double)d.x - o[0]) * (double)w.x;
        const double r1 = ((double)d.y - o[1]) * (double)w.y;
        const double r2 = ((double)d.z - o[2]) * (double)w.z;
        const double r3 = ((double)d.w - o[3]) * (double)w.w;
        acc = fma(r0, r0, acc);
        acc = fma(r1, r1, acc);
        acc = fma(r2, r2, acc);
        acc = fma(r3, r3, acc);
        return acc;
    }
};

// Rows j and j + 1 of a tile, added to acc: each ring row's B operands are kept
// for the second row's step (PSF rows of three K-chunks, k > 49: one output row
// after the other, which keeps the registers at the two-chunk level).
template <int CPR>
__device__ __forceinline__ double conv_pair_f16(const LensGeom &g, const uint16_t *ring, const uint4 *__restrict__ aop,
                                                const uint32_t *__restrict__ seg, const float *__restrict__ data,
                                                const float *__restrict__ wgt, int t, int s0, int s1, int j, int yb,
                                                double acc)
{
    if constexpr (CPR > 2) {
#pragma unroll 1
        for (int i = j; i < j + 2; ++i) {
            RowsF16<CPR> R(g, ring, aop, seg, t, s0, s1, i);
            double o[4] = {};
#pragma unroll 1
            for (int a = 0; a < g.k; ++a) {
                f16x8 av[2 * CPR], b[2 * CPR];
                R.load_a(av);
                const double c = R.load_b(b);
                R.row(av, b, c, o);
            }
            acc = R.residual(data, wgt, 0, yb, o, acc);
        }
        return acc;
    }
    RowsF16<CPR> R(g, ring, aop, seg, t, s0, s1, j);
    double o0[4] = {}, o1[4] = {};
    f16x8 b0[2 * CPR], b1[2 * CPR];
    double c0 = R.load_b(b0), c1;
#pragma unroll 1
    for (int a = 0; a < g.k; a += 2) {
        f16x8 av[2 * CPR];
        R.load_a(av);
        c1 = R.load_b(b1);
        R.row(av, b0, c0, o0);
        R.row(av, b1, c1, o1);
        if (a + 1 == g.k) break;
        R.load_a(av);
        c0 = R.load_b(b0);
        R.row(av, b1, c1, o0);
        R.row(av, b0, c0, o1);
    }
    acc = R.residual(data, wgt, 0, yb, o0, acc);
    return R.residual(data, wgt, 1, yb, o1, acc);
}

// All rows of a tile: the first two added to acc[0], the others to acc[1].
template <int CPR>
__device__ __forceinline__ void conv_quad_f16(const LensGeom &g, const uint16_t *ring, const uint4 *__restrict__ aop,
                                              const uint32_t *__restrict__ seg, const float *__restrict__ data,
                                              const float *__restrict__ wgt, int t, int s0, int s1, int yb,
                                              double (&acc)[2])
{
    constexpr int T = kRowGroup;
    RowsF16<CPR> R(g, ring, aop, seg, t, s0, s1, 0);
    // A operands of PSF row a in av[a % T]: loaded at step a - 1, after the last
    // use of row a - T's
    f16x8 av[T][2 * CPR];
    double o[T][4] = {};
    const int k = g.k;
    R.load_a(av[0]);
    const auto step = [&](auto ph, int a) {
        constexpr int PH = decltype(ph)::value;   // a % T
        if (a >= k + T - 1) return;
        f16x8 b[2 * CPR];
        const double sc = R.load_b(b);
#pragma unroll
        for (int j = T - 1; j >= 0; --j) {
            if (a - j >= 0 && a - j < k) R.row(av[(PH - j + T) % T], b, sc, o[j]);
            if (j == T - 1 && a + 1 < k) R.load_a(av[(PH + 1) % T]);
        }
    };
#pragma unroll 1
    for (int a = 0; a < k + T - 1; a += T) {
        step(std::integral_constant<int, 0>{}, a);
        step(std::integral_constant<int, 1>{}, a + 1);
        step(std::integral_constant<int, 2>{}, a + 2);
        step(std::integral_constant<int, 3>{}, a + 3);
    }
#pragma unroll
    for (int j = 0; j < T; ++j) acc[j / 2] = R.residual(data, wgt, j, yb, o[j], acc[j / 2]);
}

// Chi-square contribution of output rows [ya, yb): each wave takes two tiles
// of 16 segments at a time (one where only one is left), so that every A
// chunk loaded from L2 feeds two matrix-core products; in the FP16 split, one
// pair of rows of a tile.
template <int MODE, int NT>
__device__ __forceinline__ double conv_mfma(const LensGeom &g, const uint16_t *ring,
                                            const uint4 *__restrict__ aop, const uint32_t *__restrict__ seg,
                                            const int *__restrict__ segpre, const float *__restrict__ data,
                                            const float *__restrict__ wgt, int ya, int yb, int tid)
{
    const int wave = tid >> 6;
    double acc = 0.0;
    const int s0 = segpre[ya], s1 = segpre[yb];
    if constexpr (mode_base(MODE) == MODE_SPLIT) {
        // K-chunks per PSF row: window_len(k) / 32, at most 3 (k <= 63)
        const int cpr = g.L >> 5;
        for (int p = wave;; p += NT / 64) {
            const int t = s0 + 16 * (p >> 1), j = 2 * (p & 1);
            if (t >= s1) break;
            if (cpr == 2) acc = conv_pair_f16<2>(g, ring, aop, seg, data, wgt, t, s0, s1, j, yb, acc);
            else if (cpr == 1) acc = conv_pair_f16<1>(g, ring, aop, seg, data, wgt, t, s0, s1, j, yb, acc);
            else acc = conv_pair_f16<3>(g, ring, aop, seg, data, wgt, t, s0, s1, j, yb, acc);
        }
    } else {
        for (int t = s0 + 32 * wave; t < s1; t += 32 * (NT / 64)) {
            if (t + 16 < s1) acc += conv_tiles<MODE, 2>(g, ring, aop, seg, data, wgt, t, s0, s1);
            else acc += conv_tiles<MODE, 1>(g, ring, aop, seg, data, wgt, t, s0, s1);
        }
    }
    return acc;
}

// conv_mfma of the FP16 split over half the waves, tile by tile: wave w gives
// the sums of conv_mfma's waves 2 w and 2 w + 1.
template <int NT>
__device__ __forceinline__ void conv_mfma_quads(const LensGeom &g, const uint16_t *ring, int ya, int yb, int wave,
                                                double (&acc)[2])
{
    static_assert(kRowGroup == 4, "two pairs of rows");
    acc[0] = acc[1] = 0.0;
    const int s0 = g.segpre[ya], s1 = g.segpre[yb], cpr = g.L >> 5;
    for (int t = s0 + 16 * wave; t < s1; t += 16 * (NT / 128)) {
        if (cpr == 2) conv_quad_f16<2>(g, ring, g.aop, g.seg, g.data, g.wgt, t, s0, s1, yb, acc);
        else if (cpr == 1) conv_quad_f16<1>(g, ring, g.aop, g.seg, g.data, g.wgt, t, s0, s1, yb, acc);
        else conv_quad_f16<3>(g, ring, g.aop, g.seg, g.data, g.wgt, t, s0, s1, yb, acc);
    }
}

}  // namespace lensk
