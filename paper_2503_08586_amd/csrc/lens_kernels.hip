// lens_kernels.hip -- HIP kernels of the batched lens log-likelihood (gfx950).
//
// k_prep          one thread per proposal: domain check, FP64 b_n, derived constants.
// k_loglike_fp32  one workgroup per proposal: the whole forward model and the
//                 chi-square in one pass, the binned image never leaving LDS;
//                 PSF convolution on the vector ALU in FP32.
// k_loglike_mfma  the same with the PSF convolution as a BF16 matrix-core
//                 contraction (plain, hi+lo split or hi+mid+lo split operands).
// k_model_*       debug: full model images of one proposal.
//
// Forward model: Cao et al. (2025), Sec. 2.1 (Eqs. 1-3), Sec. 2.2 (Eq. 5), Sec. 2.4.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "lens_device.h"
#include "lens_internal.h"
#include "lens_prep.h"
#include "lens_strip.h"

namespace lensk {

// ---------------------------------------------------------------------------
// prep
// ---------------------------------------------------------------------------
// One thread per proposal; the light model of proposal i is `model`, or, with
// a per-lens table, that of the lens owning i.
__global__ void __launch_bounds__(256) k_prep(const double *__restrict__ params, int64_t n, PropBlock *__restrict__ pc,
                                              int model, const int64_t *__restrict__ pstart,
                                              const int *__restrict__ pmodel, int nl)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int lm = model;
    if (pstart) {
        int lo = 0, hi = nl;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pstart[mid] <= i) lo = mid; else hi = mid;
        }
        lm = pmodel[lo];
    }
    const double *p = params + i * kStride;
    double v[kStride];
#pragma unroll
    for (int j = 0; j < kStride; ++j) v[j] = p[j];
    pc[i] = prep_proposal(v, lm);
}

// ---------------------------------------------------------------------------
// fused likelihood: one workgroup per proposal
// ---------------------------------------------------------------------------
// Waves per SIMD that a fused kernel must leave room for: four where the
// compiler would take more than 128 registers beside the multi-lens bookkeeping,
// since workgroups of eight waves then leave a CU with one of them, two waves per
// SIMD.  A few registers go to memory instead.  The FP16 split's row pairs: 25.1 ms
// for 16 x 1,000 proposals of 200x200 px at 151 registers, 18.6 held to 128; two
// components per galaxy: 9.5 and 6.4 ms for 4 x 1,024 of 128x128 px; the power
// law, whose table and series both need theirs: BF16 4.7 and 3.5 ms, below the
// table's axis ratios 38.7 and 22.9.
template <int MODE>
constexpr int fused_waves()
{
    return mode_base(MODE) == MODE_SPLIT || mode_base(MODE) == MODE_FP32N_DBL ||
                   (mode_epl(MODE) && mode_base(MODE) != MODE_FP32N_SRC)
               ? 4
               : 1;
}

template <int MODE, int NT>
__global__ void __launch_bounds__(NT, fused_waves<MODE>())
k_loglike_mfma(const LensGeom g, const PropBlock *__restrict__ pc, const uint32_t *__restrict__ evl,
               const int *__restrict__ evpre, const int2 *__restrict__ evr, const uint4 *__restrict__ aop,
               const uint32_t *__restrict__ seg, const int *__restrict__ segpre, const float *__restrict__ data,
               const float *__restrict__ wgt, double *__restrict__ out)
{
    extern __shared__ float4 lds4[];
    uint16_t *ring = reinterpret_cast<uint16_t *>(lds4);
    const int64_t p = blockIdx.x;
    const PropBlock *c = pc + p;
    if (c->valid != 1.0) {
        if (threadIdx.x == 0) out[p] = -INFINITY;
        return;
    }
    const PropBlock P = *c;
    strip_loop<MODE, NT>(g, P, ring, evl, evpre, evr, out, p, [&](int y0, int y1) {
        return conv_mfma<MODE, NT>(g, ring, aop, seg, segpre, data, wgt, y0, y1, threadIdx.x);
    });
}

// Light amplitudes solved by NNLS (Sec. 2.3), for the light model of MODE: one
// workgroup per proposal, the NCH channels through the LDS ring and the FP32
// convolution, the moments reduced and the problem solved in the workgroup.
// amp (may be null): [n][NCH].
template <int MODE, int NT>
__global__ void __launch_bounds__(NT)
k_loglike_nnls(const LensGeom g, const PropBlock *__restrict__ pc, double *__restrict__ out,
               double *__restrict__ amp)
{
    constexpr int NCH = mode_channels(MODE);
    extern __shared__ float4 lds4[];
    float *ring = reinterpret_cast<float *>(lds4);
    const int64_t p = blockIdx.x;
    const PropBlock *c = pc + p;
    if (c->valid == 0.0) {
        if (threadIdx.x == 0) {
            out[p] = -INFINITY;
            if (amp)
                for (int a = 0; a < NCH; ++a) amp[NCH * p + a] = NAN;
        }
        return;
    }
    const PropBlock P = *c;
    strip_loop_solved<MODE, NT>(g, P, ring, g.evl, g.evpre, g.evr, out, amp, p, [&](int y0, int y1) {
        return conv_rows_solved<MODE, NT, 0>(g, ring, g.psf, y0, y1, threadIdx.x);
    });
}

// Explicit amplitudes, FP32 convolution.  K: the PSF side as a constant, or 0.
// With a constant side a PSF row's weights and window are loaded in one go and
// the kernel holds five waves per SIMD: 5.59 against 5.95 ms for 8,192 proposals
// of 128x128 px at side 13, 6.7 against 6.9 at 21.  Beyond 31 a row's weights no
// longer fit the scalar registers that the ray trace leaves (16.0 against 13.3
// ms at 200x200 px, side 41).  The pointers of the constant-side kernels are
// arguments of their own: from the descriptor they took the fifth wave again
// (5.7 ms); at run-time sides it is the other way round (14.3 against 13.3 ms).
// A call of at most three workgroups per CU, which waits for single workgroups,
// takes the constant sides up to 63 all the same: 64 proposals of 96x96 px at side 41
// 311 us, 536 at the run-time side; 512 495 and 608; 768 670 and 704; 4,096 the other
// way round.
// The power law's longer ray trace leaves no room for a constant side (3.84 against
// 3.85 ms for 4,096 proposals at side 21).
template <int MODE, int NT, int K>
__global__ void __launch_bounds__(NT, K ? 1 : NT == 256 ? 5 : 4)
k_loglike_fp32(const LensGeom g, const PropBlock *__restrict__ pc, const float *__restrict__ psf,
               const uint32_t *__restrict__ evl, const int *__restrict__ evpre, const int2 *__restrict__ evr,
               const uint32_t *__restrict__ cvl, const int *__restrict__ cvpre, const float *__restrict__ data,
               const float *__restrict__ wgt, double *__restrict__ out)
{
    extern __shared__ float4 lds4[];
    float *ring = reinterpret_cast<float *>(lds4);
    const int64_t p = blockIdx.x;
    const PropBlock *c = pc + p;
    if (c->valid != 1.0) {
        if (threadIdx.x == 0) out[p] = -INFINITY;
        return;
    }
    const PropBlock P = *c;
    if constexpr (K != 0)
        strip_loop<MODE, NT>(g, P, ring, evl, evpre, evr, out, p, [&](int y0, int y1) {
            return conv_rows<K, NT>(g, ring, psf, cvl, cvpre, data, wgt, y0, y1, threadIdx.x);
        });
    else
        strip_loop<MODE, NT>(g, P, ring, g.evl, g.evpre, g.evr, out, p, [&](int y0, int y1) {
            return conv_rows<0, NT>(g, ring, g.psf, g.cvl, g.cvpre, g.data, g.wgt, y0, y1, threadIdx.x);
        });
}

__global__ void k_reset_counter(unsigned int *counter) { *counter = 0u; }

// Work items are (lens, proposal) pairs numbered lens-major in the batch's
// order (longest per-proposal cost first); item i belongs to the lens j with
// lstart[j] <= i < lstart[j + 1], and its result goes to out[lout[j] + i - lstart[j]].
// Each workgroup takes the next item from a global counter until none is left:
// every wave leaves the loop on the same item index, so the grid drains.
template <int MODE, int NT>
__global__ void __launch_bounds__(NT, fused_waves<MODE>())
k_loglike_batch(const LensGeom *__restrict__ geoms, const int *__restrict__ lstart,
                const int64_t *__restrict__ lout, int nl, int nitems, const PropBlock *__restrict__ pc,
                double *__restrict__ out, unsigned int *__restrict__ counter)
{
    extern __shared__ float4 lds4[];
    __shared__ int s_item;
    // a workgroup never takes more than nitems items: the cap bounds the loop
    // even if the counter protocol were broken
    for (int iter = 0; iter <= nitems; ++iter) {
        if (threadIdx.x == 0) s_item = (int)atomicAdd(counter, 1u);
        __syncthreads();
        // uniform across the workgroup: readfirstlane lets the compiler keep the
        // lens descriptor and the proposal constants in scalar registers
        const int item = __builtin_amdgcn_readfirstlane(s_item);
        __syncthreads();
        if (item >= nitems) break;
        int lo = 0, hi = nl;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (lstart[mid] <= item) lo = mid; else hi = mid;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        const LensGeom g = geoms[lo];
        const int64_t p = lout[lo] + (item - lstart[lo]);
        const PropBlock *c = pc + p;
        if (mode_solved(MODE) ? c->valid == 0.0 : c->valid != 1.0) {
            if (threadIdx.x == 0) out[p] = -INFINITY;
        } else {
            const PropBlock P = *c;
            if constexpr (mode_solved(MODE)) {
                float *ring = reinterpret_cast<float *>(lds4);
                strip_loop_solved<MODE, NT>(g, P, ring, g.evl, g.evpre, g.evr, out, nullptr, p,
                                            [&](int y0, int y1) { return conv_rows_solved<MODE, NT, 0>(g, ring, g.psf, y0, y1, threadIdx.x); });
            } else if (mode_base(MODE) == MODE_FP32) {
                float *ring = reinterpret_cast<float *>(lds4);
                strip_loop<MODE, NT>(g, P, ring, g.evl, g.evpre, g.evr, out, p, [&](int y0, int y1) {
                    return conv_rows<0, NT>(g, ring, g.psf, g.cvl, g.cvpre, g.data, g.wgt, y0, y1, threadIdx.x);
                });
            } else {
                uint16_t *ring = reinterpret_cast<uint16_t *>(lds4);
                strip_loop<MODE, NT>(g, P, ring, g.evl, g.evpre, g.evr, out, p, [&](int y0, int y1) {
                    return conv_mfma<MODE, NT>(g, ring, g.aop, g.seg, g.segpre, g.data, g.wgt, y0, y1, threadIdx.x);
                });
            }
        }
        // Reconverge before thread 0 takes the next item.  Without this barrier
        // the thread-0 result store above and the thread-0 atomic at the top of
        // the loop can be merged into one divergent region spanning the back
        // edge, and the other lanes would pass the next barrier before the new
        // item has been published.
        __syncthreads();
    }
}

template <bool F16>
__global__ void k_mfma_probe(const uint16_t *__restrict__ a, const uint16_t *__restrict__ b, float *__restrict__ d)
{
    // a: 16 x 32 row-major, b: 32 x 16 row-major, d: 16 x 16 row-major; one wave;
    // BF16 or (F16) IEEE-half operands
    const int l = threadIdx.x, n = l & 15, kb = l >> 4;
    uint16_t ta[8], tb[8];
    for (int e = 0; e < 8; ++e) {
        ta[e] = a[n * 32 + 8 * kb + e];
        tb[e] = b[(8 * kb + e) * 16 + n];
    }
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    if constexpr (F16)
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, *reinterpret_cast<const uint4 *>(ta)),
                                                   __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4 *>(tb)), c,
                                                   0, 0, 0);
    else
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(ta)),
                                                    __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(tb)),
                                                    c, 0, 0, 0);
    for (int v = 0; v < 4; ++v) d[(4 * kb + v) * 16 + n] = c[v];
}

// ---------------------------------------------------------------------------
// debug model images
// ---------------------------------------------------------------------------
template <bool EPL>
__global__ void k_model_binned(const LensGeom g, const PropBlock *__restrict__ pc, float *__restrict__ img)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const PropBlock P = *pc;
    if constexpr (EPL) {
        epl_setup(P);
        __syncthreads();
    }
    if (i >= g.ny * g.nx) return;
    img[i] = binned_pixel<EPL>(g, P, i / g.nx, i % g.nx);
}

__global__ void k_model_conv(const LensGeom g, const float *__restrict__ img, float *__restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.ny * g.nx) return;
    const int y = i / g.nx, x = i % g.nx, k = g.k, r = g.r;
    double o = 0.0;
    for (int a = 0; a < k; ++a) {
        const int yy = y - r + a;
        float pr = 0.0f;
        for (int b = 0; b < k; ++b) {
            const int xx = x - r + b;
            const float v = (yy >= 0 && yy < g.ny && xx >= 0 && xx < g.nx) ? img[yy * g.nx + xx] : 0.0f;
            pr = fmaf(g.psf[a * k + b], v, pr);
        }
        o += (double)pr;
    }
    out[i] = (float)o;
}

// ---------------------------------------------------------------------------
// fixed scratch of the allocation-free entry point
// ---------------------------------------------------------------------------
// Prepared constants of up to kNoAllocMax proposals: one array per device,
// held until the process ends.  In host code the name `scratch` is a host-side
// stand-in, not a device address; noalloc_init resolves the device address
// once per device and every launch takes that pointer.
static __device__ __align__(256) PropBlock scratch[kNoAllocMax];
// and the scratch of its split launches
static __device__ __align__(256) unsigned char scratch_split[kNoAllocSplit];
static void *g_scratch_dev[kNoAllocDevices], *g_split_dev[kNoAllocDevices];
static std::mutex g_scratch_mu;

hipError_t noalloc_init(int device)
{
    if (device < 0 || device >= kNoAllocDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_dev[device]) return hipSuccess;
    void *p = nullptr, *s = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e == hipSuccess) e = hipGetSymbolAddress(&s, HIP_SYMBOL(scratch_split));
    if (e != hipSuccess) return e;
    g_scratch_dev[device] = p;
    g_split_dev[device] = s;
    return hipSuccess;
}

PropBlock *noalloc_scratch(int device)
{
    if (device < 0 || device >= kNoAllocDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return static_cast<PropBlock *>(g_scratch_dev[device]);
}

void *noalloc_split(int device)
{
    if (device < 0 || device >= kNoAllocDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_split_dev[device];
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int choose_kc(int k) { return (k + 6) / 4; }

double host_sersic_bn(double n) { return sersic_bn(n); }

// Output groups (4 wide, FP32) and segments (16 wide, matrix cores) start at
// multiples of 4 and 16 at or right of xoff, below xoff + span, and each reads
// a window of 4 KC or L ring columns from its start.
int ring_width(int mode, int k, int span)
{
    if (mode_base(mode) == MODE_FP32 || mode_solved(mode)) return (span + 3) / 4 * 4 + 4 * choose_kc(k);
    return (span + 15) / 16 * 16 + window_len(mode, k);
}

size_t ring_row_bytes(int mode, int k, int span)
{
    const size_t elem = mode_base(mode) == MODE_FP32 ? 4
                        : mode_solved(mode)          ? 4 * mode_channels(mode)
                                                     : 2 * mode_planes(mode);
    return (size_t)ring_width(mode, k, span) * elem;
}

size_t ring_bytes(const LensGeom &g) { return (size_t)g.ring_rows * ring_row_bytes(g.mode, g.k, g.span); }

size_t lds_bytes(const LensGeom &g) { return ring_bytes(g) + (g.tab_off >= 0 ? kEplTabBytes : 0); }

// Dynamic LDS one workgroup may use: the opt-in limit when the device reports
// one above the default per-block limit (gfx950 addresses all 160 KB of a CU
// from one workgroup), never more than a CU holds.
size_t max_lds_bytes()
{
    int dev = 0, v = 0, optin = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 65536;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0) v = 65536;
    if (hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, dev) != hipSuccess) optin = 0;
    if (hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess)
        per_cu = 0;
    (void)hipGetLastError();
    size_t m = (size_t)std::max(v, optin);
    if (per_cu > 0) m = std::min(m, (size_t)per_cu);
    return m;
}

hipError_t launch_prep(const double *d_params, int64_t n, PropBlock *d_pc, int model, const int64_t *d_pstart,
                       const int *d_pmodel, int nl, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int bs = prep_threads(n);
    const int64_t nb = (n + bs - 1) / bs;
    hipLaunchKernelGGL(k_prep, dim3((unsigned)nb), dim3(bs), 0, st, d_params, n, d_pc, model, d_pstart, d_pmodel, nl);
    return hipGetLastError();
}

// Every mode, with the SIE and with the elliptical power law (MODE_EPL).
#define LENS_FOR_MODES(X) \
    X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)

template <int MODE, int NT>
static decltype(&k_loglike_fp32<MODE, NT, 0>) fp32_kernel(int k, bool few = false)
{
    if constexpr (!mode_epl(MODE)) {
        switch (k) {
#define LENS_K(KK) \
    case KK: return &k_loglike_fp32<MODE, NT, KK>;
            LENS_PSF_SIDES(LENS_K)
#undef LENS_K
        default: break;
        }
        if (few) switch (k) {
#define LENS_K(KK) \
    case KK: return &k_loglike_fp32<MODE, NT, KK>;
            LENS_PSF_SIDES_FEW(LENS_K)
#undef LENS_K
            default: break;
            }
    }
    return &k_loglike_fp32<MODE, NT, 0>;
}

// The single-lens likelihood kernel of a mode: FP32, MFMA, or solved amplitudes.
template <int MODE, int NT>
static const void *mode_kernel_ptr(int k, bool few = false)
{
    if constexpr (mode_solved(MODE)) return reinterpret_cast<const void *>(&k_loglike_nnls<MODE, NT>);
    else if constexpr (mode_base(MODE) == MODE_FP32)
        return reinterpret_cast<const void *>(fp32_kernel<MODE, NT>(k, few));
    else return reinterpret_cast<const void *>(&k_loglike_mfma<MODE, NT>);
}

template <int MODE, int NT>
static hipError_t launch_mode(const LensGeom &g, int cus, const PropBlock *d_pc, int64_t n, double *d_out,
                              double *d_amp, hipStream_t st)
{
    if constexpr (mode_solved(MODE))
        hipLaunchKernelGGL((k_loglike_nnls<MODE, NT>), dim3((unsigned)n), dim3(NT), lds_bytes(g), st, g, d_pc, d_out,
                           d_amp);
    else if constexpr (mode_base(MODE) == MODE_FP32)
        hipLaunchKernelGGL((fp32_kernel<MODE, NT>(g.k, n <= 3 * cus)), dim3((unsigned)n), dim3(NT), lds_bytes(g), st, g, d_pc, g.psf,
                           g.evl, g.evpre, g.evr, g.cvl, g.cvpre, g.data, g.wgt, d_out);
    else
        hipLaunchKernelGGL((k_loglike_mfma<MODE, NT>), dim3((unsigned)n), dim3(NT), lds_bytes(g), st, g, d_pc,
                           g.evl, g.evpre, g.evr, g.aop, g.seg, g.segpre, g.data, g.wgt, d_out);
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_nt(const LensGeom &g, int cus, const PropBlock *d_pc, int64_t n, double *d_out,
                            double *d_amp, hipStream_t st)
{
    switch (g.mode) {
#define LENS_M(M) \
    case M: return launch_mode<M, NT>(g, cus, d_pc, n, d_out, d_amp, st);
        LENS_FOR_MODES(LENS_M)
#undef LENS_M
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_loglike(const LensGeom &g, int cus, const PropBlock *d_pc, int64_t n, double *d_out, double *d_amp,
                          hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (g.nt == 512) return launch_nt<512>(g, cus, d_pc, n, d_out, d_amp, st);
    if (g.nt == 256) return launch_nt<256>(g, cus, d_pc, n, d_out, d_amp, st);
    return hipErrorInvalidValue;
}

static const void *batch_kernel(int mode, int nt);

template <int NT>
static const void *loglike_kernel_nt(const LensGeom &g)
{
    switch (g.mode) {
#define LENS_M(M) \
    case M: return mode_kernel_ptr<M, NT>(g.k);
        LENS_FOR_MODES(LENS_M)
#undef LENS_M
    default: return nullptr;
    }
}

int loglike_blocks_per_cu(const LensGeom &g)
{
    const void *k = g.nt == 512 ? loglike_kernel_nt<512>(g) : g.nt == 256 ? loglike_kernel_nt<256>(g) : nullptr;
    int nb = 0;
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, g.nt, lds_bytes(g)) != hipSuccess) return 0;
    return nb;
}

// Every kernel that may hold the ring of a lens of a mode (at any PSF side).
static void ring_kernels(int mode, std::vector<const void *> &v)
{
    switch (mode) {
#define LENS_M(M)                                                                                             \
    case M:                                                                                                   \
        for (int k = 0; k <= (mode_base(M) == MODE_FP32 ? kMaxK : 0); ++k) {                                  \
            v.push_back(mode_kernel_ptr<M, 256>(k, true));                                                    \
            v.push_back(mode_kernel_ptr<M, 512>(k, true));                                                    \
        }                                                                                                     \
        break;
        LENS_FOR_MODES(LENS_M)
#undef LENS_M
    }
    v.push_back(batch_kernel(mode, 256));
    v.push_back(batch_kernel(mode, 512));
    split_kernels(mode, v);
}

// Raise every ring-using kernel's dynamic-LDS limit so that dynamic plus
// static LDS reaches `bytes`.  The limit is a mode's own: kernels with much
// static LDS take no columns from the lenses of the others.
bool set_lds_limits(size_t bytes, size_t (&usable)[kModes])
{
    for (int mode = 0; mode < kModes; ++mode) {
        std::vector<const void *> ks;
        ring_kernels(mode, ks);
        usable[mode] = bytes;
        for (const void *k : ks) {
            hipFuncAttributes a{};
            if (!k || hipFuncGetAttributes(&a, k) != hipSuccess) return false;
            const size_t dyn = bytes > a.sharedSizeBytes ? bytes - a.sharedSizeBytes : 0;
            if (dyn == 0 || hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) != hipSuccess)
                return false;
            usable[mode] = std::min(usable[mode], dyn);
        }
    }
    return true;
}

size_t lds_per_cu()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess || v <= 0) {
        (void)hipGetLastError();
        return 65536;
    }
    return (size_t)v;
}

static const void *batch_kernel(int mode, int nt)
{
    switch (mode) {
#define LENS_M(M)                                                                                    \
    case M:                                                                                          \
        return nt == 256 ? reinterpret_cast<const void *>(&k_loglike_batch<M, 256>)                  \
               : nt == 512 ? reinterpret_cast<const void *>(&k_loglike_batch<M, 512>) : nullptr;
        LENS_FOR_MODES(LENS_M)
#undef LENS_M
    default: return nullptr;
    }
}

size_t batch_static_lds(int mode, int nt)
{
    const void *k = batch_kernel(mode, nt);
    hipFuncAttributes a{};
    if (!k || hipFuncGetAttributes(&a, k) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return (size_t)a.sharedSizeBytes;
}

int batch_blocks_per_cu(int mode, int nt, size_t lds)
{
    const void *k = batch_kernel(mode, nt);
    int nb = 0;
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, nt, lds) != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

hipError_t launch_batch(int mode, int nt, int grid, size_t lds, const LensGeom *d_geoms, const int *d_lstart,
                        const int64_t *d_lout, int nl, int nitems, const PropBlock *d_pc, double *d_out,
                        unsigned int *d_counter, hipStream_t st)
{
    const void *k = batch_kernel(mode, nt);
    if (!k || grid <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, st, d_counter);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    void *args[] = {(void *)&d_geoms, (void *)&d_lstart, (void *)&d_lout, (void *)&nl, (void *)&nitems,
                    (void *)&d_pc, (void *)&d_out, (void *)&d_counter};
    return hipLaunchKernel(k, dim3(grid), dim3(nt), args, lds, st);
}

hipError_t launch_mfma_probe(bool f16, const uint16_t *d_a, const uint16_t *d_b, float *d_d, hipStream_t st)
{
    if (f16) hipLaunchKernelGGL(k_mfma_probe<true>, dim3(1), dim3(64), 0, st, d_a, d_b, d_d);
    else hipLaunchKernelGGL(k_mfma_probe<false>, dim3(1), dim3(64), 0, st, d_a, d_b, d_d);
    return hipGetLastError();
}

hipError_t launch_model_image(const LensGeom &g, const PropBlock *d_pc, int stage, float *d_img, float *d_tmp,
                              hipStream_t st)
{
    const int npix = g.ny * g.nx;
    const int bs = 256, nb = (npix + bs - 1) / bs;
    float *dst = stage == 0 ? d_img : d_tmp;
    if (mode_epl(g.mode)) hipLaunchKernelGGL((k_model_binned<true>), dim3(nb), dim3(bs), 0, st, g, d_pc, dst);
    else hipLaunchKernelGGL((k_model_binned<false>), dim3(nb), dim3(bs), 0, st, g, d_pc, dst);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || stage == 0) return e;
    hipLaunchKernelGGL(k_model_conv, dim3(nb), dim3(bs), 0, st, g, d_tmp, d_img);
    return hipGetLastError();
}

}  // namespace lensk
