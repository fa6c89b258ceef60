// lens_split.hip -- the likelihood of few proposals, spread over the whole chip (gfx950).
//
// The fused kernels (lens_kernels.hip) give a proposal to one workgroup, which
// sweeps the image strip by strip.  A call with fewer proposals than the chip
// holds workgroups then takes as long as one workgroup takes for one image, on
// a mostly idle chip.  Here the same evaluation is cut across proposals and
// pixels alike, in three launches:
//   k_split_bin     the binned pixels of every proposal, 64 to a wave, to device
//                   memory in the order of the lens's pixel list;
//   k_split_conv    one strip of one proposal per workgroup: its ring of binned
//                   rows from that image, the PSF convolution and the strip's
//                   sums, one set per wave;
//   k_split_finish  the sums added in the fused kernels' order, lnL out.
// Each piece is the fused kernels' own code (lens_strip.h) on the same tiles
// and the same waves of pixels (the wave-uniform branches of the light profile
// make a pixel's last bits depend on its wave), and the sums are added in the
// same order: the results are the same bits.
//
// Forward model: Cao et al. (2025), Sec. 2.1 (Eqs. 1-3), Sec. 2.2 (Eq. 5), Sec. 2.3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "lens_device.h"
#include "lens_internal.h"
#include "lens_strip.h"

namespace lensk {

// The lens owning index i among nl, by the prefix member `start`: the last one
// with start <= i, 64 of them looked at together (a binary search reads one
// after another, at the start of every workgroup).  All lanes are active.
template <typename F>
__device__ __forceinline__ int split_find(int nl, int i, F start)
{
    int lo = 0;
    for (int j0 = 0; j0 < nl; j0 += 64) {
        const int j = j0 + (int)(threadIdx.x & 63);
        const int n = __popcll(__builtin_amdgcn_ballot_w64(j < nl && start(min(j, nl - 1)) <= i));
        if (n == 0) break;
        lo = j0 + n - 1;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// LIGHT: MODE_FP32 for every explicit-amplitude mode, or the solved mode.  A
// wave takes about `per` of the lens's pixel waves (LensGeom::binw) in turn.  Bound by
// the vector ALU, one pixel's s x s sub-pixels per thread, as in fill_rows;
// what a workgroup does before its first pixel (the deflection table) is why
// `per` grows with the work at hand (split_per).
template <int LIGHT, bool EPL, bool MULTI>
__global__ void __launch_bounds__(kSplitBinThreads, EPL ? 5 : 6)   // waves per SIMD: 80 VGPRs without the power law
k_split_bin(const LensGeom g1, const SplitLens e1, const LensGeom *__restrict__ geoms,
            const SplitLens *__restrict__ ents, int nl, int per, const PropBlock *__restrict__ pc,
            float *__restrict__ img)
{
    constexpr int MODE = LIGHT | (EPL ? (int)MODE_EPL : 0), NT = kSplitBinThreads;
    const int b = blockIdx.x;
    const int li = MULTI ? split_find(nl, b, [&](int j) { return ents[j].bin0; }) : 0;
    const SplitLens e = MULTI ? ents[li] : e1;
    LensGeom g = MULTI ? geoms[li] : g1;
    if (EPL && g.tab_off > 0) g.tab_off = 0;   // no ring here
    const int nblk = split_blocks(g.nbinw, per);
    const int rel = b - e.bin0, it = rel / nblk, blk = rel - it * nblk;
    const PropBlock *c = pc + e.out0 + it;
    if (mode_solved(LIGHT) ? c->valid == 0.0 : c->valid != 1.0) return;
    const PropBlock P = *c;
    if constexpr (sie_tab<MODE>()) {
        if constexpr (EPL) {
            epl_setup(P);
            __syncthreads();
        }
        sie_setup_wide<NT, EPL>(g, P);
    }
    __syncthreads();
    float *dst = img + e.img0 + (int64_t)it * e.img_n;   // one plane of `needed` pixels per channel
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto pixels = [&](auto tab) {
        constexpr bool TAB = decltype(tab)::value;
        // strided over the proposal's workgroups: each gets an even share of the
        // waves (contiguous shares left the last workgroup of every proposal
        // short, and those all land on the same XCDs)
        for (int wi = blk * (NT / 64) + wave; wi < g.nbinw; wi += nblk * (NT / 64)) {
            const uint32_t w = g.binw[wi];   // first pixel << 6 | pixels - 1
            if (lane > (int)(w & 63u)) continue;
            const int f = (int)(w >> 6) + lane;
            const uint32_t px = g.evl[f];
            const int y = (int)(px >> 16), x = (int)(px & 0xffffu);
            if constexpr (mode_solved(LIGHT)) {
                constexpr int NCH = mode_channels(LIGHT);
                float ch[NCH];
                binned_pixel_channels<mode_light(LIGHT), EPL, TAB>(g, P, y, x, ch);
#pragma unroll
                for (int c = 0; c < NCH; ++c) dst[c * g.needed + f] = ch[c];
            } else {
                dst[f] = binned_pixel<EPL, TAB>(g, P, y, x);
            }
        }
    };
    if (sie_tab<MODE>() && sie_use_table<EPL>(g, P)) pixels(std::true_type{});
    else pixels(std::false_type{});
}

// A ring row of a proposal's binned image: a buffer descriptor as long as the
// row's needed columns makes the loads of all other columns return the zeros
// that the ring wants there (raw buffer of 32-bit elements: out-of-range reads
// give 0).  at(x): ring column x.
struct RingRow {
    __amdgpu_buffer_rsrc_t row;
    int lo;   // ring column of the row's first pixel
    __device__ RingRow(const LensGeom &g, const float *plane, int y, bool in)
    {
        const int yc = min(max(y, 0), g.ny - 1);
        const int2 lr = g.evr[yc];
        lo = lr.x + g.r - g.xoff;
        row = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(plane + g.evpre[yc]), 0,
                                                in && y == yc ? (lr.y - lr.x) * 4 : 0, 0x00020000);
    }
    __device__ float at(int x) const
    {
        // the whole offset in one register: with a part of it in the
        // instruction's immediate, an offset that wraps to 0 and above would
        // count as out of range
        int off = (x - lo) * 4;
        asm("" : "+v"(off));
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(row, off, 0, 0));
    }
};

// The largest lane value of a wave (every lane holds it).
__device__ __forceinline__ uint32_t wave_max(uint32_t m)
{
    const auto step = [&](auto ctrl) {
        m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, decltype(ctrl)::value, 0xf, 0xf, false));
    };
    step(std::integral_constant<int, 0x111>{});   // row_shr:1, 2, 4, 8
    step(std::integral_constant<int, 0x112>{});
    step(std::integral_constant<int, 0x114>{});
    step(std::integral_constant<int, 0x118>{});
    step(std::integral_constant<int, 0x142>{});   // row_bcast:15, 31
    step(std::integral_constant<int, 0x143>{});
    return (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
}

// Rows j0 .. of the ring of strip y0, channel c.
template <int MODE, size_t... J>
__device__ __forceinline__ void ring_rows(const LensGeom &g, void *ring, const float *plane, int c, int y0, int j0,
                                          std::index_sequence<J...>)
{
    constexpr int R = sizeof...(J);
    const int W = g.ring_w, RB = g.ring_rows, lane = threadIdx.x & 63;
    const RingRow row[R] = {RingRow(g, plane, y0 - g.r + j0 + (int)J, j0 + (int)J < RB)...};
    for (int x = lane; x < W; x += 64) {
        const float v[R] = {row[J].at(x)...};
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (j0 + j < RB) {
                const int idx = (y0 + j0 + j) % RB * W + x;
                if constexpr (mode_solved(MODE)) static_cast<float *>(ring)[c * g.plane + idx] = v[j];
                else RingStoreM<MODE>::put(ring, g.plane, idx, v[j]);
            }
    }
}

// The ring of strip y0 from a proposal's binned image, every slot written once.
// A wave takes R rows at a time, all their loads in flight together (with one
// row at a time the loads' latencies, one after another, took longer than the
// convolution).
template <int MODE, int NT>
__device__ __forceinline__ void split_ring(const LensGeom &g, void *ring, const float *img, int y0)
{
    const int W = g.ring_w, RB = g.ring_rows;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (mode_base(MODE) == MODE_SPLIT) {
        // each row's scale from its largest |value|, then the halves, two
        // columns to a lane and a 32-bit write (by 16-bit writes, with the FP32
        // values parked in the ring until the row's scale was known, the
        // staging issued more LDS instructions than the convolution).  Rows of
        // up to 128 C columns stay in registers; wider ones are read twice.
        constexpr int R = 4, C = 2;
        for (int j0 = wave * R; j0 < RB; j0 += NT / 64 * R) {
            float v[R][C][2];
            uint32_t m[R];
            const auto load = [&](const RingRow &row, int j, int x0) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int x = x0 + 128 * c + 2 * lane;
                    v[j][c][0] = row.at(x);
                    v[j][c][1] = row.at(x + 1);
                }
            };
            const auto most = [&](int j) {
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int i = 0; i < 2; ++i) m[j] = max(m[j], __float_as_uint(fabsf(v[j][c][i])));
            };
#pragma unroll
            for (int j = 0; j < R; ++j) {
                m[j] = 0u;
                load(RingRow(g, img, y0 - g.r + j0 + j, j0 + j < RB), j, 0);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) most(j);
            for (int x0 = 128 * C; x0 < W; x0 += 128 * C)
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    load(RingRow(g, img, y0 - g.r + j0 + j, j0 + j < RB), j, x0);
                    most(j);
                }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (j0 + j >= RB) break;
                const int slot = (y0 + j0 + j) % RB;
                float inv;
                const float sc = f16_row_scale(__uint_as_float(wave_max(m[j])), inv);
                if (lane == 0) f16_rowscale()[slot] = inv;
                uint32_t *hi = static_cast<uint32_t *>(ring) + (slot * W >> 1), *lo = hi + (g.plane >> 1);
                for (int x0 = 0; x0 < W; x0 += 128 * C) {
                    if (W > 128 * C) load(RingRow(g, img, y0 - g.r + j0 + j, true), j, x0);
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        const int x = x0 + 128 * c + 2 * lane;
                        uint16_t h0, h1, l0, l1;
                        f16_halves(v[j][c][0], sc, h0, l0);
                        f16_halves(v[j][c][1], sc, h1, l1);
                        if (x < W) {
                            hi[x >> 1] = (uint32_t)h1 << 16 | h0;
                            lo[x >> 1] = (uint32_t)l1 << 16 | l0;
                        }
                    }
                }
            }
        }
    } else {
        constexpr int R = 8, NCH = mode_solved(MODE) ? mode_channels(MODE) : 1;
        for (int c = 0; c < NCH; ++c)
            for (int j0 = wave * R; j0 < RB; j0 += NT / 64 * R)
                ring_rows<MODE>(g, ring, img + (size_t)c * g.needed, c, y0, j0, std::make_index_sequence<R>{});
    }
}

// conv(K) with the PSF side k as a constant where it is one of the small odd
// ones, else conv(0).  A constant side takes a row's weights and its window in
// one go, free of loop control: 12.3 against 16 us for one 128x128 px proposal
// at side 13 (where the loads' latencies show), 0.88 against 0.93 ms for 8,192.
// Beyond 31 the window's registers would halve the resident waves.
template <typename Conv>
__device__ __forceinline__ void conv_side(int k, Conv conv)
{
    switch (k) {
#define LENS_K(KK) \
    case KK: conv(std::integral_constant<int, KK>{}); break;
        LENS_PSF_SIDES(LENS_K)
#undef LENS_K
    default: conv(std::integral_constant<int, 0>{});
    }
}

// The PSF as constant memory: its weights come by scalar loads also where the
// descriptor that holds the pointer was itself loaded (as vector loads they took
// 30 registers of the multi-lens kernel).
typedef const __attribute__((address_space(4))) float *ConstF;

// Threads of a convolution workgroup: those that sweep a strip in the fused
// kernels, but half of them in the FP16 split, whose tiles of four rows are few
// (four in 16 rows of 200 masked columns) and want the registers of two waves.
template <int MODE, int NT>
__host__ __device__ constexpr int split_threads() { return mode_base(MODE) == MODE_SPLIT ? NT / 2 : NT; }

// One workgroup per (proposal, strip).  Bound by the convolution (vector ALU, or
// the matrix cores); the ring comes from the L2.
template <int MODE, int NT, bool MULTI>
__global__ void __launch_bounds__((split_threads<MODE, NT>()), (mode_base(MODE) == MODE_SPLIT ? 2 : 4))
k_split_conv(const LensGeom g1, const SplitLens e1, const LensGeom *__restrict__ geoms,
             const SplitLens *__restrict__ ents, int nl, const PropBlock *__restrict__ pc,
             const float *__restrict__ img, double *__restrict__ part)
{
    extern __shared__ float4 lds4[];
    const int b = blockIdx.x;
    const int li = MULTI ? split_find(nl, b, [&](int j) { return ents[j].conv0; }) : 0;
    const SplitLens e = MULTI ? ents[li] : e1;
    const LensGeom g = MULTI ? geoms[li] : g1;
    // strips rotated by the proposal: those at the image's edge have less to do,
    // and in a fixed order the same XCDs would get them all
    const int rel = b - e.conv0, it = rel / g.nstrips, strip = (rel + it) % g.nstrips;
    const double valid = pc[e.out0 + it].valid;
    if (mode_solved(MODE) ? valid == 0.0 : valid != 1.0) return;
    const int y0 = strip * g.strip_h, y1 = min(y0 + g.strip_h, g.ny);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    split_ring<MODE, split_threads<MODE, NT>()>(g, lds4, img + e.img0 + (int64_t)it * e.img_n, y0);
    __syncthreads();
    if constexpr (mode_solved(MODE)) {
        constexpr int NM = MomN<mode_channels(MODE)>::NM;
        MomN<mode_channels(MODE)> mo;
        conv_side(g.k, [&](auto K) {
            mo = conv_rows_solved<MODE, NT, decltype(K)::value>(g, reinterpret_cast<const float *>(lds4),
                                                                (ConstF)(uintptr_t)g.psf, y0, y1, tid);
        });
        double *o = part + e.part0 + (((int64_t)it * g.nstrips + strip) * (NT / 64) + wave) * NM;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const double s = wave_sum(mo.m[i]);
            if (lane == 0) o[i] = s;
        }
    } else {
        double *o = part + e.part0 + ((int64_t)it * g.nstrips + strip) * (NT / 64);
        if constexpr (mode_base(MODE) == MODE_SPLIT) {
            double acc[2];
            conv_mfma_quads<NT>(g, reinterpret_cast<const uint16_t *>(lds4), y0, y1, wave, acc);
            acc[0] = wave_sum(acc[0]);
            acc[1] = wave_sum(acc[1]);
            if (lane < 2) o[2 * wave + lane] = lane ? acc[1] : acc[0];
        } else {
            double acc;
            if constexpr (mode_base(MODE) == MODE_FP32)
                conv_side(g.k, [&](auto K) {
                    acc = conv_rows<decltype(K)::value, NT>(g, reinterpret_cast<const float *>(lds4),
                                                            (ConstF)(uintptr_t)g.psf, g.cvl, g.cvpre, g.data, g.wgt, y0,
                                                            y1, tid);
                });
            else
                acc = conv_mfma<MODE, NT>(g, reinterpret_cast<const uint16_t *>(lds4), g.aop, g.seg, g.segpre, g.data,
                                          g.wgt, y0, y1, tid);
            acc = wave_sum(acc);
            if (lane == 0) o[wave] = acc;
        }
    }
}

// One wave per proposal.  NCH: 0 for explicit amplitudes, else the solved
// channels.  Lane l takes wave slot l % nw of the moment l / nw (rounds of
// 64 / nw moments), strip by strip; the slots are then added wave by wave.
template <int NCH, bool MULTI>
__global__ void __launch_bounds__(64)
k_split_finish(const LensGeom g1, const SplitLens e1, const LensGeom *__restrict__ geoms,
               const SplitLens *__restrict__ ents, int nl, const PropBlock *__restrict__ pc,
               const double *__restrict__ part, double *__restrict__ out, double *__restrict__ amp)
{
    constexpr int NM = NCH ? MomN<NCH ? NCH : 1>::NM : 1;
    __shared__ double red[NM][8];
    const int b = blockIdx.x, lane = threadIdx.x;
    const int li = MULTI ? split_find(nl, b, [&](int j) { return ents[j].item0; }) : 0;
    const SplitLens e = MULTI ? ents[li] : e1;
    const LensGeom *g = MULTI ? geoms + li : &g1;
    const int it = b - e.item0, nw = g->nt >> 6, ns = g->nstrips;
    const int64_t p = e.out0 + it;
    const double valid = pc[p].valid;
    if (NCH ? valid == 0.0 : valid != 1.0) {
        if (lane == 0) {
            out[p] = -INFINITY;
            if (NCH && amp)
                for (int a = 0; a < NCH; ++a) amp[NCH * p + a] = NAN;
        }
        return;
    }
    const double *src = part + e.part0 + (int64_t)it * ns * nw * NM;
    for (int k = lane; k < NM * nw; k += 64) {
        const int i = k / nw, w = k - i * nw;
        double s = 0.0;
        for (int st = 0; st < ns; ++st) s += src[((int64_t)st * nw + w) * NM + i];
        red[i][w] = s;
    }
    __syncthreads();
    if constexpr (NCH == 0) {
        if (lane != 0) return;
        double s = 0.0;
        for (int w = 0; w < nw; ++w) s += red[0][w];
        out[p] = g->norm - 0.5 * s;
    } else {
        MomN<NCH> t{};
        for (int w = 0; w < nw; ++w)
            for (int i = 0; i < NM; ++i) t.m[i] += red[i][w];
        double s[NCH];
        const double chi2 = nnls_wave<NCH>(t, g->dd, s);
        if (lane != 0) return;
        out[p] = g->norm - 0.5 * chi2;
        if (amp)
            for (int a = 0; a < NCH; ++a) amp[NCH * p + a] = s[a];
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
SplitLens split_lens(const LensGeom &g)
{
    SplitLens e{};
    const int nch = mode_solved(g.mode) ? mode_channels(g.mode) : 1;
    e.img_n = ((int64_t)g.needed * nch + 15) / 16 * 16;
    const int nm = mode_solved(g.mode) ? nch * (nch + 1) / 2 + nch : 1;
    e.part_n = ((int64_t)g.nstrips * (g.nt / 64) * nm + 7) / 8 * 8;   // 64-byte multiples keep the images aligned
    return e;
}

size_t split_bytes(const SplitLens &e, int64_t n)
{
    return (size_t)n * ((size_t)e.img_n * sizeof(float) + (size_t)e.part_n * sizeof(double));
}

// What n proposals weigh in split_per: their pixel waves, times the work of a
// workgroup before its first pixel in units of one wave of pixels (from runs with
// one pixel wave each: 8 % more of 4 x 4 sub-pixels, with the power law 34 %).
static double split_weight(const LensGeom &g, int64_t n)
{
    return (double)n * g.nbinw * (mode_epl(g.mode) ? 5.4 : 1.3) / (g.s * g.s);
}

// Pixel waves per wave of the binning launch.  With W pixel waves in all, work h
// before the first and p of them per wave, the total grows as W (1 + h / p) and
// the chip empties over a time that grows as p: the best p goes as the root of
// W h.  The factor is from sweeps of p over 1 to 4,096 proposals (128x128 px,
// SIE: best 1 at 32 proposals, 2 to 4 at 301, 4 to 16 at 1,024; power law 2, 4 to
// 6, 14; 64x64 px without supersampling 1, 4 to 5, 4): 301 proposals 253 -> 239
// us, 64 74.7 -> 69.1 against whole powers of two by W alone, which left the last
// of few rounds half empty.
static int split_per(double weight, int cus)
{
    return std::clamp((int)lround(sqrt(weight / (2.3 * cus))), 1, 16);
}

namespace {

struct SplitArgs {
    const LensGeom *g;        // one lens: host descriptor; many: device array
    const SplitLens *e;
    int nl;                   // 0: one lens
    int mode, nt;
    int64_t bins, units, items;
    size_t lds;
    int per;                  // pixel waves per wave of the binning launch
    const PropBlock *pc;
    float *img;
    double *part, *out, *amp;
};

template <int LIGHT, bool EPL>
hipError_t bin_launch(const SplitArgs &a, hipStream_t st)
{
    if (a.bins == 0) return hipSuccess;   // nothing masked: no pixel is needed
    const dim3 grid((unsigned)a.bins), block(kSplitBinThreads);
    const size_t tab = mode_epl_tab(a.mode) ? kEplTabBytes : 0;
    if (a.nl)
        hipLaunchKernelGGL((k_split_bin<LIGHT, EPL, true>), grid, block, tab, st, LensGeom{}, SplitLens{}, a.g, a.e, a.nl,
                           a.per, a.pc, a.img);
    else
        hipLaunchKernelGGL((k_split_bin<LIGHT, EPL, false>), grid, block, tab, st, *a.g, *a.e, nullptr, nullptr, 0,
                           a.per, a.pc, a.img);
    return hipGetLastError();
}

template <int MODE, int NT>
hipError_t conv_launch(const SplitArgs &a, hipStream_t st)
{
    const dim3 grid((unsigned)a.units), block(split_threads<MODE, NT>());
    if (a.nl)
        hipLaunchKernelGGL((k_split_conv<MODE, NT, true>), grid, block, a.lds, st, LensGeom{}, SplitLens{}, a.g, a.e,
                           a.nl, a.pc, a.img, a.part);
    else
        hipLaunchKernelGGL((k_split_conv<MODE, NT, false>), grid, block, a.lds, st, *a.g, *a.e, nullptr, nullptr, 0,
                           a.pc, a.img, a.part);
    return hipGetLastError();
}

template <int NCH>
hipError_t finish_launch(const SplitArgs &a, hipStream_t st)
{
    const dim3 grid((unsigned)a.items), block(64);
    if (a.nl)
        hipLaunchKernelGGL((k_split_finish<NCH, true>), grid, block, 0, st, LensGeom{}, SplitLens{}, a.g, a.e, a.nl,
                           a.pc, a.part, a.out, a.amp);
    else
        hipLaunchKernelGGL((k_split_finish<NCH, false>), grid, block, 0, st, *a.g, *a.e, nullptr, nullptr, 0, a.pc,
                           a.part, a.out, a.amp);
    return hipGetLastError();
}

#define SPLIT_FOR_MODES(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7)

hipError_t split_launch(const SplitArgs &a, hipStream_t st)
{
    const int base = mode_base(a.mode), light = mode_solved(a.mode) ? base : (int)MODE_FP32;
    hipError_t e = hipErrorInvalidValue;
    switch (light) {
#define SPLIT_B(M) \
    case M: e = mode_epl(a.mode) ? bin_launch<M, true>(a, st) : bin_launch<M, false>(a, st); break;
        SPLIT_B(0) SPLIT_B(4) SPLIT_B(5) SPLIT_B(6) SPLIT_B(7)
#undef SPLIT_B
    default: break;
    }
    if (e != hipSuccess) return e;
    switch (base) {
#define SPLIT_C(M) \
    case M: e = a.nt == 512 ? conv_launch<M, 512>(a, st) : conv_launch<M, 256>(a, st); break;
        SPLIT_FOR_MODES(SPLIT_C)
#undef SPLIT_C
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    switch (mode_channels(a.mode)) {
    case 0: return finish_launch<0>(a, st);
    case 1: return finish_launch<1>(a, st);
    case 2: return finish_launch<2>(a, st);
    case 4: return finish_launch<4>(a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_split(const LensGeom &g, int cus, const PropBlock *d_pc, int64_t n, void *scratch, double *d_out,
                        double *d_amp, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const SplitLens e = split_lens(g);
    SplitArgs a{};
    a.g = &g;
    a.e = &e;
    a.mode = g.mode;
    a.nt = g.nt;
    a.per = split_per(split_weight(g, n), cus);
    a.bins = n * split_blocks(g.nbinw, a.per);
    a.units = n * g.nstrips;
    a.items = n;
    a.lds = ring_bytes(g);
    a.pc = d_pc;
    a.part = static_cast<double *>(scratch);
    a.img = reinterpret_cast<float *>(a.part + n * e.part_n);
    a.out = d_out;
    a.amp = d_amp;
    return split_launch(a, st);
}

bool split_chunks(const LensGeom *geoms, const int64_t *lout, const int64_t *counts, int nl, size_t cap, int cus,
                  std::vector<SplitLens> *ents, std::vector<SplitChunk> *chunks, size_t *bytes)
{
    size_t used = 0;   // of the open chunk
    double weight = 0.0;
    int64_t img = 0;
    bool open = false;
    const auto close = [&] {
        if (!open) return;
        SplitChunk &c = chunks->back();
        c.per = split_per(weight, cus);
        for (int i = 0; i < c.nl; ++i) {
            SplitLens &e = (*ents)[(size_t)c.ent + i];
            e.bin0 = (int)c.bins;
            c.bins += (int64_t)e.pad * split_blocks(geoms[c.lens + i].nbinw, c.per);   // pad: proposals, until now
            e.pad = 0;
        }
        *bytes = std::max(*bytes, used);
        open = false;
    };
    for (int i = 0; i < nl; ++i) {
        const SplitLens one = split_lens(geoms[i]);
        const size_t per = split_bytes(one, 1);
        if (per > cap) return false;
        for (int64_t at = 0; at < counts[i];) {
            if (open && used + per > cap) close();
            if (!open) {
                chunks->push_back(SplitChunk{i, (int)ents->size(), 0, 1, 0, 0, 0, 0});
                open = true;
                used = 0;
                weight = 0.0;
                img = 0;
            }
            SplitChunk &c = chunks->back();
            const int64_t n = std::min<int64_t>(counts[i] - at, (int64_t)((cap - used) / per));
            SplitLens e = one;
            e.conv0 = (int)c.units;
            e.item0 = (int)c.items;
            e.pad = (int)n;
            e.out0 = lout[i] + at;
            e.img0 = img;
            e.part0 = c.part_n;
            ents->push_back(e);
            c.nl++;
            c.units += n * geoms[i].nstrips;
            c.items += n;
            c.part_n += n * e.part_n;
            img += n * e.img_n;
            weight += split_weight(geoms[i], n);
            used += (size_t)n * per;
            at += n;
        }
    }
    close();
    return true;
}

hipError_t launch_split_chunk(int mode, int nt, size_t lds, const SplitChunk &c, const LensGeom *d_geoms,
                              const SplitLens *d_ents, const PropBlock *d_pc, void *scratch, double *d_out,
                              hipStream_t st)
{
    SplitArgs a{};
    a.g = d_geoms + c.lens;
    a.e = d_ents + c.ent;
    a.nl = c.nl;
    a.mode = mode;
    a.nt = nt;
    a.per = c.per;
    a.bins = c.bins;
    a.units = c.units;
    a.items = c.items;
    a.lds = lds;
    a.pc = d_pc;
    a.part = static_cast<double *>(scratch);
    a.img = reinterpret_cast<float *>(a.part + c.part_n);
    a.out = d_out;
    return split_launch(a, st);
}

void split_kernels(int mode, std::vector<const void *> &v)
{
    switch (mode_base(mode)) {
#define SPLIT_K(M)                                                                 \
    case M:                                                                        \
        v.push_back(reinterpret_cast<const void *>(&k_split_conv<M, 256, false>)); \
        v.push_back(reinterpret_cast<const void *>(&k_split_conv<M, 512, false>)); \
        v.push_back(reinterpret_cast<const void *>(&k_split_conv<M, 256, true>));  \
        v.push_back(reinterpret_cast<const void *>(&k_split_conv<M, 512, true>));  \
        break;
        SPLIT_FOR_MODES(SPLIT_K)
#undef SPLIT_K
    }
}

}  // namespace lensk
