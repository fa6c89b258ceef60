// Drives the library's host code with no GPU: the HIP entry points that it calls
// are defined here over host memory, and the library's own objects are linked
// against them instead of the HIP runtime (tests/test_host_runtime.py).  Device
// memory is host memory, a kernel launch computes nothing: it is counted by
// name, and the memory that the split launches would write is checked against
// the live allocations.  Captured launches are kept with their graph and checked
// again whenever it is launched.
//
// usage: host_runtime_driver SCENARIO; prints "ok" and exits with 0, or one line
// per failed check.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "lens_api.h"
#include "lens_internal.h"

static int fails = 0;
#define TRUE(cond)                                           \
    do {                                                     \
        if (!(cond)) {                                       \
            printf("FAIL line %d: %s\n", __LINE__, #cond);   \
            fails++;                                         \
        }                                                    \
    } while (0)
#define CK(expr) TRUE((expr) == LENS_OK)

// ---------------------------------------------------------------------------
// the device
// ---------------------------------------------------------------------------
namespace fake {

std::recursive_mutex mu;
std::map<const void *, std::string> kernels;        // host stub -> device name
std::map<const void *, size_t> vars;                // __device__ variables
std::map<const void *, void *> var_mem;
std::map<uintptr_t, size_t> live;                   // allocations: start -> bytes
std::map<std::string, int> launched;                // kernel family -> launches
int outside = 0;                                    // writes outside every live allocation
int legacy_ops = 0;                                 // work on the legacy default stream
int captures = 0, graph_launches = 0;
size_t hbm = (size_t)64 << 30;                      // physical memory left

struct Touch {
    const char *what;
    uintptr_t p;
    size_t n;
};
struct Graph {
    std::vector<Touch> touches;
    std::vector<std::string> names;
};
struct Stream {
    Graph *capture = nullptr;
};

void check(const Touch &t)
{
    if (t.n == 0) return;
    auto it = live.upper_bound(t.p);
    if (it != live.begin()) {
        --it;
        if (t.p + t.n <= it->first + it->second) return;
    }
    outside++;
}

void *alloc(size_t n)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (n > hbm) return nullptr;
    void *p = nullptr;
    if (posix_memalign(&p, 4096, n ? n : 1)) return nullptr;
    live[(uintptr_t)p] = n;
    hbm -= n;
    return p;
}

void release(void *p)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    auto it = live.find((uintptr_t)p);
    if (it == live.end()) return;
    hbm += it->second;
    live.erase(it);
    free(p);
}

// What a split launch writes (its arguments as declared in lens_split.hip).
void split_touches(const std::string &name, dim3 grid, void **a, std::vector<Touch> *out)
{
    const bool bin = name.find("k_split_bin") != std::string::npos;
    const bool conv = name.find("k_split_conv") != std::string::npos;
    if (!bin && !conv) return;
    const int nl = *(int *)a[4];
    const uintptr_t dst = (uintptr_t)*(void **)a[bin ? 7 : 7];
    int64_t end = 0;
    if (nl == 0) {
        const lensk::LensGeom &g = *(const lensk::LensGeom *)a[0];
        const lensk::SplitLens &e = *(const lensk::SplitLens *)a[1];
        const int64_t per = bin ? lensk::split_blocks(g.nbinw, *(int *)a[5]) : g.nstrips;
        const int64_t n = grid.x / per;
        end = bin ? e.img0 + n * e.img_n : e.part0 + n * e.part_n;
    } else {
        const lensk::LensGeom *g = *(const lensk::LensGeom **)a[2];
        const lensk::SplitLens *e = *(const lensk::SplitLens **)a[3];
        const int per = bin ? *(int *)a[5] : 0;
        for (int i = 0; i < nl; ++i) {
            const int64_t first = bin ? e[i].bin0 : e[i].conv0;
            const int64_t last = i + 1 < nl ? (bin ? e[i + 1].bin0 : e[i + 1].conv0) : (int64_t)grid.x;
            const int64_t each = bin ? lensk::split_blocks(g[i].nbinw, per) : g[i].nstrips;
            const int64_t n = each > 0 ? (last - first) / each : 0;
            end = std::max(end, bin ? e[i].img0 + n * e[i].img_n : e[i].part0 + n * e[i].part_n);
        }
    }
    out->push_back({bin ? "images" : "sums", dst, (size_t)end * (bin ? 4 : 8)});
}

// The FP16 split's row groups have to start at the strips of the launch, its pixel
// waves to cover the needed pixels once.
int bad_lists = 0;
void check_lists(const std::string &name, void **a)
{
    const bool mfma = name.find("k_loglike_mfma") != std::string::npos;
    const bool split = (name.find("k_split_bin") != std::string::npos || name.find("k_split_conv") != std::string::npos) &&
                       *(int *)a[4] == 0;
    if (!mfma && !split) return;
    const lensk::LensGeom &g = *(const lensk::LensGeom *)a[0];
    if (lensk::mode_base(g.mode) == lensk::MODE_SPLIT)
        for (int y0 = 0; y0 < g.ny; y0 += g.strip_h)
            for (int i = g.segpre[y0]; i < g.segpre[std::min(y0 + g.strip_h, g.ny)]; ++i) {
                const int y = (int)(g.seg[i] >> 16);
                bad_lists += y < y0 || y >= y0 + g.strip_h || (y - y0) % lensk::kRowGroup != 0;
            }
    if (split) {
        int at = 0;
        for (int i = 0; i < g.nbinw; ++i) {
            bad_lists += (int)(g.binw[i] >> 6) != at;
            at += (int)(g.binw[i] & 63) + 1;
        }
        bad_lists += at != g.needed;
    }
}

std::string family(const std::string &name)
{
    for (const char *f : {"k_split_bin", "k_split_conv", "k_split_finish", "k_loglike_batch", "k_loglike_fp32",
                          "k_loglike_mfma", "k_loglike_nnls", "k_prep"})
        if (name.find(f) != std::string::npos) return f;
    return "other";
}

int ran(const char *f)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    return launched[f];
}

}  // namespace fake

using fake::Stream;

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *dev, unsigned, void *, void *, dim3 *, dim3 *,
                           int *)
{
    fake::kernels[host] = dev;
}
void __hipRegisterVar(void **, void *host, char *, char *, int, size_t n, int, int) { fake::vars[host] = n; }

static thread_local struct {
    dim3 g, b;
    size_t lds;
    hipStream_t st;
} call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st)
{
    call = {g, b, lds, st};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st)
{
    *g = call.g;
    *b = call.b;
    *lds = call.lds;
    *st = call.st;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3, void **args, size_t, hipStream_t st)
{
    std::lock_guard<std::recursive_mutex> lk(fake::mu);
    const std::string &name = fake::kernels[f];
    std::vector<fake::Touch> t;
    fake::split_touches(name, grid, args, &t);
    Stream *s = (Stream *)st;
    if (s && s->capture) {
        s->capture->touches.insert(s->capture->touches.end(), t.begin(), t.end());
        s->capture->names.push_back(fake::family(name));
    } else {
        if (!s) fake::legacy_ops++;
        for (const auto &x : t) fake::check(x);
        fake::check_lists(name, args);
        fake::launched[fake::family(name)]++;
    }
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    *p = fake::alloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    fake::release(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned)
{
    *d = h;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    fake::legacy_ops++;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    if (st && ((Stream *)st)->capture) return hipSuccess;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t)
{
    *f = *t = fake::hbm;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *sym)
{
    void *&m = fake::var_mem[sym];
    if (!m) m = fake::alloc(fake::vars[sym]);
    *p = m;
    return hipSuccess;
}

hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 65536 : 163840;
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *)
{
    memset(a, 0, sizeof(*a));
    a->sharedSizeBytes = 4096;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    *s = (hipStream_t) new Stream();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    delete (Stream *)s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    *st = s && ((Stream *)s)->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    fake::captures++;
    ((Stream *)s)->capture = new fake::Graph();
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    *g = (hipGraph_t)((Stream *)s)->capture;
    ((Stream *)s)->capture = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *e = (hipGraphExec_t) new fake::Graph(*(fake::Graph *)g);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete (fake::Graph *)g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e)
{
    delete (fake::Graph *)e;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t)
{
    std::lock_guard<std::recursive_mutex> lk(fake::mu);
    fake::graph_launches++;
    for (const auto &t : ((fake::Graph *)e)->touches) fake::check(t);
    for (const auto &n : ((fake::Graph *)e)->names) fake::launched[n]++;
    return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t) new int(0); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (int *)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }

}  // extern "C"

// ---------------------------------------------------------------------------
// scenarios
// ---------------------------------------------------------------------------
namespace {

constexpr int64_t MB = 1 << 20;

lens_ctx *open(int64_t budget, lens_dev_alloc_fn a = nullptr, lens_dev_free_fn f = nullptr)
{
    lens_init_opts o{};
    o.hbm_budget_bytes = budget;
    o.dev_alloc = a;
    o.dev_free = f;
    lens_ctx *c = nullptr;
    TRUE(lens_init(&o, &c) == LENS_OK);
    return c;
}

struct Kind {
    int px = 64, k = 11, prec = LENS_PREC_FP32, amps = 0, light = 0, mass = 0, s = 2;
};

lens_status try_load(lens_ctx *c, lens_id *id, const Kind &K)
{
    std::vector<double> psf((size_t)K.k * K.k, 1.0 / (K.k * K.k)), img((size_t)K.px * K.px, 0.0),
        sigma((size_t)K.px * K.px, 0.01);
    std::vector<uint8_t> mask((size_t)K.px * K.px, 1);
    lens_data_desc d{};
    d.ny = d.nx = K.px;
    d.pixel_scale = 0.05;
    d.supersample = K.s;
    d.psf_size = K.k;
    d.psf = psf.data();
    d.data = img.data();
    d.sigma = sigma.data();
    d.mask = mask.data();
    d.precision = K.prec;
    d.amplitudes = K.amps;
    d.light_model = K.light;
    d.mass_model = K.mass;
    return lens_load_data(c, &d, id);
}

lens_id load(lens_ctx *c, const Kind &K = Kind())
{
    lens_id id = 0;
    CK(try_load(c, &id, K));
    return id;
}

int64_t used(lens_ctx *c)
{
    lens_stats s{};
    CK(lens_get_stats(c, &s));
    return s.hbm_used_bytes;
}

// A caller's pool: a freed block of a megabyte or more is handed out again, at its
// own address, for any such request that fits it.  The memory stays allocated at its first size; only
// the bytes asked for count as live.
struct Pool {
    std::map<void *, size_t> size;   // of every block ever made
    std::vector<void *> idle;
} pool;
void *pool_alloc(size_t n, void *, void *)
{
    for (size_t i = 0; n >= (size_t)MB && i < pool.idle.size(); ++i) {
        void *p = pool.idle[i];
        if (pool.size[p] < n) continue;
        pool.idle.erase(pool.idle.begin() + (long)i);
        fake::live[(uintptr_t)p] = n;
        return p;
    }
    void *p = fake::alloc(n);
    if (p) pool.size[p] = n;
    return p;
}
void pool_free(void *p, void *, void *)
{
    fake::live.erase((uintptr_t)p);
    if (pool.size[p] >= (size_t)MB) pool.idle.insert(pool.idle.begin(), p);
}

// A multi-lens call shape is captured with the split scratch of that moment.
// The budget then takes the scratch back, and later leaves room for a smaller
// one only, which the pool hands out at the old address: the captured launches
// must not run in it.
void plan_scratch()
{
    lens_ctx *c = open(80 * MB, pool_alloc, pool_free);
    const lens_id ids[2] = {load(c), load(c)};
    const int64_t counts[2] = {300, 300};
    std::vector<double> par((size_t)600 * LENS_PARAM_STRIDE, 0.5), out(600);
    CK(lens_loglike_multi(c, 2, ids, counts, par.data(), out.data()));
    CK(lens_loglike_multi(c, 2, ids, counts, par.data(), out.data()));
    TRUE(fake::ran("k_split_bin") > 0 && fake::ran("k_loglike_batch") == 0);
    const int graphs = fake::graph_launches;
    TRUE(graphs > 0 && fake::outside == 0);
    // load until the scratch has been taken back and the budget is full, then
    // make room for a smaller one
    std::vector<lens_id> more;
    lens_id id;
    while (try_load(c, &id, Kind()) == LENS_OK) more.push_back(id);
    while (more.size() > 100 && !fails) {
        CK(lens_unload(c, more.back()));
        more.pop_back();
        const int g = fake::graph_launches;
        CK(lens_loglike_multi(c, 2, ids, counts, par.data(), out.data()));
        TRUE(fake::outside == 0);
        TRUE(fake::graph_launches == g + 1);   // captured anew, not left without a graph
    }
    // with room again it goes through the split launches as before
    while (!more.empty()) {
        CK(lens_unload(c, more.back()));
        more.pop_back();
    }
    const int b = fake::ran("k_loglike_batch"), s = fake::ran("k_split_bin");
    CK(lens_loglike_multi(c, 2, ids, counts, par.data(), out.data()));
    TRUE(fake::outside == 0 && fake::ran("k_loglike_batch") == b && fake::ran("k_split_bin") > s);
    lens_shutdown(c);
}

// A call whose constants need most of the budget is served whatever split
// scratch its own stream holds.
void own_scratch()
{
    const int64_t n = 50000;
    std::vector<double> par((size_t)n * LENS_PARAM_STRIDE, 0.5), out(n);
    for (int held = 0; held < 2; ++held) {   // the stream's first call, or one after it
        lens_ctx *c = open(16 * MB);
        const lens_id id = load(c);
        Stream st;
        if (held) CK(lens_loglike_batch_device(c, id, par.data(), 64, out.data(), &st));
        const int f = fake::ran("k_loglike_fp32") + fake::ran("k_split_bin");
        CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
        TRUE(fake::ran("k_loglike_fp32") + fake::ran("k_split_bin") > f && fake::outside == 0);
        TRUE(used(c) <= 16 * MB);
        CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
        TRUE(fake::outside == 0);
        lens_shutdown(c);
    }
}

// Device memory that others have taken: the split scratch goes before any call is
// refused, though the budget has room.
void memory_shared_with_others()
{
    lens_ctx *c = open(1 << 30);
    const lens_id id = load(c);
    const int64_t n = 20000;
    std::vector<double> par((size_t)n * LENS_PARAM_STRIDE, 0.5), out(n);
    Stream st[3];
    for (Stream &s : st) CK(lens_loglike_batch_device(c, id, par.data(), 64, out.data(), &s));
    CK(lens_loglike_batch(c, id, par.data(), 64, out.data()));
    TRUE(fake::ran("k_split_bin") == 4);
    const size_t left = fake::hbm;
    fake::hbm = 0;
    lens_id other = 0;
    CK(try_load(c, &other, Kind()));                                          // a lens
    fake::hbm = 0;
    CK(lens_loglike_batch_device(c, id, par.data(), 64, out.data(), &st[0]));
    CK(lens_loglike_batch(c, id, par.data(), 64, out.data()));
    fake::hbm = left;
    lens_shutdown(c);
    // a stream's own scratch: the only memory that can be had for its constants
    c = open(1 << 30);
    const lens_id id2 = load(c);
    CK(lens_loglike_batch_device(c, id2, par.data(), 4000, out.data(), &st[0]));
    fake::hbm = 0;
    CK(lens_loglike_batch_device(c, id2, par.data(), n, out.data(), &st[0]));
    TRUE(fake::outside == 0);
    lens_shutdown(c);
}

// The split launches of a call: scratch of what the calls need, grown with them, and
// with too little of it for chunks that fill the chip the fused kernel.
void scratch_grows()
{
    const int64_t n = 20000;
    std::vector<double> par((size_t)n * LENS_PARAM_STRIDE, 0.5), out(n);
    Kind solved;   // split at any number of proposals
    solved.amps = LENS_AMP_NNLS;
    Stream st;
    lens_ctx *c = open(4096 * MB);
    lens_id id = load(c, solved);
    CK(lens_loglike_batch_device(c, id, par.data(), 1, out.data(), &st));
    const int64_t one = used(c);
    CK(lens_loglike_batch_device(c, id, par.data(), 100, out.data(), &st));
    TRUE(used(c) <= one + 8 * MB);       // not 256 MB for a few images
    CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
    TRUE(used(c) > one + 128 * MB && used(c) < one + 300 * MB);
    TRUE(fake::ran("k_loglike_nnls") == 0 && fake::outside == 0);
    lens_shutdown(c);

    // chunks of all the scratch that there may be, however little a chunk's work
    c = open(4096 * MB);
    Kind plain = solved;
    plain.s = 1;
    id = load(c, plain);
    CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
    TRUE(fake::ran("k_loglike_nnls") == 0 && fake::outside == 0);
    lens_shutdown(c);

    // little budget at the stream's first call, much at a later one
    c = open(1024 * MB);
    id = load(c, solved);
    std::vector<lens_id> fill;
    Kind big;
    big.px = 2048;
    lens_id l;
    while (try_load(c, &l, big) == LENS_OK) fill.push_back(l);
    TRUE(fill.size() > 2);
    CK(lens_unload(c, fill.back()));
    fill.pop_back();
    int split = fake::ran("k_split_conv"), fused = fake::ran("k_loglike_nnls");
    CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
    TRUE(used(c) <= 1024 * MB);
    // not a hundred chunks of a few proposals each
    TRUE(fake::ran("k_split_conv") - split <= 16 && fake::ran("k_split_conv") - split + fake::ran("k_loglike_nnls") - fused > 0);
    for (lens_id f : fill) CK(lens_unload(c, f));
    split = fake::ran("k_split_conv");
    fused = fake::ran("k_loglike_nnls");
    CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
    TRUE(fake::ran("k_split_conv") - split >= 1 && fake::ran("k_split_conv") - split <= 4);
    TRUE(fake::ran("k_loglike_nnls") == fused && fake::outside == 0);
    lens_shutdown(c);

    // a budget that never has much: no chunk fills the chip
    c = open(16 * MB);
    id = load(c, solved);
    split = fake::ran("k_split_conv");
    fused = fake::ran("k_loglike_nnls");
    CK(lens_loglike_batch_device(c, id, par.data(), n, out.data(), &st));
    TRUE(fake::ran("k_split_conv") == split && fake::ran("k_loglike_nnls") == fused + 1);
    CK(lens_loglike_batch_device(c, id, par.data(), 16, out.data(), &st));
    TRUE(fake::ran("k_split_conv") == split + 1 && fake::outside == 0);
    lens_shutdown(c);
}

// The serving streams get their split scratch back once the budget has room again.
void serving_scratch()
{
    lens_ctx *c = open(400 * MB);
    const lens_id id = load(c);
    std::vector<double> par((size_t)300 * LENS_PARAM_STRIDE, 0.5), out(300);
    const auto served = [&] {
        lens_req r = 0;
        CK(lens_submit(c, id, par.data(), 300, out.data(), &r));
        CK(lens_wait(c, r, -1));
    };
    served();
    TRUE(fake::ran("k_split_bin") == 1 && fake::ran("k_loglike_batch") == 0);
    std::vector<lens_id> fill;
    Kind big;
    big.px = 1024;
    lens_id l;
    while (try_load(c, &l, big) == LENS_OK) fill.push_back(l);
    const int b = fake::ran("k_loglike_batch"), s = fake::ran("k_split_bin");
    served();
    TRUE(fake::ran("k_loglike_batch") == b + 1 && fake::ran("k_split_bin") == s);
    for (lens_id f : fill) CK(lens_unload(c, f));
    for (int i = 0; i < 4; ++i) served();   // both streams
    TRUE(fake::ran("k_loglike_batch") == b + 1 && fake::ran("k_split_bin") == s + 4 && fake::outside == 0);
    lens_shutdown(c);
}

// Loading works on the context's own stream alone: an operation on the legacy default
// stream would wait for other threads' work and break their captures.
void load_stream()
{
    for (int autotune = 0; autotune < 2; ++autotune) {
        lens_init_opts o{};
        o.autotune = autotune;
        lens_ctx *c = nullptr;
        CK(lens_init(&o, &c));
        for (int prec = 0; prec < 4; ++prec) {
            Kind k;
            k.prec = prec;
            load(c, k);
        }
        lens_shutdown(c);
    }
    TRUE(fake::legacy_ops == 0);
}

// The autotuner times what a batch runs: the split launches where they are the rule,
// and every strip height with lists of its own.
void autotune_lists()
{
    lens_init_opts o{};
    o.autotune = 1;
    lens_ctx *c = nullptr;
    CK(lens_init(&o, &c));
    Kind k;
    k.prec = LENS_PREC_F16_SPLIT;
    k.px = 50;
    k.k = 21;
    std::vector<double> par(LENS_PARAM_STRIDE, 0.5);
    double out = 0.0;
    const lens_id f16 = load(c, k);
    TRUE(fake::ran("k_loglike_mfma") > 0 && fake::bad_lists == 0);
    k.prec = LENS_PREC_FP32;
    k.amps = LENS_AMP_NNLS;
    const lens_id solved = load(c, k);
    TRUE(fake::ran("k_split_bin") > 0 && fake::ran("k_loglike_nnls") == 0 && fake::bad_lists == 0);
    CK(lens_loglike_batch(c, f16, par.data(), 1, &out));
    CK(lens_loglike_batch(c, solved, par.data(), 1, &out));
    TRUE(fake::bad_lists == 0);
    lens_shutdown(c);
}

const std::map<std::string, std::function<void()>> scenarios = {
    {"load_stream", load_stream},
    {"autotune_lists", autotune_lists},
    {"serving_scratch", serving_scratch},
    {"scratch_grows", scratch_grows},
    {"memory_shared_with_others", memory_shared_with_others},
    {"own_scratch", own_scratch},
    {"plan_scratch", plan_scratch},
};

}  // namespace

int main(int argc, char **argv)
{
    const auto it = argc == 2 ? scenarios.find(argv[1]) : scenarios.end();
    if (it == scenarios.end()) return 2;
    it->second();
    if (!fails) printf("ok\n");
    return fails ? 1 : 0;
}
