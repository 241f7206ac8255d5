// The library's runtime (libscylla_pdhg.so) on a HIP runtime that has no
// device: the functions below replace libamdhip64's, device memory is host
// memory, and work queued on a stream is done when something waits for it, so
// what a queued kernel would read is what lies there by then, as on a stream
// that is behind.  Kernels do not run; of a few the driver does what the host
// reads afterwards (states), and of the others it checks the launch and, where
// they read staged data, what they would have read.
//
// usage: runtime_driver SCENARIO [args]; prints "ok" or what is wrong.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include "../../paper_2307_03466_amd/csrc/kernels.h"

using namespace scy;

namespace {

// (registered by the library's initialisers, which run before this file's)
std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> m;
    return m;
}
std::map<const char *, size_t> g_live;   // device allocations
size_t g_largest = 0;                    // bytes of the largest allocation
long g_mallocs = 0, g_fail_at = -1;      // hipMalloc calls; the one that fails
std::vector<std::function<void()>> g_queue;
hipStream_t g_capturing = nullptr;       // the library's own capture
bool g_caller_captures = false;          // the handle's stream is captured by the caller
std::map<std::string, long> g_launches;  // by kernel name
long g_faults = 0;
int g_checks_to_run = 1;                 // decisions after which every instance has stopped
long g_instantiate_ms = 0;               // time a graph takes to instantiate
std::vector<std::pair<uint64_t, uint64_t>> g_blends;  // sums of the bits that every blend read

void fault(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    if (g_faults++ < 10) {
        vprintf(fmt, ap);
        printf("\n");
    }
    va_end(ap);
}

void drain()
{
    std::vector<std::function<void()>> q;
    q.swap(g_queue);
    for (auto &f : q) f();
}

// Whether [p, p + bytes) is device memory.
bool on_device(const void *p, size_t bytes)
{
    if (!p) return false;
    auto it = g_live.upper_bound((const char *)p);
    if (it == g_live.begin()) return false;
    --it;
    return (const char *)p + bytes <= it->first + it->second;
}

uint64_t byte_sum(const uint8_t *p, size_t n)
{
    uint64_t s = n;
    for (size_t i = 0; p && i < n; ++i) s = s * 31 + p[i];
    return p ? s : 0;
}

// What a pass kernel reads and writes is device memory of the sizes it needs.
template <class V>
void check_pass(const std::string &name, const PassArgs<V> &p, bool check)
{
    auto is = [&](const char *k) { return name.find(k) != std::string::npos; };
    auto need = [&](const void *q, size_t bytes, const char *what) {
        if (!on_device(q, std::max<size_t>(bytes, 1))) fault("%s: %s", name.c_str(), what);
    };
    const bool combine = is("9k_combine") || is("15k_combine_check") || is("6k_bseg");
    const bool rows = is("10k_bcombine") || is("16k_bcombine_check");
    need(p.st, sizeof(InstState), "states");
    if (combine) {
        need(p.longs, 16 * (size_t)p.nlong, "long rows");
        // the last long row's segments (uploads are queued: read after them)
        const int4 *longs = p.longs;
        const int nlong = p.nlong;
        const void *seg = check ? (const void *)p.seg64 : (const void *)p.seg;
        const size_t width = check ? 8 : sizeof(V);
        if (is("15k_combine_check")) need(p.lpart, 8 * CHK * (size_t)nlong, "partials of long rows");
        if (on_device(longs, 16 * (size_t)nlong)) g_queue.push_back([=] {
            const int4 L = longs[nlong - 1];
            if (!on_device(seg, width * (size_t)(L.y + L.z))) fault("%s: segments", name.c_str());
        });
    } else if (rows) {
        need(p.ctiles, 16 * (size_t)p.nctiles, "combine tiles");
        if (check) need(p.P64, 8 * (size_t)p.B * p.rows, "block partials");
        else need(p.P, sizeof(V) * (size_t)p.B * p.rows, "block partials");
        if (check) need(p.part, 8 * CHK * (size_t)p.nctiles, "partials");
    } else if (is("6k_dpass")) {
        need(p.dtiles, 16 * (size_t)p.ndtiles, "direct tiles");
        need(p.gofs, 4, "offsets");
    } else {
        need(p.tiles, 16 * (size_t)p.ntiles, "tiles");
        if (is("7k_check")) need(p.part, 8 * CHK * (size_t)p.ntiles, "partials");
        if (is("7k_bpart")) {
            need(p.bptr, 4 * (size_t)p.B * (p.rows + 1), "block pointers");
            need(p.seg, 1, "segments");
        }
        if (is("7k_spass")) {
            need(p.gofs, 4, "offsets");
            need(p.sub, 0, "sub-tiles");
            if (p.xS > 0) {
                need(p.xP, sizeof(V) * (size_t)p.xS * p.rows, "slice partials");
                need(p.X.ptr, 4 * (size_t)p.xS * (p.rows + 1), "slice pointers");
                need(p.X.ent, 4, "slice entries");
                need(p.xsub, 16, "slice sub-tiles");
                need(p.xSq, 4, "slices");
            }
        }
        need(p.M.ptr, 4, "row pointers");
        need(p.M.ent, 4, "entries");
    }
}

template <class V>
void launched_t(const std::string &name, dim3 grid, void **args)
{
    if (name.find("k_norm_part") != std::string::npos) {
        const NormArgs a = *(NormArgs *)args[0];
        const BlendArgs b = *(BlendArgs *)args[1];
        if (name.find("Li1E") == std::string::npos) return;  // NORM_BLEND
        const InstInfo *info = a.info;
        const int q = a.q0;
        g_queue.push_back([=] {
            const size_t n = (size_t)(info[q].col1 - info[q].col0 + 7) / 8;
            g_blends.emplace_back(byte_sum(b.xbits, n), byte_sum(b.ibits, n));
        });
    } else if (name.find("k_begin") != std::string::npos) {
        const BeginArgs<V> a = *(BeginArgs<V> *)args[0];
        g_queue.push_back([=] {
            for (int q = 0; q < a.count; ++q) {
                a.mirror[q] = InstState{};
                a.mirror[q].status = a.limits && a.limits[q] <= 0 ? ST_ITER : ST_RUN;
            }
        });
    } else if (name.find("k_decide") != std::string::npos) {
        const DecideArgs d = *(DecideArgs *)args[0];
        const int count = (int)grid.x;
        g_queue.push_back([=] {
            if (--g_checks_to_run > 0) return;
            for (int q = 0; q < count; ++q) d.mirror[q].status = ST_ITER;
        });
    } else if (name.find("k_tiny") != std::string::npos) {
        const TinyArgs<V> a = *(TinyArgs<V> *)args[0];
        const int count = (int)grid.x;
        g_queue.push_back([=] {
            for (int q = 0; q < count; ++q) a.mirror[q].status = ST_ITER;
        });
    } else if (name.find("8PassArgs") != std::string::npos) {
        // (k_bpart and k_bseg take the check as an argument)
        const bool dynamic = name.find("7k_bpart") != std::string::npos || name.find("6k_bseg") != std::string::npos;
        check_pass<V>(name, *(PassArgs<V> *)args[0], dynamic ? *(int *)args[2] != 0 : name.find("check") != std::string::npos);
    }
}

}  // namespace

// ------------------------------------------------------------ the HIP runtime
extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *m;
    return &m;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, uint3 *, uint3 *, dim3 *,
                           dim3 *, int *)
{
    kernels()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

static dim3 g_grid, g_block;
static size_t g_shmem;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    g_grid = g;
    g_block = b;
    g_shmem = sh;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s)
{
    *g = g_grid;
    *b = g_block;
    *sh = g_shmem;
    *s = g_stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t)
{
    const std::string &name = kernels()[f];
    for (const char *base : {"k_norm_part", "k_take_avg", "k_tiny", "k_begin", "k_decide", "k_force_stop", "k_put"})
        if (name.find(base) != std::string::npos) ++g_launches[base];
    ++g_launches["all"];
    // the limit of a dimension: 2^32 - 1 threads
    if ((uint64_t)g.x * b.x >= (uint64_t)1 << 32 || g.x == 0) fault("%s: grid %u x %u", name.c_str(), g.x, b.x);
    // (what a graph launches is checked when it is captured)
    if (g_capturing && name.find("8PassArgs") == std::string::npos) return hipSuccess;
    // (the precision is the first template argument of every kernel concerned
    // but the decision's, which has none)
    const bool dbl = name.find("IdL") != std::string::npos || name.find("IdE") != std::string::npos;
    if (dbl) launched_t<double>(name, g, args);
    else launched_t<float>(name, g, args);
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    if (g_mallocs++ == g_fail_at) return hipErrorOutOfMemory;
    *p = calloc(n, 1);
    g_live[(char *)*p] = n;
    g_largest = std::max(g_largest, n);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    drain();
    auto it = g_live.find((char *)p);
    if (it == g_live.end()) return hipErrorInvalidValue;
    g_live.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = calloc(n, 1);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    if (!g_queue.empty()) fault("pinned memory freed under queued work");
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind k, hipStream_t)
{
    if (k == hipMemcpyHostToDevice) {
        std::vector<char> copy((const char *)src, (const char *)src + n);
        g_queue.push_back([dst, copy] { memcpy(dst, copy.data(), copy.size()); });
    } else {
        g_queue.push_back([=] { memcpy(dst, src, n); });
    }
    return hipSuccess;
}
hipError_t hipMemcpyWithStream(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t)
{
    drain();
    memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t)
{
    g_queue.push_back([=] { memset(p, v, n); });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    if (g_caller_captures) return hipErrorStreamCaptureUnsupported;
    drain();
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s)
{
    *s = g_caller_captures ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t)
{
    drain();
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    static uintptr_t n = 0;
    *s = (hipStream_t)(++n);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    g_capturing = s;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    g_capturing = nullptr;
    *g = (hipGraph_t)(uintptr_t)1;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    std::this_thread::sleep_for(std::chrono::milliseconds(g_instantiate_ms));
    *x = (hipGraphExec_t)(uintptr_t)1;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof(*p));
    strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 160 * 1024;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }

}  // extern "C"

namespace {

// m rows of `len` ones each over n columns.
struct Lp {
    std::vector<int64_t> ptr;
    std::vector<int32_t> col;
    std::vector<double> val, c, b, l, u;
    std::vector<char> sense;
    Lp(int m, int n, int len) : c(n, 1.0), b(m, 1.0), l(n, 0.0), u(n, 1.0), sense(m, 'G')
    {
        ptr.push_back(0);
        for (int i = 0; i < m; ++i) {
            const int first = (int)((int64_t)i * (n - len) / m);
            for (int k = 0; k < len; ++k) col.push_back(first + k);
            ptr.push_back((int64_t)col.size());
        }
        val.assign(col.size(), 1.0);
    }
    scylla_lp view() const
    {
        scylla_lp v{};
        v.A.m = (int32_t)b.size();
        v.A.n = (int32_t)c.size();
        v.A.nnz = (int64_t)col.size();
        v.A.row_ptr = ptr.data();
        v.A.col_idx = col.data();
        v.A.val = val.data();
        v.c = c.data();
        v.b = b.data();
        v.senses = sense.data();
        v.l = l.data();
        v.u = u.data();
        return v;
    }
};

scylla_params solve_params(int precision)
{
    scylla_params p;
    scylla_params_default(&p);
    p.precision = precision;
    p.autotune = 0;
    p.iter_limit = 128;
    return p;
}

scylla_batch *create(const std::vector<scylla_lp> &lps, int precision)
{
    scylla_batch *h = nullptr;
    if (scylla_batch_create(lps.data(), (int32_t)lps.size(), precision, nullptr, &h) != 0)
        fault("create: %s", scylla_last_error());
    return h;
}

void must(int rc, const char *what)
{
    if (rc != 0) fault("%s: %d %s", what, rc, scylla_last_error());
}

// Rounding bits staged by many updates while the stream is behind: every
// update must read its own.
void blends(int n, int updates, bool objectives)
{
    const Lp lp(4, n, 2), other(3, 5000, 2);
    scylla_batch *h = create({lp.view(), other.view()}, SCYLLA_FP32);
    std::vector<uint8_t> x((n + 7) / 8), i((n + 7) / 8);
    std::vector<double> c(5000);
    std::vector<std::pair<uint64_t, uint64_t>> want;
    for (int k = 0; k < updates; ++k) {
        for (size_t j = 0; j < x.size(); ++j) {
            x[j] = (uint8_t)(j * 7 + k);
            i[j] = (uint8_t)(j * 13 + 5 * k + 1);
        }
        want.emplace_back(byte_sum(x.data(), x.size()), byte_sum(i.data(), i.size()));
        must(scylla_batch_set_blend(h, 0, x.data(), i.data(), 0.5, 1.0), "set_blend");
        if (objectives && k % 3 == 0) must(scylla_batch_set_objective(h, 1, c.data()), "set_objective");
    }
    std::vector<double> out((size_t)n + 5000);
    must(scylla_batch_get_x_all(h, out.data()), "get_x_all");
    if (g_blends.size() != want.size()) fault("%zu blends of %zu", g_blends.size(), want.size());
    for (size_t k = 0; k < want.size() && k < g_blends.size(); ++k)
        if (g_blends[k] != want[k]) fault("update %zu read other bits", k);
    scylla_batch_destroy(h);
}

// One large LP among many small ones: launches and buffers grow with what
// there is, not with the number of instances times the largest.
void uneven(int small, int rows, int cols)
{
    const Lp big(rows, cols, 2), lp(1, 2, 1);
    std::vector<scylla_lp> lps(small, lp.view());
    lps.push_back(big.view());
    scylla_batch *h = create(lps, SCYLLA_FP32);
    const size_t bound = 64 * ((size_t)3 * rows + cols) + 1024 * (size_t)lps.size();
    if (g_largest > bound) fault("an allocation of %zu bytes", g_largest);
    scylla_params p = solve_params(SCYLLA_FP32);
    p.restart_avg = 1;
    std::vector<scylla_result> res(lps.size());
    if (h) must(scylla_batch_solve(h, &p, 0, res.data()), "solve");
    if (g_launches["k_take_avg"] == 0 || g_launches["k_norm_part"] != 1) fault("launches");
    scylla_batch_destroy(h);
}

// The fused window with the largest iteration limit there is.
void limit(int period)
{
    const Lp lp(5, 9, 2);
    scylla_batch *h = create({lp.view()}, SCYLLA_FP64);
    scylla_params p = solve_params(SCYLLA_FP64);
    p.check_period = period;
    scylla_result res;
    for (int64_t lim : {INT64_MAX, INT64_MAX - 1, INT64_MAX - period, (int64_t)0, (int64_t)1, (int64_t)period}) {
        p.iter_limit = lim;
        g_launches.clear();
        must(scylla_batch_solve(h, &p, 0, &res), "solve");
        if (g_launches["k_tiny"] != 1 || res.status != ST_ITER)
            fault("limit %lld: %ld launches, status %d", (long long)lim, g_launches["k_tiny"], res.status);
    }
    scylla_batch_destroy(h);
}

// Updates while the caller captures the handle's stream are refused and queue
// nothing.
void captured(int n)
{
    const Lp lp(4, n, 2);
    scylla_batch *h = create({lp.view()}, SCYLLA_FP32);
    std::vector<double> c(n, 2.0);
    std::vector<uint8_t> bits((n + 7) / 8, 5);
    must(scylla_batch_set_objective(h, 0, c.data()), "set_objective");
    must(scylla_batch_set_quadratic(h, 0, c.data()), "set_quadratic");
    must(hipStreamSynchronize(nullptr), "synchronize");
    g_caller_captures = true;
    const long before = g_launches["all"];
    if (scylla_batch_set_objective(h, 0, c.data()) >= 0) fault("set_objective is accepted");
    if (scylla_batch_set_quadratic(h, 0, c.data()) >= 0) fault("set_quadratic is accepted");
    if (scylla_batch_set_quadratic(h, 0, nullptr) >= 0) fault("set_quadratic (none) is accepted");
    if (scylla_batch_set_blend(h, 0, bits.data(), nullptr, 0.5, 1.0) >= 0) fault("set_blend is accepted");
    if (scylla_batch_set_blend(h, 0, bits.data(), bits.data(), 0.5, 1.0) >= 0) fault("set_blend (bits) is accepted");
    if (g_launches["all"] != before || !g_queue.empty()) fault("work was queued");
    g_caller_captures = false;
    must(scylla_batch_set_objective(h, 0, c.data()), "set_objective afterwards");
    scylla_batch_destroy(h);
}

// A graph that takes long to make (once for a layout and check period) does not
// use up a solve's time limit, nor count as its time.
void slow_graph()
{
    const Lp lp(300, 500, 3);
    scylla_batch *h = create({lp.view()}, SCYLLA_FP32);
    scylla_params p = solve_params(SCYLLA_FP32);
    p.fused_window = 0;
    p.iter_limit = 1 << 20;
    p.time_limit_s = 0.25;
    g_instantiate_ms = 500;
    for (int k = 0; k < 2; ++k) {
        g_checks_to_run = 4;
        scylla_result res;
        must(scylla_batch_solve(h, &p, 0, &res), "solve");
        if (g_launches["k_force_stop"] != 0) fault("solve %d was stopped", k);
        if (res.solve_seconds > 0.25) fault("solve %d took %g s", k, res.solve_seconds);
    }
    scylla_batch_destroy(h);
}

// Every allocation of a layout change or a solve fails once: the call says so,
// and whatever follows, the same call again or a solve, launches nothing on
// buffers that are not there.
void allocations(const std::string &what, int precision)
{
    // long rows (segments), an instance whose vectors fit the LDS, one whose
    // vectors only fit in slices
    const Lp one(40, 30000, 9000), two(300, 500, 3), three(100, 90000, 20);
    const std::vector<scylla_lp> lps = {one.view(), two.view(), three.view()};
    std::vector<scylla_result> res(lps.size());
    scylla_params p = solve_params(precision), avg = p;
    p.fused_window = avg.fused_window = 0;
    avg.restart_avg = 1;
    int layout[5] = {};
    if (sscanf(what.c_str(), "layout:%d,%d,%d,%d", layout, layout + 1, layout + 2, layout + 3) != 4) layout[1] = 0;
    auto change = [&](scylla_batch *h) {
        if (layout[1]) return scylla_batch_set_layout(h, layout[0], layout[1], layout[2], layout[3]);
        return scylla_batch_solve(h, &avg, 0, res.data());
    };
    for (int again = 0; again < 2; ++again) {
        long failed = 0;
        for (long k = 0;; ++k) {
            scylla_batch *h = create(lps, precision);
            if (!h) return;
            // from another layout with the same and with other tiles
            must(scylla_batch_set_layout(h, k % 2 ? 2 : 0, layout[1] ? layout[1] : 8, 0, 4), "first layout");
            g_fail_at = g_mallocs + k;
            const int rc = change(h);
            const bool reached = g_mallocs > g_fail_at;
            g_fail_at = -1;
            if (reached && rc != -12) fault("allocation %ld fails: %d", k, rc);
            if (!reached) must(rc, "no allocation fails");
            if (again) must(change(h), "again");
            must(scylla_batch_solve(h, &p, 0, res.data()), "solve");
            if (layout[1]) {
                double r, c;
                must(scylla_batch_time_passes(h, 1, &r, &c), "time_passes");
                must(change(h), "at last");
                must(scylla_batch_solve(h, &avg, 0, res.data()), "solve to the average");
            }
            scylla_batch_destroy(h);
            if (!reached) break;
            ++failed;
            if (g_faults > 0) {
                printf("(allocation %ld failed first, the call %s)\n", k, again ? "made again" : "not made again");
                return;
            }
        }
        if (failed == 0) fault("no allocation was reached");
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    auto arg = [&](int k) { return atoi(argv[k]); };
    if (what == "blends") blends(arg(2), arg(3), arg(4) != 0);
    else if (what == "uneven") uneven(arg(2), arg(3), arg(4));
    else if (what == "allocations") allocations(argv[2], arg(3));
    else if (what == "limit") limit(arg(2));
    else if (what == "captured") captured(arg(2));
    else if (what == "slow_graph") slow_graph();
    else fault("unknown scenario");
    if (g_faults == 0) printf("ok\n");
    return g_faults == 0 ? 0 : 1;
}
