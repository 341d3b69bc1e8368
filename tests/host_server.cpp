// The server's host code (ps_server.cpp, ps_protocol.cpp, ps_layout.cpp) on a
// machine without a GPU: the HIP calls it makes, with host memory as device
// memory, and its kernel launches run as plain loops over the coordinates, each
// logged. tests/host_server.py builds it all into one shared library with the C
// ABI of include/ps.h and these calls beside it:
//
//   host_reset(run)        clear the log and the planned failure; run = 0: launches
//                          are logged and not run, and device memory is address
//                          space that nothing touches (for vectors of any length)
//   host_launches()        launches logged
//   host_launch(i, out)    the i-th: kind (0 apply, 1 synchronous step, 2 pull, 3 steps,
//                          4 synchronous steps), k, r, gradient and replica type, fronts_log2,
//                          blocks per CU, group
//   host_fail_launch(i)    the launch that would be logged as the i-th (and no other)
//                          fails, and does nothing; -1: none
//   host_fail_alloc(i)     the i-th allocation from now on that the server makes throws;
//                          -1: none. Returns what was left of the count before
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <functional>
#include <new>
#include <vector>

#include "ps_kernels.h"

static long g_allocs = -1;   // until the one that throws
static bool g_own = false;   // in this file: none of these throws

void *operator new(size_t n) {
    if (!g_own && g_allocs >= 0 && g_allocs-- == 0) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

namespace {

struct Logged {
    int v[8];
};
std::vector<Logged> g_log;
long g_fail = -1;
bool g_run = true;

// A captured graph: the launches made while its stream was captured.
using Work = std::vector<std::function<void()>>;
Work *g_capture = nullptr;

template <class F>
hipError_t launch(const Logged &l, F work) {
    struct Own {
        Own() { g_own = true; }
        ~Own() { g_own = false; }
    } own;
    if (g_fail == static_cast<long>(g_log.size())) {
        g_fail = -1;
        return hipErrorLaunchFailure;
    }
    g_log.push_back(l);
    if (g_capture) g_capture->push_back(work);
    else if (g_run) work();
    return hipSuccess;
}

float widen(uint16_t b) {
    const uint32_t u = static_cast<uint32_t>(b) << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

uint16_t narrow(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40);
    return static_cast<uint16_t>((u + 0x7fff + ((u >> 16) & 1)) >> 16);
}

float load(const void *g, int dtype, uint64_t i) {
    if (dtype == PS_BF16) {
        uint16_t b;
        std::memcpy(&b, static_cast<const char *>(g) + 2 * i, 2);
        return widen(b);
    }
    float f;
    std::memcpy(&f, static_cast<const char *>(g) + 4 * i, 4);
    return f;
}

void store(void *d, int dtype, uint64_t i, float w) {
    if (dtype == PS_BF16) {
        const uint16_t b = narrow(w);
        std::memcpy(static_cast<char *>(d) + 2 * i, &b, 2);
    } else {
        std::memcpy(static_cast<char *>(d) + 4 * i, &w, 4);
    }
}

void step(float &w, float *v, float g, float lr, float m) {
    if (v) {
        const float t = m * *v;
        *v = t + g;
        const float p = lr * *v;
        w = w - p;
    } else {
        const float p = lr * g;
        w = w - p;
    }
}

// The kernels' order: a coordinate's gradients are all read before its
// replicas are written, and coordinates do not wait for each other.
void run_steps(const gadei::StepsArgs &a, bool sync, int gdt, int pdt) {
    for (uint64_t i = 0; i < a.n; ++i) {
        float g[PS_MAX_QUEUE_DEPTH];
        for (int j = 0; j < a.k; ++j) g[j] = load(a.g[j], gdt, i);
        float w = a.w[i], v = a.v ? a.v[i] : 0.0f, s = 0.0f;
        int r = 0, count = 0;
        for (int j = 0; j < a.k; ++j) {
            const int mark = static_cast<int>(a.rend[j >> 3] >> (8 * (j & 7))) & 255;
            if (sync) {
                s = s + g[j];
                ++count;
                if (mark & gadei::kLastOfStep) {
                    const float kf = static_cast<float>(count);
                    step(w, a.v ? &v : nullptr, s / kf, a.lr, a.m);
                    s = 0.0f;
                    count = 0;
                }
            } else {
                step(w, a.v ? &v : nullptr, g[j], a.lr, a.m);
            }
            for (const int end = mark & (gadei::kLastOfStep - 1); r < end; ++r)
                store(a.dst[r], pdt, i, w);
        }
        a.w[i] = w;
        if (a.v) a.v[i] = v;
    }
}

}  // namespace

namespace gadei {

hipError_t launch_apply(const ApplyArgs &a, int gdt, int pdt, int, const Shape &s, const Geometry &,
                        hipStream_t) {
    StepsArgs x;
    std::memset(&x, 0, sizeof x);
    static_cast<ApplyArgs &>(x) = a;
    x.rend[(a.k - 1) >> 3] = static_cast<uint64_t>(a.r) << (8 * ((a.k - 1) & 7));
    return launch({{0, a.k, a.r, gdt, pdt, a.fronts_log2, s.blocks_per_cu, s.group}},
                  [=] { run_steps(x, false, gdt, pdt); });
}

hipError_t launch_sync(const ApplyArgs &a, int gdt, int, const Shape &s, const Geometry &,
                       hipStream_t) {
    StepsArgs x;
    std::memset(&x, 0, sizeof x);
    static_cast<ApplyArgs &>(x) = a;
    x.rend[(a.k - 1) >> 3] = static_cast<uint64_t>(kLastOfStep) << (8 * ((a.k - 1) & 7));
    return launch({{1, a.k, a.r, gdt, -1, a.fronts_log2, s.blocks_per_cu, s.group}},
                  [=] { run_steps(x, true, gdt, PS_F32); });
}

hipError_t launch_steps(const StepsArgs &a, bool sync, int gdt, int pdt, int blocks, const Geometry &,
                        hipStream_t) {
    return launch({{sync ? 4 : 3, a.k, a.r, gdt, pdt, a.fronts_log2, blocks, 0}},
                  [=] { run_steps(a, sync, gdt, pdt); });
}

hipError_t launch_pull(const PullArgs &a, int pdt, int, const Geometry &, hipStream_t) {
    return launch({{2, 0, a.r, -1, pdt, 0, 0, 0}}, [=] {
        for (int r = 0; r < a.r; ++r)
            for (uint64_t i = 0; i < a.n; ++i) store(a.dst[r], pdt, i, a.w[i]);
    });
}

hipError_t launch_zero(float *p, uint64_t n, hipStream_t) {
    if (g_run) std::memset(p, 0, n * sizeof(float));
    return hipSuccess;
}

unsigned blocks_per_cu_lds(int) { return 0; }

}  // namespace gadei

extern "C" {

void host_reset(int run) {
    g_log.clear();
    g_fail = -1;
    g_run = run != 0;
}
int host_launches(void) { return static_cast<int>(g_log.size()); }
void host_launch(int i, int *out) { std::memcpy(out, g_log[i].v, sizeof g_log[i].v); }
void host_fail_launch(int i) { g_fail = i; }
long host_fail_alloc(long i) {
    const long left = g_allocs;
    g_allocs = i;
    return left;
}

// ---------------------------------------------------------------- HIP

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error of the host build"; }
hipError_t hipMalloc(void **p, size_t bytes) {
    // (address space that is backed where it is touched)
    *p = mmap(nullptr, bytes + 64, PROT_READ | PROT_WRITE,
              MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (*p == MAP_FAILED) return hipErrorOutOfMemory;
    *static_cast<size_t *>(*p) = bytes + 64;
    *p = static_cast<char *>(*p) + 64;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (p) {
        char *base = static_cast<char *>(p) - 64;
        munmap(base, *reinterpret_cast<size_t *>(base));
    }
    return hipSuccess;
}
hipError_t hipMemset(void *p, int c, size_t n) {
    if (g_run) std::memset(p, c, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (g_run) std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(d, s, n, k);
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(reinterpret_cast<void *>(e));
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    g_capture = new Work;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = reinterpret_cast<hipGraph_t>(g_capture);
    g_capture = nullptr;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
    *e = reinterpret_cast<hipGraphExec_t>(new Work(*reinterpret_cast<Work *>(g)));
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
    if (g_run)
        for (const auto &f : *reinterpret_cast<Work *>(e)) f();
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    delete reinterpret_cast<Work *>(e);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    delete reinterpret_cast<Work *>(g);
    return hipSuccess;
}
hipError_t hipIpcGetMemHandle(hipIpcMemHandle_t *, void *) { return hipErrorNotSupported; }
hipError_t hipIpcOpenMemHandle(void **, hipIpcMemHandle_t, unsigned) { return hipErrorNotSupported; }
hipError_t hipIpcCloseMemHandle(void *) { return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *, size_t *, hipDeviceptr_t) {
    return hipErrorNotSupported;
}

}  // extern "C"
