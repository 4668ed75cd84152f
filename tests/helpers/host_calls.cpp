// The host side of libgccd against a HIP runtime of this file's own, on the CPU: device
// memory is host memory, launches do nothing and every call is noted.  The
// executable's definitions come before those of the HIP library.  Usage: host_calls
// CASE; prints what failed and exits with 1.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "gccd.h"

namespace {

struct Stream {
    long launches = 0;  // kernels given to it
};
struct Event {
    Stream* stream = nullptr;
    long launches = 0;
};

Stream null_stream;
Stream* of(hipStream_t s) { return s ? reinterpret_cast<Stream*>(s) : &null_stream; }

// (the library registers its kernels before this file's objects are made)
std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> k;
    return k;
}
std::vector<std::string> launched;            // kernel names, in order
std::map<Stream*, long> joined;               // launches of a stream that the null stream waits for
std::vector<Stream*> streams;
long fail_at = -1;                            // the launch to fail, counted down
hipError_t last_error = hipSuccess;
int captures = 0;
uint32_t holes = 0, after_step = 0;           // what the device counts say

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* handle = nullptr;
    return &handle;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
    kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
static dim3 pushed_grid, pushed_block;
static hipStream_t pushed_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t s) {
    pushed_grid = g;
    pushed_block = b;
    pushed_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
    *g = pushed_grid;
    *b = pushed_block;
    *m = 0;
    *s = pushed_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t s) {
    if (fail_at >= 0 && fail_at-- == 0) return last_error = hipErrorLaunchFailure;
    launched.push_back(kernels()[f]);
    ++of(s)->launches;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "planted"; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    return *n = 4, hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
    return (*p = std::calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorInvalidSymbol; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
    std::memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* n, hipDeviceptr_t p) {
    *base = p;
    *n = (size_t)1 << 40;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
    std::memcpy(d, s, n);
    if (k == hipMemcpyDeviceToHost) {  // the counts: words 0-2 holes, 4 last step; or per event
        uint32_t* w = static_cast<uint32_t*>(d);
        w[0] = holes;
        if (n == 64) w[1] = w[2] = holes, w[3] = 0u, w[4] = after_step;
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    return hipMemcpyAsync(d, s, n, k, nullptr);
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    streams.push_back(new Stream);
    *s = reinterpret_cast<hipStream_t>(streams.back());
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    joined[of(s)] = of(s)->launches;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete reinterpret_cast<Event*>(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    *reinterpret_cast<Event*>(e) = Event{of(s), of(s)->launches};
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    const Event& ev = *reinterpret_cast<Event*>(e);
    if (of(s) == &null_stream && ev.stream) joined[ev.stream] = ev.launches;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = reinterpret_cast<hipGraph_t>(&captures);
    return hipSuccess;
}
hipError_t hipGraphGetNodes(hipGraph_t, hipGraphNode_t*, size_t* n) { return *n = 0, hipSuccess; }
hipError_t hipGraphNodeGetType(hipGraphNode_t, hipGraphNodeType*) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
    ++captures;
    *x = reinterpret_cast<hipGraphExec_t>(&captures);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"

namespace {

int failures = 0;
#define EXPECT(cond, ...)                   \
    do {                                    \
        if (!(cond)) {                      \
            std::printf(__VA_ARGS__);       \
            std::printf(" (%s)\n", #cond);  \
            ++failures;                     \
        }                                   \
    } while (0)

struct Context {
    gccd_ctx* c = nullptr;
    std::vector<double> p, out;
    std::vector<float> rho = std::vector<float>(32 * 32 * 32), w;
    explicit Context(bool closure = false) {
        gccd_params q{};
        q.abi_version = GCCD_ABI_VERSION;
        q.thickness_um = 675.0;
        q.a1_Vcm_per_um = 3.0;
        q.a2_Vcm = 2200.0;
        q.temperature_K = 140.0;
        q.eps_r = 11.7;
        q.softening_um = 1e-3;
        q.coulomb = q.diffusion = q.collected_are_sources = 1;
        if (gccd_init(&q, nullptr, &c) != GCCD_OK) std::exit(2);
        if (closure) {
            w.assign(GCCD_CLOSURE_WEIGHTS, 0.01f);
            if (gccd_set_closure(c, w.data(), (int64_t)w.size(), 0) != GCCD_OK) std::exit(2);
        }
    }
    ~Context() { gccd_destroy(c); }
    int load(int64_t n) {
        holes = (uint32_t)n;
        p.assign(n, 300.0);
        out.assign(n, 0.0);
        return gccd_load(c, n, p.data(), p.data(), p.data());
    }
    int run(int64_t steps) {
        gccd_stats_t s;
        if (gccd_stats(c, &s) != GCCD_OK) return -99;
        after_step = (uint32_t)(s.step + steps);
        return gccd_run(c, dt, steps, nullptr, nullptr);
    }
    int field() { return gccd_field(c, out.data(), out.data(), out.data()); }
    int parts() {
        double* o = out.data();
        return gccd_closure_parts(c, o, o, o, o, o, o, rho.data(), o);
    }
    double dt = 10.0;
};

// Whatever launch of a closure call fails, the caller's stream has to be waiting for
// the near sum on the side stream when the call returns.
void join() {
    for (int call = 0; call < 3; ++call) {
        for (long k = 0;; ++k) {
            Context x(true);
            if (x.load(3000) != GCCD_OK) std::exit(2);
            fail_at = k;
            const int r = call == 0 ? x.run(1) : call == 1 ? x.field() : x.parts();
            const bool hit = fail_at < 0;
            fail_at = -1;
            last_error = hipSuccess;
            for (Stream* s : streams)
                EXPECT(joined[s] == s->launches, "call %d, launch %ld failed: %ld of %ld joined",
                       call, k, joined[s], s->launches);
            if (!hit) {
                EXPECT(r == GCCD_OK && k > 20, "call %d: status %d after %ld launches", call, r, k);
                break;
            }
            EXPECT(r == GCCD_E_DEVICE, "call %d, launch %ld: status %d", call, k, r);
        }
    }
}

// The tuner after a field call between sorts: the field call left its own order's
// positions, so the tuner has to gather the run's before it times a launch.
void autotune() {
    Context x;
    EXPECT(x.load(3000) == GCCD_OK && x.run(5) == GCCD_OK && x.field() == GCCD_OK, "set-up");
    launched.clear();
    EXPECT(gccd_autotune(x.c, nullptr, nullptr, nullptr) == GCCD_OK, "autotune");
    for (const std::string& s : launched) {
        if (s.find("gather") != std::string::npos) return;
        if (s.find("field") != std::string::npos) break;
    }
    EXPECT(false, "the first timed launch runs over the field call's positions");
}

// The steps captured for a load serve the next one of the same shape.
void graphs() {
    for (int64_t n : {700, 20000, 75000}) {  // (from 5e9 pairs on pipelined)
        Context x;
        captures = 0;
        auto pass = [&](int64_t m, int steps, int want, const char* what) {
            EXPECT(x.load(m) == GCCD_OK && x.run(steps) == GCCD_OK, "%s", what);
            EXPECT(captures == want, "%ld holes, %s: %d captures, not %d", (long)n, what, captures,
                   want);
        };
        pass(n, 64, 1, "first load");
        pass(n, 64, 1, "same shape");
        pass(n, 96, 1, "same shape, longer");
        pass(n + 1, 64, 2, "another shape");
        pass(n, 64, 3, "the first shape");
        x.dt = 5.0;
        pass(n, 64, 4, "another time step");
        // the closure's buffers may grow past the captured ones: at most one capture more
        x.w.assign(GCCD_CLOSURE_WEIGHTS, 0.01f);
        EXPECT(gccd_set_closure(x.c, x.w.data(), (int64_t)x.w.size(), 0) == GCCD_OK, "closure");
        EXPECT(x.load(n) == GCCD_OK && x.run(40) == GCCD_OK && x.parts() == GCCD_OK, "closure");
        EXPECT(captures == 4, "closure steps were captured");
        EXPECT(gccd_set_closure(x.c, nullptr, 0, 0) == GCCD_OK, "closure off");
        EXPECT(x.load(n) == GCCD_OK && x.run(64) == GCCD_OK && captures <= 5, "%d", captures);
        const int after = captures;
        pass(n, 64, after, "same shape after the closure");
        gccd_stats_t s;
        EXPECT(gccd_stats(x.c, &s) == GCCD_OK && s.graph_usable == 1 && s.graph_replays == 17,
               "%ld replays", (long)s.graph_replays);
    }
}

}  // namespace

int main(int argc, char** argv) {
    const std::string c = argc > 1 ? argv[1] : "";
    if (c == "join")
        join();
    else if (c == "autotune")
        autotune();
    else if (c == "graphs")
        graphs();
    else
        return 2;
    return failures ? 1 : 0;
}
