// Stand-in for the HIP runtime (test infrastructure, CPU only): the library's host
// code runs against it, no kernel does (but the self-test, on the host emulation).
// It keeps the documented order of work: a memset returns at once and happens on
// the null stream; a non-blocking stream does not wait for that one.  A launch on
// such a stream while a memset may still be on its way counts as a hazard.
// A device synchronisation while any stream is being captured fails and breaks that
// capture; the launches that follow are refused, but events are still recorded and
// waited for, and a stream forked by them is no part of the capture (all measured on
// ROCm 7.0).  What a capturing thread sends to a stream that is not capturing runs at
// once and counts as stray.
#include "../kernel_emu/emu.cpp"

#include <chrono>
#include <map>
#include <set>
#include <string>

#define API extern "C" __attribute__((visibility("default")))

struct dim3 {
    uint32_t x, y, z;
};
struct Stream {
    bool blocking = true, capturing = false, broken = false;
    Stream *origin = nullptr;   // of the capture that this one was forked into
};
struct Event {
    Stream *captured = nullptr;
};
using stream_t = Stream *;

static std::recursive_mutex mu;
static std::map<const void *, std::string> names;
static int pending = 0;   // memsets on their way
static int hazards = 0, launches = 0, breaks = 0;
static int capture_ms = 0;   // how long a capture takes at least
static std::set<stream_t> captures;
static std::map<stream_t, std::set<stream_t>> forked;
static thread_local int last_error = 0, capturing_here = 0;
static int strays = 0;
constexpr int kUnsupported = 900, kInvalidated = 901;

static int on_stream(stream_t s) {   // work goes to s
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (s && s->capturing) return s->broken ? last_error = kInvalidated : 0;
    ++launches;
    strays += capturing_here;
    if (s && !s->blocking) hazards += pending > 0;
    else pending = 0;   // (ordered after it)
    return 0;
}
static int waited() {   // the host waited for the null stream
    std::lock_guard<std::recursive_mutex> lk(mu);
    pending = 0;
    return 0;
}

API int fake_hazards(void) { return hazards; }
API int fake_launches(void) { return launches; }
API int fake_breaks(void) { return breaks; }
API int fake_strays(void) { return strays; }
API void fake_capture_ms(int ms) { capture_ms = ms; }

API int hipMemset(void *, int, size_t) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    ++pending;
    return 0;
}
API int hipMemsetAsync(void *, int, size_t, stream_t s) {
    return on_stream(s);
}
API int hipDeviceSynchronize(void) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (captures.empty()) return waited();
    for (stream_t s : captures) s->broken = true;
    ++breaks;
    return last_error = kUnsupported;
}
API int hipStreamSynchronize(stream_t s) { return s && !s->blocking ? 0 : waited(); }

API int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, stream_t s) {
    if (int e = on_stream(s)) return e;
    if (names[f].find("self_test") != std::string::npos) {
        uint32_t *out = *(uint32_t **)args[0];
        const uint32_t n = *(uint32_t *)args[1];
        for (uint32_t b = 0; b < grid.x; ++b)
            for (uint32_t w = 0; w < block.x / 64; ++w) {   // one emulated wave after the other
                kemu::blockIdx_.x = b * (block.x / 64) + w;
                kemu::blockDim_.x = 64;
                if (!kemu::run_wave([&] { rk::self_test(out, n); }, 16)) std::abort();
            }
    }
    return 0;
}
API int hipGraphLaunch(void *, stream_t s) {
    return on_stream(s);
}
API int hipMemcpyAsync(void *, const void *, size_t, int, stream_t s) {
    return on_stream(s);
}
API int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, stream_t s) {
    return on_stream(s);
}

static thread_local dim3 cfg_grid, cfg_block;
static thread_local size_t cfg_lds;
static thread_local stream_t cfg_stream;
API int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, stream_t s) {
    cfg_grid = g;
    cfg_block = b;
    cfg_lds = lds;
    cfg_stream = s;
    return 0;
}
API int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, stream_t *s) {
    *g = cfg_grid;
    *b = cfg_block;
    *lds = cfg_lds;
    *s = cfg_stream;
    return 0;
}
API void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
API void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *,
                               dim3 *, int *) {
    names[host] = name;
}
API void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
API void __hipUnregisterFatBinary(void **) {}

API int hipMalloc(void **p, size_t n) { return (*p = std::malloc(n)) ? 0 : 2; }
API int hipFree(void *p) {
    std::free(p);
    return 0;
}
API int hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? 0 : 2; }
API int hipHostFree(void *p) { return hipFree(p); }
API int hipGetSymbolAddress(void **p, const void *s) {
    *p = (void *)s;
    return 0;
}

API int hipStreamCreateWithFlags(stream_t *s, unsigned flags) {
    *s = new Stream();
    (*s)->blocking = (flags & 1u) == 0u;
    return 0;
}
API int hipStreamDestroy(stream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    for (auto &f : forked) f.second.erase(s);
    forked.erase(s);
    delete s;
    return 0;
}
API int hipStreamBeginCapture(stream_t s, int) {
    {
        std::lock_guard<std::recursive_mutex> lk(mu);
        s->capturing = true;
        s->broken = false;
        captures.insert(s);
        capturing_here = 1;
    }
    std::this_thread::sleep_for(std::chrono::milliseconds(capture_ms));
    return 0;
}
API int hipStreamEndCapture(stream_t s, void **g) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    captures.erase(s);
    capturing_here = 0;
    *g = nullptr;
    if (s->broken) return last_error = kInvalidated;   // (stays so)
    s->capturing = false;
    for (stream_t f : forked[s]) f->capturing = false;
    forked.erase(s);
    return 0;
}
API int hipStreamQuery(stream_t) { return 0; }
API int hipStreamIsCapturing(stream_t s, int *status) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    *status = !s->capturing ? 0 : s->broken ? 2 : 1;
    return 0;
}
API int hipStreamWaitEvent(stream_t s, Event *e, unsigned) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (!e->captured || s->capturing) return 0;
    s->capturing = true;
    forked[s->origin = e->captured].insert(s);
    return 0;
}
API int hipGraphInstantiate(void **e, void *, void *, char *, size_t) {
    *e = e;
    return 0;
}
API int hipGraphDestroy(void *) { return 0; }
API int hipGraphExecDestroy(void *) { return 0; }
API int hipEventCreateWithFlags(Event **e, unsigned) {
    *e = new Event();
    return 0;
}
API int hipEventCreate(Event **e) { return hipEventCreateWithFlags(e, 0); }
API int hipEventDestroy(Event *e) {
    delete e;
    return 0;
}
API int hipEventElapsedTime(float *ms, void *, void *) {
    *ms = 0.0f;
    return 0;
}
API int hipEventQuery(void *) { return 0; }
API int hipEventRecord(Event *e, stream_t s) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    e->captured = s && s->capturing && !s->broken ? (s->origin ? s->origin : s) : nullptr;
    return 0;
}
API int hipEventSynchronize(void *) { return 0; }
API int hipGetDevice(int *d) {
    *d = 0;
    return 0;
}
API int hipGetDeviceCount(int *n) {
    *n = 1;
    return 0;
}
API int hipSetDevice(int) { return 0; }
API int hipDeviceGetAttribute(int *v, int, int) {
    *v = 256;
    return 0;
}
API int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 2;
    return 0;
}
API int hipGetLastError(void) {
    const int e = last_error;
    last_error = 0;
    return e;
}
API const char *hipGetErrorString(int) { return "fake"; }
