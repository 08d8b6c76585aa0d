// Stand-in for the HIP runtime (test infrastructure, CPU only): the library's host
// code runs against it, no kernel does (but the self-test, on the host emulation).
// It keeps the documented order of work: a memset returns at once and happens on
// the null stream; a non-blocking stream does not wait for that one.  A launch on
// such a stream while a memset may still be on its way counts as a hazard.
#include "../kernel_emu/emu.cpp"

#include <map>
#include <string>

#define API extern "C" __attribute__((visibility("default")))

struct dim3 {
    uint32_t x, y, z;
};
struct Stream {
    bool blocking = true, capturing = false;
};
using stream_t = Stream *;

static std::recursive_mutex mu;
static std::map<const void *, std::string> names;
static int pending = 0;   // memsets on their way
static int hazards = 0, launches = 0;

static void on_stream(stream_t s) {   // work goes to s
    std::lock_guard<std::recursive_mutex> lk(mu);
    if (s && s->capturing) return;
    ++launches;
    if (s && !s->blocking) hazards += pending > 0;
    else pending = 0;   // (ordered after it)
}
static int waited() {   // the host waited for the null stream
    std::lock_guard<std::recursive_mutex> lk(mu);
    pending = 0;
    return 0;
}

API int fake_hazards(void) { return hazards; }
API int fake_launches(void) { return launches; }

API int hipMemset(void *, int, size_t) {
    std::lock_guard<std::recursive_mutex> lk(mu);
    ++pending;
    return 0;
}
API int hipMemsetAsync(void *, int, size_t, stream_t s) {
    on_stream(s);
    return 0;
}
API int hipDeviceSynchronize(void) { return waited(); }
API int hipStreamSynchronize(stream_t s) { return s && !s->blocking ? 0 : waited(); }

API int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t, stream_t s) {
    on_stream(s);
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
    on_stream(s);
    return 0;
}
API int hipMemcpyAsync(void *, const void *, size_t, int, stream_t s) {
    on_stream(s);
    return 0;
}
API int hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, int, stream_t s) {
    on_stream(s);
    return 0;
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
    delete s;
    return 0;
}
API int hipStreamBeginCapture(stream_t s, int) {
    s->capturing = true;
    return 0;
}
API int hipStreamEndCapture(stream_t s, void **g) {
    s->capturing = false;
    *g = nullptr;
    return 0;
}
API int hipStreamQuery(stream_t) { return 0; }
API int hipStreamWaitEvent(stream_t, void *, unsigned) { return 0; }
API int hipGraphInstantiate(void **e, void *, void *, char *, size_t) {
    *e = e;
    return 0;
}
API int hipGraphDestroy(void *) { return 0; }
API int hipGraphExecDestroy(void *) { return 0; }
API int hipEventCreateWithFlags(void **e, unsigned) {
    *e = e;
    return 0;
}
API int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
API int hipEventDestroy(void *) { return 0; }
API int hipEventElapsedTime(float *ms, void *, void *) {
    *ms = 0.0f;
    return 0;
}
API int hipEventQuery(void *) { return 0; }
API int hipEventRecord(void *, stream_t) { return 0; }
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
API int hipGetLastError(void) { return 0; }
API const char *hipGetErrorString(int) { return "fake"; }
