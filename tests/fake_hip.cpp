// A HIP runtime for host tests: it runs no kernel and records what the library
// asks for, in order.  Loaded (globally) before libquan.so, whose hip* calls
// then come here: every host decision (plans, buffers, launches, locks) is the
// product's own.
#include <hip/hip_runtime_api.h>
#include <unistd.h>

#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <utility>
#include <vector>

namespace {

struct Event {
    char what;       // 'L' launch, 'M' malloc, 'F' free, 'S' memset, 'D' device and 'W' stream synchronize
    int tag;         // the calling thread's (fake_tag)
    void *stream;
    std::string name;  // of the kernel, mangled
    void *ptr;       // buffer, or a launch's first argument word
    size_t bytes;    // of a buffer; work-groups of a launch
    int in_capture;  // (of the launch's stream, or of any for the others)
};

std::mutex g_mutex;
std::vector<Event> g_events;
std::map<const void *, std::string> g_kernels;
std::map<char *, size_t> g_live;
std::set<void *> g_capturing;
char *g_next = reinterpret_cast<char *>(0x600000000000);
int g_delay_us = 0;
size_t g_limit = size_t(1) << 40;  // bytes that may be live
thread_local int t_tag = 0;
thread_local hipError_t t_last = hipSuccess;
thread_local hipStreamCaptureMode t_mode = hipStreamCaptureModeGlobal;

struct Config {
    dim3 grid, block;
    size_t shmem;
    hipStream_t stream;
};
thread_local std::vector<Config> t_configs;

hipError_t done(hipError_t e)
{
    if (e != hipSuccess)
        t_last = e;
    return e;
}

void add(char what, void *stream, const std::string &name, void *ptr, size_t bytes, int in_capture)
{
    g_events.push_back({what, t_tag, stream, name, ptr, bytes, in_capture});
}

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *module = nullptr;
    return &module;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *,
                           dim3 *, int *)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_kernels[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream)
{
    t_configs.push_back({grid, block, shmem, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *stream)
{
    const Config c = t_configs.back();
    t_configs.pop_back();
    *grid = c.grid;
    *block = c.block;
    *shmem = c.shmem;
    *stream = c.stream;
    return hipSuccess;
}

hipError_t hipGetDevice(int *dev)
{
    *dev = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;  // the one attribute asked for: compute units
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError()
{
    const hipError_t e = t_last;
    t_last = hipSuccess;
    return e;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char array[64];
    *p = array;
    return hipSuccess;
}

// As the runtime does while any stream is captured: the calls that touch
// memory or wait are refused, unless the thread is in the relaxed mode.
bool refused() { return !g_capturing.empty() && t_mode != hipStreamCaptureModeRelaxed; }

hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *mode)
{
    std::swap(*mode, t_mode);
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    size_t live = 0;
    for (const auto &b : g_live)
        live += b.second;
    const bool capturing = refused();
    if (capturing || live + bytes > g_limit) {
        add('M', nullptr, "refused", nullptr, bytes, capturing);
        return done(capturing ? hipErrorStreamCaptureUnsupported : hipErrorOutOfMemory);
    }
    *p = g_next;
    g_live[g_next] = bytes;
    g_next += (bytes + 4095) / 4096 * 4096 + 4096;
    add('M', nullptr, "", *p, bytes, 0);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    const bool capturing = refused();
    add('F', nullptr, capturing ? "refused" : "", p, 0, capturing);
    if (capturing)
        return done(hipErrorStreamCaptureUnsupported);
    return g_live.erase(static_cast<char *>(p)) ? hipSuccess : done(hipErrorInvalidValue);
}
hipError_t hipMemsetAsync(void *p, int, size_t bytes, hipStream_t s)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    add('S', s, "", p, bytes, int(g_capturing.count(s)));
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    std::lock_guard<std::mutex> lock(g_mutex);
    const bool capturing = !g_capturing.empty();  // in every mode
    add('D', nullptr, capturing ? "refused" : "", nullptr, 0, capturing);
    return capturing ? done(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    const bool capturing = refused();
    add('W', s, capturing ? "refused" : "", nullptr, 0, capturing);
    return capturing ? done(hipErrorStreamCaptureUnsupported) : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *status)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    *status = g_capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3, void **args, size_t, hipStream_t s)
{
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        void *first = nullptr;
        std::memcpy(&first, args[0], sizeof(first));
        add('L', s, g_kernels[fn], first, grid.x, int(g_capturing.count(s)));
    }
    // (another thread's launch comes between this call's, if it may)
    if (g_delay_us > 0)
        usleep(unsigned(g_delay_us));
    return hipSuccess;
}

// ---- for the tests
void fake_tag(int tag) { t_tag = tag; }
void fake_delay(int us) { g_delay_us = us; }
void fake_limit(size_t bytes) { g_limit = bytes; }
void fake_capture(void *stream, int on)
{
    std::lock_guard<std::mutex> lock(g_mutex);
    if (on)
        g_capturing.insert(stream);
    else
        g_capturing.erase(stream);
}
void fake_clear()
{
    std::lock_guard<std::mutex> lock(g_mutex);
    g_events.clear();
}
int fake_events() { return int(g_events.size()); }
char fake_event(int i, int *tag, void **stream, const char **name, void **ptr, size_t *bytes, int *in_capture)
{
    const Event &e = g_events[size_t(i)];
    *tag = e.tag;
    *stream = e.stream;
    *name = e.name.c_str();
    *ptr = e.ptr;
    *bytes = e.bytes;
    *in_capture = e.in_capture;
    return e.what;
}

}  // extern "C"
