// A HIP runtime that runs nothing: device and pinned memory are host memory,
// launches are written to a log, every call succeeds at once.  Loaded before
// libflb.so it takes the place of the real one, so that the library's host
// side (launch grouping, transfers, tuning) can be tested without a GPU.
//
// What it keeps of the real one: a thread's current device; streams and events
// that belong to the device they were made on, and no event on a stream of
// another; streams under capture, which cannot be synchronised; freed pinned
// memory, which faults when touched.  Events take the time of a clock that the
// launches advance (hs_cost).  hs_hold stops calls of one function until
// hs_release, to put threads into a given order.
#include <cxxabi.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <chrono>
#include <condition_variable>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

namespace {

constexpr int kOk = 0, kInvalid = 1, kNoMemory = 2, kInvalidHandle = 400, kCapture = 900;

struct Dim {
    uint32_t x, y, z;
};
struct Stream {
    int device;
    bool capturing;
};
struct Event {
    int device;
    double ms;
};
struct Hold {
    const void *only = nullptr;  // calls on this object, or all
    bool armed = false;
    int held = 0;
};
struct State {
    std::mutex m;
    std::condition_variable cv;
    std::vector<std::string> log;
    std::map<const void *, std::string> kernels;
    std::map<std::string, Hold> holds;
    std::vector<std::pair<std::string, double>> costs;
    std::map<void *, size_t> pinned;
    size_t pinned_now = 0, pinned_peak = 0;
    double clock = 0.0;
};
State &st()
{
    static State *s = new State();
    return *s;
}
thread_local int t_device = 0;
thread_local struct {
    Dim grid, block;
    size_t lds;
    void *stream;
} t_config;

void stop(const char *fn, const void *object)
{
    State &s = st();
    std::unique_lock<std::mutex> lock(s.m);
    auto it = s.holds.find(fn);
    if (it == s.holds.end() || !it->second.armed) return;
    Hold &h = it->second;
    if (h.only && h.only != object) return;
    ++h.held;
    s.cv.notify_all();
    s.cv.wait(lock, [&] { return !h.armed; });
    --h.held;
    s.cv.notify_all();
}

void note(const char *fmt, ...) __attribute__((format(printf, 1, 2)));
void note(const char *fmt, ...)
{
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    std::lock_guard<std::mutex> lock(st().m);
    st().log.push_back(line);
}

}  // namespace

extern "C" {

// ------------------------------------------------------------ for the tests
void hs_hold(const char *fn, const void *object)
{
    std::lock_guard<std::mutex> lock(st().m);
    Hold &h = st().holds[fn];
    h.only = object;
    h.armed = true;
}
// whether n calls wait (after at most ms milliseconds)
int hs_held(const char *fn, int n, int ms)
{
    State &s = st();
    std::unique_lock<std::mutex> lock(s.m);
    Hold &h = s.holds[fn];
    return s.cv.wait_for(lock, std::chrono::milliseconds(ms), [&] { return h.held >= n; });
}
void hs_release(const char *fn)
{
    std::lock_guard<std::mutex> lock(st().m);
    st().holds[fn].armed = false;
    st().cv.notify_all();
}
void hs_cost(const char *part_of_name, double ms)
{
    std::lock_guard<std::mutex> lock(st().m);
    st().costs.emplace_back(part_of_name, ms);
}
int hs_log_size()
{
    std::lock_guard<std::mutex> lock(st().m);
    return (int)st().log.size();
}
const char *hs_log(int i) { return st().log[i].c_str(); }
void hs_log_clear()
{
    std::lock_guard<std::mutex> lock(st().m);
    st().log.clear();
}
size_t hs_pinned_now() { return st().pinned_now; }
size_t hs_pinned_peak() { return st().pinned_peak; }
void hs_capture(void *stream, int on) { static_cast<Stream *>(stream)->capturing = on != 0; }

// --------------------------------------------------------------- the runtime
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *)
{
    int status = 0;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::lock_guard<std::mutex> lock(st().m);
    st().kernels[host] = status == 0 ? plain : name;
    free(plain);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    t_config = {grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = t_config.grid;
    *block = t_config.block;
    *lds = t_config.lds;
    *stream = t_config.stream;
    return kOk;
}
// Log: "launch <kernel> grid=.. stream=.. src=.. dst=.. steps=..", the last
// three for the kernels that step from one buffer into another.
int hipLaunchKernel(const void *fn, Dim grid, Dim, void **args, size_t, void *stream)
{
    std::string name;
    {
        std::lock_guard<std::mutex> lock(st().m);
        name = st().kernels[fn];
        for (const auto &c : st().costs)
            if (name.find(c.first) != std::string::npos) {
                st().clock += c.second;
                break;
            }
    }
    const std::string anonymous = "(anonymous namespace)::";
    for (size_t at; (at = name.find(anonymous)) != std::string::npos;) name.erase(at, anonymous.size());
    name = name.substr(0, name.find('('));
    const size_t at = name.find("flbdev::");
    if (at != std::string::npos) name = name.substr(at + 8);
    auto is = [&](const char *k) { return name.compare(0, strlen(k), k) == 0; };
    void *src = nullptr, *dst = nullptr;
    int steps = 0;
    if (is("step_kernel") || is("step2_") || is("step3_") || is("march_") || is("patch_")) {
        src = static_cast<void **>(args[0])[0];
        dst = static_cast<void **>(args[0])[1];
        steps = is("step2_") ? 2 : is("step3_") ? 3 : 1;
        if (is("patch_")) steps = *static_cast<int *>(args[3]);
        if (is("march_")) steps = atoi(name.c_str() + name.rfind(',') + 1);
    } else if (is("dq_step_") || is("dq_line_kernel")) {
        src = *static_cast<void **>(args[0]);
        dst = *static_cast<void **>(args[1]);
        steps = is("dq_line_kernel") ? *static_cast<int *>(args[4]) : 1;
    }
    for (char &c : name)
        if (c == ' ') c = '_';
    note("launch %s grid=%u stream=%p src=%p dst=%p steps=%d", name.c_str(), grid.x, stream, src,
         dst, steps);
    stop("hipLaunchKernel", stream);
    return kOk;
}
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;  // compute units
    return kOk;
}
int hipGetDevice(int *d)
{
    *d = t_device;
    return kOk;
}
int hipSetDevice(int d)
{
    t_device = d;
    return kOk;
}
int hipGetLastError() { return kOk; }
const char *hipGetErrorString(int e) { return e == kInvalidHandle ? "invalid handle" : "error"; }
int hipGetSymbolAddress(void **, const void *) { return kInvalid; }

int hipStreamCreateWithFlags(void **s, unsigned)
{
    *s = new Stream{t_device, false};
    return kOk;
}
int hipStreamDestroy(void *s)
{
    delete static_cast<Stream *>(s);
    return kOk;
}
int hipStreamSynchronize(void *s)
{
    stop("hipStreamSynchronize", s);
    return s && static_cast<Stream *>(s)->capturing ? kCapture : kOk;
}
int hipStreamWaitEvent(void *s, void *e, unsigned)
{
    note("wait stream=%p event=%p", s, e);
    return kOk;
}
int hipStreamIsCapturing(void *s, int *status)
{
    *status = s && static_cast<Stream *>(s)->capturing ? 1 : 0;
    return kOk;
}
int hipEventCreateWithFlags(void **e, unsigned)
{
    *e = new Event{t_device, 0.0};
    return kOk;
}
int hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void *e)
{
    delete static_cast<Event *>(e);
    return kOk;
}
int hipEventRecord(void *e, void *s)
{
    Event *ev = static_cast<Event *>(e);
    if (s && static_cast<Stream *>(s)->device != ev->device) return kInvalidHandle;
    note("record stream=%p event=%p", s, e);
    std::lock_guard<std::mutex> lock(st().m);
    ev->ms = st().clock;
    return kOk;
}
int hipEventSynchronize(void *e)
{
    stop("hipEventSynchronize", nullptr);
    (void)e;
    return kOk;
}
int hipEventElapsedTime(float *ms, void *a, void *b)
{
    *ms = (float)(static_cast<Event *>(b)->ms - static_cast<Event *>(a)->ms);
    return kOk;
}
int hipMalloc(void **p, size_t n)
{
    *p = calloc(1, n ? n : 1);
    return *p ? kOk : kNoMemory;
}
int hipFree(void *p)
{
    free(p);
    return kOk;
}
int hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (*p == MAP_FAILED) return kNoMemory;
    note("hipHostMalloc bytes=%zu", n);
    std::lock_guard<std::mutex> lock(st().m);
    st().pinned[*p] = n;
    st().pinned_now += n;
    if (st().pinned_now > st().pinned_peak) st().pinned_peak = st().pinned_now;
    return kOk;
}
int hipHostFree(void *p)
{
    stop("hipHostFree", nullptr);
    size_t n = 0;
    {
        std::lock_guard<std::mutex> lock(st().m);
        n = st().pinned[p];
        st().pinned_now -= n;
        st().pinned.erase(p);
    }
    note("hipHostFree bytes=%zu", n);
    return mprotect(p, n, PROT_NONE) == 0 ? kOk : kInvalid;
}
int hipMemcpy(void *d, const void *s, size_t n, int)
{
    memcpy(d, s, n);
    return kOk;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *)
{
    memcpy(d, s, n);
    return kOk;
}
int hipMemsetAsync(void *d, int v, size_t n, void *)
{
    memset(d, v, n);
    return kOk;
}

}  // extern "C"
