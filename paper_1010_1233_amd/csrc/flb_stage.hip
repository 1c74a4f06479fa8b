// flb_stage.hip -- see flb_stage.h.
#include "flb_stage.h"

#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace flbdev {

namespace {

std::mutex g_use;    // one transfer at a time; guards the slots
std::mutex g_count;  // guards the reference count
int g_refs = 0;
double *g_slots = nullptr;

// (caller holds g_use)
hipError_t slots(double **p)
{
    if (!g_slots) {
        void *m = nullptr;
        // portable: the transfers of every device go through the same slots
        const hipError_t e = hipHostMalloc(&m, kStageSlots * kStageSlotDoubles * sizeof(double),
                                           hipHostMallocPortable);
        if (e != hipSuccess) return e;
        g_slots = static_cast<double *>(m);
    }
    *p = g_slots;
    return hipSuccess;
}

hipError_t transfer(int device, hipStream_t s, double *host, size_t n, bool to_host,
                    const StageKernel &kernel)
{
    if (!n) return hipStreamSynchronize(s);
    std::lock_guard<std::mutex> use(g_use);
    double *slot0 = nullptr;
    hipError_t e = slots(&slot0);
    if (e != hipSuccess) return e;
    const size_t chunks = (n + kStageSlotDoubles - 1) / kStageSlotDoubles;
    if (chunks == 1) {
        if (!to_host) memcpy(slot0, host, n * sizeof(double));
        if ((e = kernel(slot0, 0, n, s)) != hipSuccess) return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (to_host) memcpy(host, slot0, n * sizeof(double));
        return hipSuccess;
    }

    // worker w takes the chunks w, w + workers, ...
    const int workers = (int)std::min<size_t>(chunks, kStageSlots);
    std::mutex enqueue;
    std::atomic<int> failed{0};
    std::atomic<size_t> turn{0};
    auto work = [&](bool own_thread) {
        if (own_thread) {
            const hipError_t d = hipSetDevice(device);
            if (d != hipSuccess) {
                failed = d;
                return;
            }
        }
        hipEvent_t ev = nullptr;
        hipError_t q = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        const int w = (int)(turn++ % kStageSlots);
        double *slot = slot0 + (size_t)w * kStageSlotDoubles;
        bool pending = false;  // a kernel may still read the slot
        for (size_t c = (size_t)w; c < chunks && q == hipSuccess && !failed; c += workers) {
            const size_t first = c * kStageSlotDoubles;
            const size_t m = std::min(kStageSlotDoubles, n - first);
            if (!to_host) {
                if (pending) q = hipEventSynchronize(ev);
                if (q != hipSuccess) break;
                memcpy(slot, host + first, m * sizeof(double));
            }
            {
                std::lock_guard<std::mutex> one(enqueue);
                q = kernel(slot, first, m, s);
                if (q == hipSuccess) q = hipEventRecord(ev, s);
            }
            pending = q == hipSuccess;
            if (to_host && pending) {
                q = hipEventSynchronize(ev);
                if (q == hipSuccess) memcpy(host + first, slot, m * sizeof(double));
            }
        }
        if (ev) (void)hipEventDestroy(ev);
        if (q != hipSuccess) failed = q;
    };
    std::vector<std::thread> threads;
    threads.reserve(workers);
    for (int w = 1; w < workers; ++w) {
        try {
            threads.emplace_back(work, true);
        } catch (const std::system_error &) {
            break;  // fewer threads: the missing workers' chunks are done below
        }
    }
    const int missing = workers - 1 - (int)threads.size();
    work(false);
    for (std::thread &t : threads) t.join();
    for (int w = 0; w < missing; ++w) work(false);
    if (failed) {
        (void)hipStreamSynchronize(s);  // nothing uses the slots any more
        return (hipError_t)failed.load();
    }
    return hipStreamSynchronize(s);
}

}  // namespace

void stage_retain()
{
    std::lock_guard<std::mutex> lock(g_count);
    ++g_refs;
}

void stage_release()
{
    std::lock_guard<std::mutex> lock(g_count);
    if (--g_refs > 0) return;
    std::lock_guard<std::mutex> use(g_use);
    if (g_slots) (void)hipHostFree(g_slots);
    g_slots = nullptr;
}

hipError_t stage_out(int device, hipStream_t s, double *out, size_t n, const StageKernel &kernel)
{
    return transfer(device, s, out, n, true, kernel);
}

hipError_t stage_in(int device, hipStream_t s, const double *in, size_t n,
                    const StageKernel &kernel)
{
    return transfer(device, s, const_cast<double *>(in), n, false, kernel);
}

}  // namespace flbdev
