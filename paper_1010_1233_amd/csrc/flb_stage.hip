// flb_stage.hip -- see flb_stage.h.
#include "flb_stage.h"

#include <string.h>

#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <exception>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

namespace flbdev {

namespace {

// One transfer: the threads that have joined it take its chunks in turn.
struct Job {
    int device;
    hipStream_t stream;
    double *host;
    size_t n, chunks;
    bool to_host;
    const StageKernel *kernel;
    double *const *pairs;  // two slots of each seat
    int seats = 0;         // threads that may still join (pairs left)
    int active = 0;        // threads at work (guarded by the pool's mutex)
    int joined = 1;        // pairs handed out, the caller's first
    std::mutex m;    // guards next and failed, and orders the launches
    size_t next = 0;
    hipError_t failed = hipSuccess;
};

// Takes the next chunk and enqueues its kernel into `slot` (from the
// caller's memory: after copying the chunk there).  chunk: its index, or
// job.chunks when none is left.
hipError_t take(Job &j, double *slot, hipEvent_t ev, size_t &chunk)
{
    size_t first = 0, m = 0;
    auto range = [&](size_t c) {
        first = c * kStageSlotDoubles;
        m = std::min(kStageSlotDoubles, j.n - first);
    };
    {
        std::lock_guard<std::mutex> lock(j.m);
        chunk = j.failed != hipSuccess ? j.chunks : std::min(j.next, j.chunks);
        if (chunk == j.chunks) return hipSuccess;
        ++j.next;
        range(chunk);
        if (j.to_host) {
            hipError_t e = (*j.kernel)(slot, first, m, StageDone{nullptr, 0}, j.stream);
            if (e == hipSuccess) e = hipEventRecord(ev, j.stream);
            return e;
        }
    }
    memcpy(slot, j.host + first, m * sizeof(double));
    std::lock_guard<std::mutex> lock(j.m);
    hipError_t e = (*j.kernel)(slot, first, m, StageDone{nullptr, 0}, j.stream);
    if (e == hipSuccess) e = hipEventRecord(ev, j.stream);
    return e;
}

// A thread's share, through its two slots: one chunk's kernel runs while
// the other's is copied.
void work(Job &j, int seat)
{
    double *slot[2];
    hipEvent_t ev[2] = {nullptr, nullptr};
    size_t chunk[2] = {j.chunks, j.chunks};  // in flight in each slot
    hipError_t e = hipSuccess;
    for (int q = 0; q < 2 && e == hipSuccess; ++q) {
        slot[q] = j.pairs[seat] + q * kStageSlotDoubles;
        e = hipEventCreateWithFlags(&ev[q], hipEventDisableTiming);
        if (e == hipSuccess) e = take(j, slot[q], ev[q], chunk[q]);
    }
    for (int q = 0; e == hipSuccess && chunk[q] != j.chunks; q ^= 1) {
        e = hipEventSynchronize(ev[q]);
        if (e != hipSuccess) break;
        if (j.to_host) {
            const size_t first = chunk[q] * kStageSlotDoubles;
            memcpy(j.host + first, slot[q],
                   std::min(kStageSlotDoubles, j.n - first) * sizeof(double));
        }
        e = take(j, slot[q], ev[q], chunk[q]);
    }
    for (hipEvent_t x : ev)
        if (x) (void)hipEventDestroy(x);
    if (e != hipSuccess) {
        std::lock_guard<std::mutex> lock(j.m);
        j.failed = e;
    }
}

// Pinned memory of a transfer, made as transfers need it and kept from one to
// the next (freeing some to make more would wait for the device): a small
// place with flags, and pairs of slots.
struct SlotSet {
    double *small = nullptr;  // kStageSmallDoubles
    uint32_t *flags = nullptr;
    uint32_t seq = 0;  // of the last transfer with flags; 0 is never one's
    double *pairs[kStageWorkers] = {};
    int npairs = 0;
    bool busy = false;  // (extra sets; guarded by the pool's mutex m)

    // portable: the transfers of every device go through the same slots;
    // coherent: the flags are read while the kernel runs
    static hipError_t pinned(void **mem, size_t bytes)
    {
        return hipHostMalloc(mem, bytes, hipHostMallocPortable | hipHostMallocCoherent);
    }
    hipError_t make_small()
    {
        if (small) return hipSuccess;
        void *mem = nullptr;
        const size_t bytes = kStageSmallDoubles * sizeof(double);
        if (hipError_t e = pinned(&mem, bytes + kStageFlags * sizeof(uint32_t)); e != hipSuccess)
            return e;
        small = static_cast<double *>(mem);
        flags = reinterpret_cast<uint32_t *>(static_cast<char *>(mem) + bytes);
        memset(flags, 0, kStageFlags * sizeof(uint32_t));
        return hipSuccess;
    }
    // at least one pair, and up to `want` of them
    hipError_t make_pairs(int want)
    {
        while (npairs < want) {
            void *mem = nullptr;
            if (hipError_t e = pinned(&mem, 2 * kStageSlotDoubles * sizeof(double)); e != hipSuccess) {
                (void)hipGetLastError();
                return npairs ? hipSuccess : e;
            }
            pairs[npairs++] = static_cast<double *>(mem);
        }
        return hipSuccess;
    }
    void release()
    {
        if (small) (void)hipHostFree(small);
        for (int i = 0; i < npairs; ++i) (void)hipHostFree(pairs[i]);
    }
};

// The helper threads and the slots of the handles that are open together.
struct Pool {
    std::mutex use;  // held by the transfer that has `set` and the helpers
    SlotSet set;
    // for transfers that find it taken: its holder may be waiting for steps
    // still to run on its stream (two slots each, no helpers)
    SlotSet extra[kStageExtra];
    std::mutex m;  // guards the rest
    std::condition_variable wake, done;
    std::vector<std::thread> threads;
    Job *job = nullptr;
    bool stop = false;

    // No transfer is running: ends the helpers and gives the slots back.
    void close()
    {
        {
            std::lock_guard<std::mutex> lock(m);
            stop = true;
        }
        wake.notify_all();
        for (std::thread &t : threads) t.join();
        set.release();
        for (SlotSet &x : extra) x.release();
    }

    void helper()
    {
        std::unique_lock<std::mutex> lock(m);
        for (;;) {
            wake.wait(lock, [&] { return stop || (job && job->seats > 0); });
            if (stop) return;
            Job &j = *job;
            const int seat = j.joined++;
            --j.seats;
            ++j.active;
            lock.unlock();
            const hipError_t e = hipSetDevice(j.device);
            if (e == hipSuccess) work(j, seat);  // (else: the others do it all)
            lock.lock();
            if (--j.active == 0) done.notify_all();
        }
    }
};

// The pool of the open handles.  The last of them takes it along and closes it
// on its own: a handle opened meanwhile gets another, so that no slot is given
// back under a transfer.  (Never destroyed: helpers of handles still open at
// the process's end sleep through it.)
struct Open {
    std::mutex m;  // guards the rest
    int handles = 0;
    Pool *pool = nullptr;
};
Open &open_handles()
{
    static Open *o = new Open();
    return *o;
}
// Called for an open handle, whose pool stays for as long as it is open.
Pool &pool()
{
    Open &o = open_handles();
    std::lock_guard<std::mutex> lock(o.m);
    return *o.pool;
}

// The slots of one transfer: the main set, an extra one, or whichever the
// main set's holder gives back.
struct SlotUse {
    Pool &p;
    std::unique_lock<std::mutex> lock;
    bool mine;  // the main set
    SlotSet &set;

    explicit SlotUse(Pool &pool)
        : p(pool), lock(p.use, std::try_to_lock), mine(lock.owns_lock()), set(pick())
    {
    }
    ~SlotUse()
    {
        if (mine) return;
        std::lock_guard<std::mutex> l(p.m);
        set.busy = false;
    }
    SlotSet &pick()
    {
        if (!mine) {
            {
                std::lock_guard<std::mutex> l(p.m);
                for (SlotSet &x : p.extra)
                    if (!x.busy) {
                        x.busy = true;
                        return x;
                    }
            }
            lock.lock();
            mine = true;
        }
        return p.set;
    }
};

// Waits for the flags of all blocks, at most 100 us (the stream may have
// more work before the kernel): false if some are missing.
bool all_done(const StageDone &done, size_t blocks)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (size_t b = 0; b < blocks;) {
        for (int spin = 0; spin < 64 && b < blocks; ++spin)
            while (b < blocks && __atomic_load_n(&done.flag[b], __ATOMIC_ACQUIRE) == done.seq) ++b;
        if (b < blocks &&
            std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(100))
            return false;
    }
    return true;
}

// The handle's device made the thread's current one, and the caller's again: an
// event cannot be recorded on another device's stream.
struct DeviceUse {
    int was = -1;
    hipError_t error;
    explicit DeviceUse(int device)
    {
        int cur = device;
        error = hipGetDevice(&cur);
        if (error != hipSuccess || cur == device) return;
        error = hipSetDevice(device);
        if (error == hipSuccess) was = cur;
    }
    ~DeviceUse()
    {
        if (was >= 0) (void)hipSetDevice(was);
    }
};

hipError_t transfer(int device, hipStream_t s, double *host, size_t n, bool to_host,
                    const StageKernel &kernel)
{
    if (!n) return hipStreamSynchronize(s);
    DeviceUse current(device);
    if (current.error != hipSuccess) return current.error;
    Pool &p = pool();
    SlotUse use(p);
    SlotSet &set = use.set;
    Job j;
    j.device = device;
    j.stream = s;
    j.host = host;
    j.n = n;
    j.chunks = (n + kStageSlotDoubles - 1) / kStageSlotDoubles;
    j.to_host = to_host;
    j.kernel = &kernel;
    j.pairs = set.pairs;
    if (j.chunks == 1) {
        const bool small = n <= kStageSmallDoubles;
        hipError_t e = small ? set.make_small() : set.make_pairs(1);
        if (e != hipSuccess) return e;
        double *slot = small ? set.small : set.pairs[0];
        const size_t blocks = (n + kStageBlock - 1) / kStageBlock;
        const bool flags = to_host && small && blocks <= (size_t)kStageFlags;
        if (!to_host) memcpy(slot, host, n * sizeof(double));
        StageDone done{nullptr, 0};
        if (flags) {
            done.flag = set.flags;
            if (++set.seq == 0) set.seq = 1;
            done.seq = set.seq;
        }
        if ((e = kernel(slot, 0, n, done, s)) != hipSuccess) return e;
        if (!flags || !all_done(done, blocks))
            if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (to_host) memcpy(host, slot, n * sizeof(double));
        return hipSuccess;
    }
    // a helper for every two chunks past the caller's own two
    int helpers = use.mine ? (int)std::min<size_t>((j.chunks - 1) / 2, kStageWorkers - 1) : 0;
    if (hipError_t e = set.make_pairs(1 + helpers); e != hipSuccess) return e;
    helpers = std::min(helpers, set.npairs - 1);
    if (helpers) {
        std::lock_guard<std::mutex> lock(p.m);
        try {
            while ((int)p.threads.size() < helpers)
                p.threads.emplace_back([&p] { p.helper(); });
        } catch (const std::exception &) {
            // fewer helpers, or none: the caller's thread does the rest
        }
        j.seats = helpers;
        p.job = &j;
    }
    for (int i = 0; i < helpers; ++i) p.wake.notify_one();
    work(j, 0);
    if (helpers) {
        // no more joining; wait for those at work
        std::unique_lock<std::mutex> lock(p.m);
        p.job = nullptr;
        p.done.wait(lock, [&] { return j.active == 0; });
    }
    // every kernel that uses a slot has ended (a failed transfer may have
    // left some behind)
    const hipError_t e = hipStreamSynchronize(s);
    return j.failed != hipSuccess ? j.failed : e;
}

}  // namespace

void stage_retain()
{
    Open &o = open_handles();
    std::lock_guard<std::mutex> lock(o.m);
    if (o.handles == 0) o.pool = new Pool();
    ++o.handles;
}

void stage_release()
{
    Open &o = open_handles();
    Pool *last = nullptr;
    {
        std::lock_guard<std::mutex> lock(o.m);
        if (--o.handles > 0) return;
        std::swap(last, o.pool);
    }
    last->close();
    delete last;
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
