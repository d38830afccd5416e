// Checkpoints between pageable host memory and the parameter arenas, through a small ring of pinned memory.
//
// A copy of pageable memory by the runtime costs a pass over the link, a pass through its own staging and, with the
// blob layout made on the host, one more pass and a fresh buffer: 4.6 ms for a 16 MB member.  Here the layout is made
// by the kernel that crosses the link (pack_state.hip) and up to eight threads copy between the ring and the caller's
// buffer while the next chunks are on the link, so that the page faults of a fresh destination (4 KB at a time:
// 4.8 GB/s on one thread, 12.6 GB/s on four, 20 GB/s on eight) overlap with each other and with the transfer.
// Measured, checkpoints of all members: 8 x 16.8 MB 37.5 -> 6.8 ms, 32 members of 0.8 to 16 MB 46.3 -> 15.6 ms,
// 4 convolutional members of 19 MB 26.9 -> 3.9 ms.  (Asking for the destination's pages in one call before the copy,
// MADV_POPULATE_WRITE, changed nothing: what remains is the zeroing of fresh pages.)
#include "pack_internal.h"

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <utility>

namespace packk {
namespace {

constexpr size_t CHUNK_BYTES = (size_t)1 << 19;
constexpr int MAX_THREADS = 8, SLOTS = 2 * MAX_THREADS;    // helpers; per helper a chunk being copied and one on the link

struct Ring {
    int device = -1;
    char* host = nullptr;
    char* dev = nullptr;
    hipEvent_t done[SLOTS] = {};
};

// One idle ring (8 MB) is kept for the next transfer, whichever pack asks for it, while there is a pack; every further one
// is released when its transfer ends, and the last one with the last pack.  (A transfer that makes and releases its own
// spends some 60 us on it; the first of a process, whose pages the system has yet to pin and clear, 3 ms.)
std::mutex g_mu;
Ring* g_idle = nullptr;
int g_packs = 0;

void destroy(Ring* r) {
    if (!r) return;
    for (hipEvent_t e : r->done)
        if (e) (void)hipEventDestroy(e);
    if (r->host) (void)hipHostFree(r->host);
    delete r;
}

hipError_t acquire(int device, Ring** out) {
    Ring* stale = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (g_idle) {
            if (g_idle->device == device) {
                *out = g_idle;
                g_idle = nullptr;
                return hipSuccess;
            }
            stale = g_idle;
            g_idle = nullptr;
        }
    }
    destroy(stale);
    Ring* r = new (std::nothrow) Ring();
    if (!r) return hipErrorOutOfMemory;
    r->device = device;
    hipError_t e = hipHostMalloc((void**)&r->host, SLOTS * CHUNK_BYTES, hipHostMallocMapped | hipHostMallocPortable);
    if (e == hipSuccess) e = hipHostGetDevicePointer((void**)&r->dev, r->host, 0);
    for (int i = 0; i < SLOTS && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&r->done[i], hipEventDisableTiming);
    if (e != hipSuccess) {
        (void)hipGetLastError();   // (a later launch is not to report it)
        destroy(r);
        return e;
    }
    *out = r;
    return hipSuccess;
}

void give_back(Ring* r) {
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (!g_idle) {
            g_idle = r;
            return;
        }
    }
    destroy(r);
}

// One transfer, chunk by chunk through the ring's slots.  The calling thread launches every kernel and records every
// event, in chunk order: a stream handle may name another stream in another thread (hipStreamPerThread), and work that
// helpers launched on it would run beside the pack's steps.  Helper threads wait for events and copy between the ring and
// the caller's buffer.  (Against threads that launch and copy their own chunks: 6.3 MB out 0.30 -> 0.28 ms and in
// 0.29 -> 0.26, 16.8 MB 0.62 -> 0.59 and 0.69 -> 0.63.)
struct Transfer {
    Ring* ring;
    char* host;
    size_t bytes, chunks;
    bool to_host;
    std::mutex mu;
    std::condition_variable work;         // a chunk to copy, or the end
    size_t launched = 0;                  // chunks whose kernel is on the stream, its event behind it
    size_t next = 0;                      // next chunk to copy
    std::atomic<size_t> copied[SLOTS];    // 1 + the last chunk copied out of (into) the slot
    std::atomic<hipError_t> failed;
    std::thread helpers[MAX_THREADS];
    int wanted;
    std::atomic<int> started{0};

    Transfer(Ring* r, float* h, size_t n, bool out, hipError_t e)
        : ring(r), host((char*)h), bytes(n * sizeof(float)), chunks((bytes + CHUNK_BYTES - 1) / CHUNK_BYTES), to_host(out), failed(e),
          wanted((int)std::min<size_t>(MAX_THREADS, chunks - 1)) {
        for (auto& c : copied) c = 0;
    }
    // a chunk can be copied out once its kernel has been launched, and in once the kernel that reads the slot's previous
    // chunk has been
    bool can_copy() const { return next < chunks && next < (to_host ? launched : launched + SLOTS); }
    bool over() const { return failed != hipSuccess || next == chunks; }
    // chunk c's kernel may be launched: the slot's previous chunk is out, or this one is in
    bool can_launch(size_t c) const {
        const size_t last = copied[c % SLOTS].load(std::memory_order_acquire);
        return to_host ? c < SLOTS || last == c - SLOTS + 1 : last == c + 1;
    }

    void fail(hipError_t e) {   // under the lock
        if (failed.load() == hipSuccess) failed.store(e);
        work.notify_all();
    }
    void copy_next(std::unique_lock<std::mutex>& lock) {
        const size_t c = next++, s = c % SLOTS, at = c * CHUNK_BYTES, len = std::min(CHUNK_BYTES, bytes - at);
        if (next == chunks) work.notify_all();
        lock.unlock();
        char* const slot = ring->host + s * CHUNK_BYTES;
        const hipError_t e = to_host || c >= SLOTS ? hipEventSynchronize(ring->done[s]) : hipSuccess;
        if (e == hipSuccess) {
            std::memcpy(to_host ? host + at : slot, to_host ? slot : host + at, len);
            copied[s].store(c + 1, std::memory_order_release);
        }
        lock.lock();
        if (e != hipSuccess) fail(e);
    }
    void help() {
        std::unique_lock<std::mutex> lock(mu);
        while (!over()) {
            if (can_copy()) copy_next(lock);
            else work.wait(lock);
        }
    }
    // Starts helper i, which first starts two more: a thread takes longer to start than a kernel, and the launching thread
    // is not to spend its time on eight.
    void start_helper(int i) {
        if (i >= wanted) return;
        try {
            helpers[i] = std::thread([this, i] {
                start_helper(2 * i + 2);
                start_helper(2 * i + 3);
                help();
            });
            ++started;
        } catch (...) {
            // no more threads to be had: the others, or the launching thread, do their share
        }
    }
    void join() {
        for (std::thread& h : helpers)   // (a helper is started by one with a smaller number)
            if (h.joinable()) h.join();
    }
    // the launching thread, until chunk c may be launched; it copies meanwhile only where there are fewer helpers than
    // would keep the link busy, and does not sleep: being woken takes as long as a chunk
    void wait_for(size_t c) {
        if (started < MAX_THREADS) {
            std::unique_lock<std::mutex> lock(mu);
            while (!over() && !can_launch(c) && can_copy()) copy_next(lock);
        }
        while (failed == hipSuccess && !can_launch(c)) std::this_thread::yield();
    }
};

}  // namespace

void transfer_open() {
    std::lock_guard<std::mutex> lock(g_mu);
    ++g_packs;
}
void transfer_close() {
    Ring* last = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (--g_packs == 0) std::swap(last, g_idle);
    }
    destroy(last);
}

// Moves n floats.  `enqueue(slot, first, count)` launches the kernel that fills (to_host) or drains (!to_host) the pinned
// slot; `prepare()` is called once before, when everything that can be short of memory is there.  Every kernel has ended
// when this returns, also on an error.
template <typename Prepare, typename Enqueue>
static hipError_t move_blob(int device, hipStream_t st, float* host, size_t n, bool to_host, Prepare&& prepare, Enqueue&& enqueue) {
    if (n == 0) return hipStreamSynchronize(st);
    int current = -1;
    hipError_t e = hipGetDevice(&current);
    if (e != hipSuccess) return e;
    Ring* ring = nullptr;
    e = acquire(device, &ring);
    if (e != hipSuccess) return e;
    if (current != device) e = hipSetDevice(device);
    if (e == hipSuccess) e = prepare();
    Transfer t(ring, host, n, to_host, e);
    const size_t per = CHUNK_BYTES / sizeof(float);
    for (size_t c = 0; c < t.chunks; ++c) {
        // (into the arena there is something to copy at once, out of it when the first kernels have been launched)
        if (c == (to_host ? std::min<size_t>(2, t.chunks - 1) : 0)) {
            t.start_helper(0);
            t.start_helper(1);
        }
        t.wait_for(c);
        if (t.failed != hipSuccess) break;
        const size_t s = c % SLOTS;
        e = enqueue((float*)(ring->dev + s * CHUNK_BYTES), c * per, (int)std::min(per, n - c * per));
        if (e == hipSuccess && (to_host || c + SLOTS < t.chunks)) e = hipEventRecord(ring->done[s], st);   // (where somebody waits for it)
        std::unique_lock<std::mutex> lock(t.mu);
        if (e != hipSuccess) {
            t.fail(e);
            break;
        }
        t.launched = c + 1;
        lock.unlock();
        t.work.notify_one();
    }
    t.help();
    t.join();
    e = hipStreamSynchronize(st);
    if (current != device) (void)hipSetDevice(current);
    if (e == hipSuccess) give_back(ring);   // (a ring that a kernel may still be using is neither used again nor released)
    return t.failed != hipSuccess ? t.failed.load() : e;
}

hipError_t export_blob(int device, hipStream_t st, const float* arena, const BlobSeg* segs, int n_segs, size_t n, float* host) {
    return move_blob(device, st, host, n, true, [] { return hipSuccess; }, [&](float* slot, size_t first, int count) {
        return launch_export_blob(arena, segs, n_segs, (long long)first, count, slot, st);
    });
}

hipError_t import_blob(int device, hipStream_t st, float* arena, void* shadow, const BlobSeg* segs, int n_segs, size_t n, const float* host,
                       size_t clear, float value) {
    auto prepare = [&] {
        hipError_t e = clear ? launch_fill_value(arena, (long long)clear, value, st) : hipSuccess;
        if (e == hipSuccess && clear && shadow) e = launch_fill_zero(shadow, (long long)clear * 2, st);
        return e;
    };
    return move_blob(device, st, const_cast<float*>(host), n, false, prepare, [&](float* slot, size_t first, int count) {
        return launch_import_blob(arena, shadow, segs, n_segs, (long long)first, count, slot, st);
    });
}

}  // namespace packk
