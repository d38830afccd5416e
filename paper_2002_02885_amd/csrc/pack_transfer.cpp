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
#include <cstring>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace packk {
namespace {

constexpr size_t CHUNK_BYTES = (size_t)1 << 19;
constexpr int MAX_THREADS = 8, SLOTS = 2 * MAX_THREADS;    // two chunks in flight per thread

struct Ring {
    int device = -1;
    char* host = nullptr;
    char* dev = nullptr;
    hipEvent_t done[SLOTS] = {};
};

// One idle ring (8 MB) is kept for the next transfer, whichever pack asks for it; every further one is released
// when its transfer ends.  (Pinning 8 MB and touching it for the first time takes 3 ms, as long as a transfer of 150 MB.)
std::mutex g_mu;
Ring* g_idle = nullptr;

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

}  // namespace

// Moves n floats chunk by chunk.  `enqueue(slot, first, count)` launches the kernel that fills (to_host) or drains
// (!to_host) the pinned slot; `prepare()` is called once before, when everything that can be short of memory is there.
// Every kernel has ended when this returns, also on an error.
template <typename Prepare, typename Enqueue>
static hipError_t move_blob(int device, hipStream_t st, float* host, size_t n, bool to_host, Prepare&& prepare, Enqueue&& enqueue) {
    if (n == 0) return hipStreamSynchronize(st);
    int current = -1;
    hipError_t e = hipGetDevice(&current);
    if (e != hipSuccess) return e;
    Ring* ring = nullptr;
    e = acquire(device, &ring);
    if (e != hipSuccess) return e;
    const size_t per = CHUNK_BYTES / sizeof(float);
    const size_t chunks = (n + per - 1) / per;
    const int threads = (int)std::min<size_t>(MAX_THREADS, std::max<size_t>(1, chunks));
    std::atomic<int> failed{(int)prepare()};
    auto work = [&](int t, bool helper) {
        hipError_t we = failed.load() ? (hipError_t)failed.load() : helper || current != device ? hipSetDevice(device) : hipSuccess;
        auto count = [&](size_t c) { return std::min(per, n - c * per); };
        auto slot_of = [&](size_t i) { return 2 * t + (int)(i & 1); };
        auto slot_dev = [&](int s) { return (float*)(ring->dev + (size_t)s * CHUNK_BYTES); };
        auto slot_host = [&](int s) { return (float*)(ring->host + (size_t)s * CHUNK_BYTES); };
        auto start = [&](size_t i) {
            const size_t c = t + i * threads;
            const int s = slot_of(i);
            hipError_t q = enqueue(slot_dev(s), c * per, (int)count(c));
            if (q == hipSuccess) q = hipEventRecord(ring->done[s], st);
            return q;
        };
        const size_t mine = chunks > (size_t)t ? (chunks - t + threads - 1) / threads : 0;
        size_t started = 0, ended = 0;
        if (to_host) {
            for (; we == hipSuccess && started < std::min<size_t>(2, mine); ++started) we = start(started);
            for (; we == hipSuccess && ended < mine; ++ended) {
                const size_t c = t + ended * threads;
                const int s = slot_of(ended);
                we = hipEventSynchronize(ring->done[s]);
                if (we != hipSuccess) break;
                std::memcpy(host + c * per, slot_host(s), count(c) * sizeof(float));
                if (started < mine) we = start(started++);
            }
        } else {
            for (; we == hipSuccess && started < mine; ++started) {
                const size_t c = t + started * threads;
                const int s = slot_of(started);
                if (started >= 2) we = hipEventSynchronize(ring->done[s]);
                if (we != hipSuccess) break;
                std::memcpy(slot_host(s), host + c * per, count(c) * sizeof(float));
                we = start(started);
            }
        }
        if (we != hipSuccess) {
            int none = 0;
            failed.compare_exchange_strong(none, (int)we);
        }
    };
    std::vector<std::thread> pool;
    int handed = 1;
    try {
        for (; handed < threads; ++handed) pool.emplace_back(work, handed, true);
    } catch (const std::system_error&) {
        // no more threads to be had: this one does their share
    }
    work(0, false);
    for (int t = handed; t < threads; ++t) work(t, false);
    for (std::thread& t : pool) t.join();
    e = hipStreamSynchronize(st);
    if (current != device) (void)hipSetDevice(current);
    give_back(ring);
    return failed.load() ? (hipError_t)failed.load() : e;
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
