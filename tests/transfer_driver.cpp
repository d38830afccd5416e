// Driver of the library's host code on a made-up GPU: tests/test_transfer_host.py compiles it together with
// csrc/pack_api.cpp and csrc/pack_transfer.cpp (host code only) and runs one scenario per process.  Every HIP call the
// two files make is defined here: a stream is a queue with a thread of its own that runs what was enqueued late and in
// order, hipStreamPerThread names another stream in every host thread, device memory is host memory.  The few kernels
// that matter (state in and out, seeding, clearing, the fused update) are plain loops, the others do nothing.
#include "../include/pack.h"
#include "pack_internal.h"

#include <dlfcn.h>
#include <pthread.h>
#include <unistd.h>

#include <atomic>
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <random>
#include <string>
#include <thread>
#include <vector>

using namespace packk;

static std::atomic<int> g_fail_at{-1};          // the n-th fallible call from now fails (negative: none)
static std::atomic<bool> g_no_pinned{false};    // pinned allocations fail
static std::atomic<int> g_threads_left{-1};     // threads that may still be started (negative: any number)
static std::atomic<int> g_pinned{0}, g_events{0};
static std::atomic<long long> g_launches{0};
static std::mutex g_mu;
static std::vector<std::string> g_errors;
static std::atomic<bool> g_capturing{false};    // the streams are being captured: waiting for one is an error
static std::thread::id g_main;
static std::map<const char*, size_t> g_host;    // live pinned allocations

static void error(const std::string& s) {
    std::lock_guard<std::mutex> l(g_mu);
    if (g_errors.size() < 20) g_errors.push_back(s);
}
static thread_local hipError_t g_last = hipSuccess;   // what hipGetLastError reports, as a launch does after it
static bool fails() { return g_fail_at.load() >= 0 && g_fail_at.fetch_sub(1) == 0; }

extern "C" int pthread_create(pthread_t* t, const pthread_attr_t* a, void* (*f)(void*), void* arg) {
    typedef int (*fn)(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*);
    static fn real = (fn)dlsym(RTLD_NEXT, "pthread_create");
    if (g_threads_left.load() >= 0 && g_threads_left.fetch_sub(1) <= 0) { g_threads_left = 0; return EAGAIN; }
    return real(t, a, f, arg);
}

static thread_local long long t_new_left = -1;   // allocations of this thread that still succeed (negative: all)
void* operator new(size_t n) {
    if (t_new_left >= 0 && t_new_left-- == 0) throw std::bad_alloc();
    if (void* p = malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

struct Queue {
    std::mutex mu;
    std::condition_variable cv;
    std::deque<std::function<void()>> q;
    bool busy = false;
    void run() {
        std::mt19937 rng(7);
        for (;;) {
            std::function<void()> f;
            {
                std::unique_lock<std::mutex> l(mu);
                busy = false;
                cv.notify_all();
                cv.wait(l, [&] { return !q.empty(); });
                f = std::move(q.front());
                q.pop_front();
                busy = true;
            }
            usleep(rng() % 300);
            f();
        }
    }
    void push(std::function<void()> f) {
        std::lock_guard<std::mutex> l(mu);
        q.push_back(std::move(f));
        cv.notify_all();
    }
    void drain() {
        std::unique_lock<std::mutex> l(mu);
        cv.wait(l, [&] { return q.empty() && !busy; });
    }
};
static std::mutex g_streams_mu;
static std::map<std::pair<hipStream_t, std::thread::id>, Queue*> g_streams;
static Queue* queue_of(hipStream_t s) {
    const auto key = std::make_pair(s, s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id());
    std::lock_guard<std::mutex> l(g_streams_mu);
    Queue*& q = g_streams[key];
    if (!q) {
        q = new Queue();
        const int left = g_threads_left.exchange(-1);
        std::thread([q] { q->run(); }).detach();
        g_threads_left = left;
    }
    return q;
}
static bool idle() {
    std::lock_guard<std::mutex> l(g_streams_mu);
    for (auto& q : g_streams) {
        std::lock_guard<std::mutex> lq(q.second->mu);
        if (!q.second->q.empty() || q.second->busy) return false;
    }
    return true;
}
static hipError_t enqueue(hipStream_t st, std::function<void()> f) {
    if (std::this_thread::get_id() != g_main) error("a kernel was launched from another thread than the caller's");
    ++g_launches;
    if (fails()) return hipErrorLaunchFailure;
    if (g_last != hipSuccess) return hipGetLastError();
    queue_of(st)->push(std::move(f));
    return hipSuccess;
}
static void check_pinned(const void* p, size_t n) {
    std::lock_guard<std::mutex> l(g_mu);
    auto it = g_host.upper_bound((const char*)p);
    if (it == g_host.begin() || (--it, (const char*)p + n > it->first + it->second)) g_errors.push_back("a kernel used pinned memory that is no longer there");
}

struct Event {
    std::mutex mu;
    std::condition_variable cv;
    long long recorded = 0, reached = 0;
};

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); std::memset(*p, 0xCD, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) { queue_of(st)->push([=] { std::memcpy(d, s, n); }); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) { queue_of(st)->push([=] { std::memset(d, v, n); }); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t st) {
    if (g_capturing) return hipErrorStreamCaptureUnsupported;
    queue_of(st)->drain();
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = g_last; g_last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "made-up error"; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (g_no_pinned || fails()) return g_last = hipErrorOutOfMemory;
    *p = malloc(n);
    std::lock_guard<std::mutex> l(g_mu);
    g_host[(const char*)*p] = n;
    ++g_pinned;
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipHostFree(void* p) {
    std::lock_guard<std::mutex> l(g_mu);
    g_host.erase((const char*)p);
    --g_pinned;
    std::memset(p, 0xEE, 64);   // (not given back to the system: a late reader is to be noticed, not to crash)
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event(); ++g_events; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { --g_events; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t ev, hipStream_t st) {
    if (fails()) return hipErrorUnknown;
    Event* e = (Event*)ev;
    long long n;
    {
        std::lock_guard<std::mutex> l(e->mu);
        n = ++e->recorded;
    }
    queue_of(st)->push([=] { std::lock_guard<std::mutex> l(e->mu); e->reached = n; e->cv.notify_all(); });
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t ev) {
    if (fails()) return hipErrorUnknown;
    Event* e = (Event*)ev;
    std::unique_lock<std::mutex> l(e->mu);
    const long long n = e->recorded;
    e->cv.wait(l, [&] { return e->reached >= n; });
    return hipSuccess;
}
}

namespace packk {
static long long place(const BlobSeg* segs, int n_segs, long long e) {
    int k = n_segs - 1;
    while (segs[k].blob_off > e) --k;
    const BlobSeg& s = segs[k];
    const long long i = e - s.blob_off, r = i / s.inner, j = i % s.inner;
    const long long a = s.conv ? j % 9 : j / s.cin, b = s.conv ? j / 9 : j % s.cin;
    return s.arena_off + r * s.ldw + a * s.cpad + b;
}
hipError_t launch_export_blob(const float* arena, const BlobSeg* segs, int n_segs, long long e0, int n, float* out, hipStream_t st) {
    return enqueue(st, [=] { check_pinned(out, n * 4); for (int i = 0; i < n; ++i) out[i] = arena[place(segs, n_segs, e0 + i)]; });
}
hipError_t launch_import_blob(float* arena, void*, const BlobSeg* segs, int n_segs, long long e0, int n, const float* in, hipStream_t st) {
    return enqueue(st, [=] { check_pinned(in, n * 4); for (int i = 0; i < n; ++i) arena[place(segs, n_segs, e0 + i)] = in[i]; });
}
hipError_t launch_seed_blob(float* arena, void*, const BlobSeg* segs, int n_segs, long long n, unsigned long long, unsigned long long, hipStream_t st) {
    return enqueue(st, [=] { for (long long i = 0; i < n; ++i) arena[place(segs, n_segs, i)] = 0.5f; });
}
hipError_t launch_fill_value(float* d, long long n, float v, hipStream_t st) { return enqueue(st, [=] { for (long long i = 0; i < n; ++i) d[i] = v; }); }
hipError_t launch_fill_zero(void* d, long long n, hipStream_t st) { return enqueue(st, [=] { std::memset(d, 0, n); }); }
// what the matrix products and reductions of a step were handed over with
struct GemmCall { int mode, tile_cfg; bool opt; };
static std::vector<GemmCall> g_gemms;
static int g_reduces = 0, g_reduces_opt = 0, g_updates = 0;
// the fused update adds 1 to every weight it owns, some milliseconds after it was enqueued
hipError_t launch_gemm(int mode, bool, int tile_cfg, const GemmProb* probs, const TileRef* tiles, int n, const void*, char*, const LrTable& lr, hipStream_t st) {
    g_gemms.push_back({mode, tile_cfg, lr.opt != nullptr});
    if (mode != LIN_DW) return hipSuccess;
    return enqueue(st, [=] {
        usleep(5000);
        std::map<int, bool> done;
        for (int t = 0; t < n; ++t) {
            if (tiles[t].prob < 0 || done[tiles[t].prob]) continue;
            done[tiles[t].prob] = true;
            const GemmProb& g = probs[tiles[t].prob];
            for (int r = 0; r < g.R; ++r)
                for (int q = 0; q < g.Q && g.upd_w; ++q) g.upd_w[(size_t)r * g.ldc + q] += 1.f;
        }
    });
}
int conv_dw_halo_cfg(bool, const GemmProb&) { return -1; }
int conv_rows_halo_cfg(bool, int, const GemmProb&) { return -1; }
#define NOTHING(name, ...) hipError_t name(__VA_ARGS__) { return hipSuccess; }
hipError_t launch_reduce(const ReduceProb*, const int2*, int, const char*, const LrTable& lr, hipStream_t) {
    ++g_reduces;
    g_reduces_opt += lr.opt != nullptr;
    return hipSuccess;
}
NOTHING(static_scratch, char**)
NOTHING(launch_ce, bool, const CeProb*, const int2*, int, const int32_t*, int*, hipStream_t)
NOTHING(launch_ce_loss, const CeProb*, int, hipStream_t)
NOTHING(launch_head, bool, int, const HeadProb*, const int2*, int, const int32_t*, int*, hipStream_t)
NOTHING(launch_head_loss, const HeadProb*, int, hipStream_t)
NOTHING(launch_gap, bool, bool, const GapProb*, const int2*, int, hipStream_t)
NOTHING(launch_shortcut_bwd, bool, const ShortcutProb*, const int2*, int, hipStream_t)
NOTHING(launch_sgd, float*, const float*, void*, long long, const long long*, int, const LrTable&, hipStream_t)
hipError_t launch_opt(float*, const float*, void*, float*, float*, long long, const long long*, const OptStatic*, int, const OptTable&, hipStream_t) {
    ++g_updates;
    return hipSuccess;
}
NOTHING(launch_im2col, bool, const Im2colProb*, const int2*, int, const void*, hipStream_t)
NOTHING(launch_wtranspose, bool, const TransposeProb*, const int2*, int, hipStream_t)
NOTHING(launch_ceiling_copy, const void*, void*, long long, hipStream_t)
NOTHING(launch_ceiling_mfma, bool, float*, int, int, double*, hipStream_t)
NOTHING(launch_gather_rows, const void*, const int32_t*, const long long*, long long, int, long long, void*, int32_t*, int*, hipStream_t)
std::string conv_dw_halo_walk(bool, bool, const GemmProb&, const TileRef&, long long, long long, bool, long long*, long long*) { return ""; }
std::string conv_rows_halo_walk(bool, bool, bool, const GemmProb&, const TileRef&, long long, long long*, long long*) { return ""; }
std::string gemm_fetch_walk(bool, int, int, int, const GemmProb&, const TileRef&, unsigned long long*, unsigned long long*, unsigned long long*, unsigned long long*, long long*) { return ""; }
}  // namespace packk

// ---- scenarios -------------------------------------------------------------------------------------------
static int g_bad = 0;
#define EXPECT(cond) do { if (!(cond)) { ++g_bad; std::printf("FAIL line %d: %s (last error: %s)\n", __LINE__, #cond, pack_last_error()); } } while (0)

// a member of `features` x `width` + a head: features 3001 and width 997 make 13 MB, more chunks than the ring has slots
struct Member {
    pack_t* p = nullptr;
    int features, width;
    size_t n = 0;
    Member(void* stream, int f, int w) : features(f), width(w) {
        const pack_layer layers[] = {{PACK_LINEAR, w, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 300, 0}};
        const pack_model_spec m{layers, 3, 4};
        const pack_input_spec in{4, 1, 1, f, PACK_F32};
        EXPECT(pack_create(&in, &m, 1, 0, stream, &p) == PACK_OK);
        n = pack_num_params(p, 0);
    }
    ~Member() { pack_destroy(p); }
    bool bias(size_t i) const {
        const size_t w1 = (size_t)features * width, w2 = w1 + width + (size_t)width * 300;
        return (i >= w1 && i < w1 + width) || i >= w2;
    }
};
static std::vector<float> blob(size_t n, int seed) {
    std::mt19937 rng(seed);
    std::vector<float> b(n);
    for (float& v : b) v = (float)(rng() % 100000);
    return b;
}

// weights written, a step, weights read, all on `stream`: each call sees what the one before it did
static void order(void* stream, int features, int width) {
    Member m(stream, features, width);
    alignas(16) static float x[4 * 4096];
    static int32_t y[4];
    const float lr = 0.f;
    for (int round = 0; round < 3; ++round) {
        const std::vector<float> b = blob(m.n, round);
        std::vector<float> given = b, got(m.n);
        EXPECT(pack_write_weights(m.p, 0, given.data(), m.n) == PACK_OK);
        std::fill(given.begin(), given.end(), -1.f);   // the caller's buffer is the caller's again
        EXPECT(pack_step(m.p, x, y, &lr) == PACK_OK);
        EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK);
        size_t wrong = 0;
        for (size_t i = 0; i < m.n; ++i) wrong += got[i] != b[i] + (m.bias(i) ? 0.f : 1.f);
        EXPECT(wrong == 0);
    }
}

// no pinned memory to be had: the calls report it and the member is what it was
static void no_pinned() {
    Member m(nullptr, 301, 97);
    const pack_opt_spec adagrad{PACK_OPT_ADAGRAD, 0.f, 0.5f, 0.f, 0.f, 0.f};
    EXPECT(pack_set_optimizer(m.p, 0, &adagrad) == PACK_OK);
    EXPECT(hipStreamSynchronize(nullptr) == hipSuccess);
    const long long before = g_launches;
    const std::vector<float> b = blob(m.n, 1);
    std::vector<float> got(m.n);
    g_no_pinned = true;
    EXPECT(pack_write_weights(m.p, 0, b.data(), m.n) == PACK_ENOMEM);
    EXPECT(pack_write_opt_state(m.p, 0, 0, b.data(), m.n, 7) == PACK_ENOMEM);
    EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_ENOMEM);
    EXPECT(g_launches == before);
    g_no_pinned = false;
    int64_t steps = -1;
    EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK);
    for (float v : got) if (v != 0.5f) { EXPECT(!"the weights are unchanged"); break; }
    EXPECT(pack_read_opt_state(m.p, 0, 0, got.data(), m.n, &steps) == PACK_OK && steps == 0);
    for (float v : got) if (v != 0.5f) { EXPECT(!"the state is unchanged"); break; }
}

// fewer threads than wanted, down to none
static void few_threads() {
    for (int left : {0, 1, 3}) {
        Member m(nullptr, 3001, 997);
        const std::vector<float> b = blob(m.n, left);
        std::vector<float> got(m.n);
        EXPECT(hipStreamSynchronize(nullptr) == hipSuccess);
        g_threads_left = left;
        EXPECT(pack_write_weights(m.p, 0, b.data(), m.n) == PACK_OK);
        g_threads_left = left;
        EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK);
        g_threads_left = -1;
        EXPECT(got == b);
    }
}

// the n-th launch, event or wait of a transfer fails: it says so and ends, and the next one works
static void failures() {
    Member m(nullptr, 3001, 997);
    const std::vector<float> b = blob(m.n, 3);
    std::vector<float> got(m.n);
    EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK);
    for (int n = 0; n < 47; n += n < 6 ? 1 : 9) {
        g_fail_at = n;
        EXPECT(pack_write_weights(m.p, 0, b.data(), m.n) == PACK_EDEVICE);
        g_fail_at = n;
        EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_EDEVICE);
        g_fail_at = -1;
        EXPECT(pack_write_weights(m.p, 0, b.data(), m.n) == PACK_OK);
        EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK && got == b);
    }
}

// what a call has set up is there when it returns, for a thread whose stream is another one too, and no pack is created on
// a stream that only records
static void ready() {
    Member m((void*)hipStreamPerThread, 301, 97);
    const pack_opt_spec adagrad{PACK_OPT_ADAGRAD, 0.f, 0.25f, 0.f, 0.f, 0.f};
    const pack_layer layers[] = {{PACK_LINEAR, 3, 0}};
    const pack_model_spec one{layers, 1, 4};
    std::vector<float> got(m.n), state(m.n, 0.f), joined;
    EXPECT(idle());
    auto elsewhere = [&](auto f) {
        std::thread([&] { g_main = std::this_thread::get_id(); f(); }).join();
        g_main = std::this_thread::get_id();
    };
    elsewhere([&] { EXPECT(pack_read_weights(m.p, 0, got.data(), m.n) == PACK_OK); });
    EXPECT(got == std::vector<float>(m.n, 0.5f));
    EXPECT(pack_set_optimizer(m.p, 0, &adagrad) == PACK_OK && idle());
    elsewhere([&] { EXPECT(pack_read_opt_state(m.p, 0, 0, state.data(), m.n, nullptr) == PACK_OK); });
    EXPECT(state == std::vector<float>(m.n, 0.25f));
    int32_t k = -1;
    EXPECT(pack_load(m.p, &one, 1, &k) == PACK_OK && k == 1 && idle());
    joined.resize(pack_num_params(m.p, 1));
    elsewhere([&] { EXPECT(pack_read_weights(m.p, 1, joined.data(), joined.size()) == PACK_OK); });
    EXPECT(joined == std::vector<float>(joined.size(), 0.5f));
    const pack_input_spec in{4, 1, 1, 30, PACK_F32};
    pack_t* p = nullptr;
    g_capturing = true;
    EXPECT(pack_create(&in, &one, 1, 0, (void*)0x2000, &p) == PACK_EDEVICE && !p);
    g_capturing = false;
}

// the pinned memory kept between transfers: one ring while there is a pack, nothing after the last one
static void released() {
    for (int round = 0; round < 2; ++round) {
        Member a(nullptr, 301, 97);
        std::vector<float> got(a.n);
        {
            Member b(nullptr, 301, 97);
            EXPECT(pack_read_weights(b.p, 0, got.data(), b.n) == PACK_OK && g_pinned == 1);
            EXPECT(pack_read_weights(a.p, 0, got.data(), a.n) == PACK_OK && g_pinned == 1);
        }
        EXPECT(g_pinned == 1);
        EXPECT(pack_write_weights(a.p, 0, got.data(), a.n) == PACK_OK && g_pinned == 1);
        pack_destroy(a.p);
        a.p = nullptr;
        EXPECT(g_pinned == 0 && g_events == 0);
    }
}

// multiply-adds as the layers define them, whatever the rows are padded to: 5 -> 12 -> 9 channels, 3 x 3 x 9 -> 11 -> 20 features
static void work() {
    const pack_layer layers[] = {{PACK_CONV3X3, 12, 1}, {PACK_RELU, 0, 0}, {PACK_CONV3X3, 9, 2}, {PACK_RELU, 0, 0},
                                 {PACK_LINEAR, 11, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 20, 0}};
    for (int dtype : {PACK_F32, PACK_BF16}) {
        const pack_model_spec m{layers, 7, 4};
        const pack_input_spec in{4, 6, 6, 5, dtype};
        pack_t* p = nullptr;
        EXPECT(pack_create(&in, &m, 1, 0, nullptr, &p) == PACK_OK);
        std::map<std::string, double> got;
        for (int i = 0; i < pack_num_launches(p); ++i) {
            char name[64];
            double f = 0.0;
            EXPECT(pack_launch_name(p, i, name, sizeof name) == PACK_OK && pack_launch_flops(p, i, &f) == PACK_OK);
            got[std::string(name).substr(0, std::string(name).find('+'))] += f;
        }
        const double c1 = 2.0 * 4 * 36 * 45 * 12, c2 = 2.0 * 4 * 9 * 108 * 9, l1 = 2.0 * 4 * 81 * 11, l2 = 2.0 * 4 * 11 * 20;
        EXPECT(got["gemm_conv_fwd"] == c1 + c2);
        EXPECT(got["gemm_conv_dw"] == c1 + c2);
        EXPECT(got["gemm_conv_dx"] == c2);   // (each product of the stride-2 layer once: parity classes)
        EXPECT(got["gemm_lin_fwd"] == l1 + l2);
        EXPECT(got["gemm_lin_dw"] == l1 + l2);
        EXPECT(got["gemm_lin_dx"] == l1 + l2);
        pack_destroy(p);
    }
}

// the update as a launch of its own: products and reductions are the plain ones, whatever their tiles, and nothing in them
// is told of the optimisers; applied where the gradients come from, no launch of its own is left
static void separate_update() {
    const pack_layer layers[] = {{PACK_LINEAR, 1024, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 300, 0}};
    for (int batch : {64, 9000})   // (reductions of a few chunks on large tiles; split ones)
        for (bool fused : {false, true}) {
            const pack_model_spec m{layers, 3, batch};
            const pack_input_spec in{batch, 1, 1, 3072, PACK_BF16};
            const pack_opt_spec momentum{PACK_OPT_MOMENTUM, 0.9f, 0.f, 0.f, 0.f, 0.f};
            setenv("PACK_MIN_TILES", "1", 1);
            if (!fused) setenv("PACK_NO_FUSED_UPDATE", "1", 1);
            pack_t* p = nullptr;
            EXPECT(pack_create(&in, &m, 1, 0, nullptr, &p) == PACK_OK);
            EXPECT(pack_set_optimizer(p, 0, &momentum) == PACK_OK);
            unsetenv("PACK_MIN_TILES");
            unsetenv("PACK_NO_FUSED_UPDATE");
            alignas(16) static float x[1];
            static int32_t y[1];
            const float lr = 0.f;
            g_gemms.clear();
            g_reduces = g_reduces_opt = g_updates = 0;
            EXPECT(pack_step(p, x, y, &lr) == PACK_OK);
            bool large = false;
            for (const GemmCall& c : g_gemms) {
                if (c.mode != LIN_DW) continue;
                large = large || GEMM_TILE_M[c.tile_cfg] == 128;
                if (!fused) EXPECT(!c.opt);
            }
            EXPECT(g_updates == !fused);
            EXPECT(fused ? g_reduces_opt == g_reduces : g_reduces_opt == 0);
            EXPECT(fused || large);
            EXPECT((batch == 9000) == (g_reduces > 0));
            EXPECT(hipStreamSynchronize(nullptr) == hipSuccess);
            pack_destroy(p);
        }
}

// algorithmic bytes of the launch that applies the optimisers: those in force, whatever the order in which they were chosen
static void update_bytes() {
    const pack_layer layers[] = {{PACK_LINEAR, 48, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 40, 0}};
    const double params = 64 * 48 + 48 * 40;   // (weights; biases are not counted)
    for (int dtype : {PACK_F32, PACK_BF16}) {
        const pack_model_spec m{layers, 3, 4}, models[3] = {m, m, m};
        const pack_input_spec in{4, 1, 1, 64, dtype};
        pack_t* p = nullptr;
        EXPECT(pack_create(&in, models, 3, 0, nullptr, &p) == PACK_OK);
        auto bytes = [&] {
            double sum = 0.0;
            for (int i = 0; i < pack_num_launches(p); ++i) {
                char name[64];
                double b = 0.0;
                EXPECT(pack_launch_name(p, i, name, sizeof name) == PACK_OK && pack_launch_bytes(p, i, &b) == PACK_OK);
                if (std::string(name).rfind("gemm_lin_dw", 0) == 0) sum += b;
            }
            return sum;
        };
        auto choose = [&](int k, int kind) {
            const pack_opt_spec o{kind, 0.9f, 0.1f, 0.9f, 0.999f, 1e-8f};
            EXPECT(pack_set_optimizer(p, k, &o) == PACK_OK);
        };
        const double sgd = bytes();
        for (int k : {1, 0, 2}) choose(k, PACK_OPT_MOMENTUM);
        EXPECT(bytes() == sgd + 3 * params * (4 + 8));     // (packs with such members store their gradients too)
        for (int k : {2, 0, 1}) choose(k, PACK_OPT_ADAM);
        EXPECT(bytes() == sgd + 3 * params * (4 + 16));
        choose(1, PACK_OPT_SGD);
        EXPECT(bytes() == sgd + 3 * params * 4 + 2 * params * 16);
        choose(0, PACK_OPT_ADAGRAD);
        EXPECT(bytes() == sgd + 3 * params * 4 + params * (8 + 16));
        pack_destroy(p);
    }
}

// rows and columns of the tiles of the launches of a kind, in the order of the step
static std::vector<std::pair<int, int>> tiles_of(const pack_t* p, const char* kind) {
    std::vector<std::pair<int, int>> out;
    for (int i = 0; i < pack_num_launches(p); ++i) {
        char name[64];
        int rows = 0, cols = 0, lean = 0;
        EXPECT(pack_launch_name(p, i, name, sizeof name) == PACK_OK && pack_launch_tile(p, i, &rows, &cols, &lean) == PACK_OK);
        if (std::string(name).rfind(kind, 0) == 0) out.emplace_back(rows, cols);
    }
    return out;
}

// the tiles of products with few outputs: small ones in a pack of few members, those that fill the compute units in one of many
static void slim_tiles() {
    const pack_layer layers[] = {{PACK_LINEAR, 512, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 512, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 10, 0}};
    typedef std::vector<std::pair<int, int>> tiles;
    for (int dtype : {PACK_F32, PACK_BF16})
        for (int K : {1, 4, 5, 8, 24, 32, 64}) {
            const pack_model_spec m{layers, 5, 256};
            const std::vector<pack_model_spec> models(K, m);
            const pack_input_spec in{256, 1, 1, 784, dtype};
            pack_t* p = nullptr;
            EXPECT(pack_create(&in, models.data(), K, 0, nullptr, &p) == PACK_OK);
            const std::pair<int, int> want = K <= (dtype == PACK_F32 ? 5 : 4) ? std::make_pair(32, 32) : K <= 8 || (K == 24 && dtype == PACK_F32) ? std::make_pair(64, 64) :
                                             K == 64 && dtype == PACK_BF16 ? std::make_pair(128, 128) : std::make_pair(128, 64);
            EXPECT(tiles_of(p, "gemm_lin_fwd") == tiles(2, want) && tiles_of(p, "gemm_lin_dx") == tiles(1, want));
            pack_destroy(p);
        }
    // fp32 members under Adam next to others: in one launch while they are few
    for (int K : {4, 16}) {
        const pack_model_spec m{layers, 5, 256};
        const std::vector<pack_model_spec> models(K, m);
        const pack_input_spec in{256, 1, 1, 784, PACK_F32};
        pack_t* p = nullptr;
        EXPECT(pack_create(&in, models.data(), K, 0, nullptr, &p) == PACK_OK);
        for (int k = 1; k < K; ++k) {
            const pack_opt_spec o{PACK_OPT_ADAM, 0.9f, 0.1f, 0.9f, 0.999f, 1e-8f};
            EXPECT(pack_set_optimizer(p, k, &o) == PACK_OK);
        }
        EXPECT(tiles_of(p, "gemm_lin_fwd").size() == (K == 4 ? 2 : 4));
        pack_destroy(p);
    }
}

// single-precision weight gradients of convolutions on maps that are no power of two: 64 x 64 tiles where larger ones multiply
// for padding, larger ones where they do not
static void gather_tiles() {
    typedef std::vector<std::pair<int, int>> tiles;
    for (int width : {24, 40, 64, 128}) {
        const pack_layer layers[] = {{PACK_CONV3X3, width, 1}, {PACK_RELU, 0, 0}, {PACK_CONV3X3, 2 * width, 1}, {PACK_RELU, 0, 0},
                                     {PACK_CONV3X3, 4 * width, 2}, {PACK_RELU, 0, 0}, {PACK_GAP, 0, 0}, {PACK_LINEAR, 10, 0}};
        const pack_model_spec m{layers, 8, 32}, models[2] = {m, m};
        const pack_input_spec in{32, 28, 28, 3, PACK_F32};
        pack_t* p = nullptr;
        EXPECT(pack_create(&in, models, 2, 0, nullptr, &p) == PACK_OK);
        const std::pair<int, int> want = width == 128 ? std::make_pair(128, 128) : width == 64 ? std::make_pair(128, 64) : std::make_pair(64, 64);
        EXPECT(tiles_of(p, "gemm_conv_dw") == tiles(1, want));
        pack_destroy(p);
    }
}

// a change of optimiser that changes the form of a member's products, in a pack whose launches are being timed
static void timing() {
    const pack_layer layers[] = {{PACK_LINEAR, 48, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 40, 0}};
    const pack_model_spec m{layers, 3, 4}, models[3] = {m, m, m};
    const pack_input_spec in{4, 1, 1, 64, PACK_F32};
    pack_t* p = nullptr;
    EXPECT(pack_create(&in, models, 3, 0, nullptr, &p) == PACK_OK);
    auto choose = [&](int k, int kind) {
        const pack_opt_spec o{kind, 0.9f, 0.1f, 0.9f, 0.999f, 1e-8f};
        EXPECT(pack_set_optimizer(p, k, &o) == PACK_OK);
    };
    for (int k = 0; k < 3; ++k) choose(k, k == 1 ? PACK_OPT_ADAM : PACK_OPT_MOMENTUM);
    alignas(16) static float x[4 * 64];
    static int32_t y[4];
    const float lr[3] = {0.f, 0.f, 0.f};
    EXPECT(pack_profile_start(p, -1, 1) == PACK_OK);
    EXPECT(pack_step(p, x, y, lr) == PACK_OK);
    choose(0, PACK_OPT_ADAM);       // slim and staged problems share their launches before and after
    EXPECT(pack_step(p, x, y, lr) == PACK_OK);
    auto samples = [&] {
        std::vector<float> ms(pack_num_launches(p));
        std::vector<int32_t> count(pack_num_launches(p));
        EXPECT(pack_profile_stop(p, ms.data(), count.data()) == PACK_OK);
        return count;
    };
    EXPECT(samples() == std::vector<int32_t>(pack_num_launches(p), 2));
    EXPECT(pack_profile_start(p, -1, 1) == PACK_OK);
    choose(2, PACK_OPT_ADAM);
    EXPECT(pack_step(p, x, y, lr) == PACK_OK);
    for (int32_t n : samples()) EXPECT(n == 1);
    pack_destroy(p);
}

// host memory that ends anywhere while a change of optimiser plans the launches again: the pack is what it was
static void no_host_memory() {
    const pack_layer layers[] = {{PACK_LINEAR, 48, 0}, {PACK_RELU, 0, 0}, {PACK_LINEAR, 40, 0}};
    const pack_model_spec m{layers, 3, 4}, models[2] = {m, m};
    const pack_input_spec in{4, 1, 1, 64, PACK_F32};
    pack_t* p = nullptr;
    EXPECT(pack_create(&in, models, 2, 0, nullptr, &p) == PACK_OK);
    const pack_opt_spec adam{PACK_OPT_ADAM, 0.9f, 0.1f, 0.9f, 0.999f, 1e-8f}, momentum{PACK_OPT_MOMENTUM, 0.9f, 0.1f, 0.9f, 0.999f, 1e-8f};
    EXPECT(pack_set_optimizer(p, 0, &adam) == PACK_OK && pack_set_optimizer(p, 1, &momentum) == PACK_OK);
    const auto forms = tiles_of(p, "");
    const size_t bytes = pack_device_bytes(p);
    int n = 0;
    for (;; ++n) {
        t_new_left = n;
        const pack_status st = pack_set_optimizer(p, 1, &adam);
        const bool reached = t_new_left < 0;
        t_new_left = -1;
        if (st == PACK_OK) break;
        EXPECT(reached && st == PACK_ENOMEM && tiles_of(p, "") == forms && pack_device_bytes(p) == bytes);
    }
    EXPECT(n > 20);
    pack_destroy(p);
}

int main(int argc, char** argv) {
    if (argc < 2) return 2;
    alarm(100);
    g_main = std::this_thread::get_id();
    const std::string s = argv[1];
    if (s == "order") {
        for (int i = 0; i < 3; ++i) order(i == 0 ? nullptr : i == 1 ? (void*)hipStreamPerThread : (void*)0x1000, 3001, 997);
        order((void*)hipStreamPerThread, 5, 3);
    } else if (s == "no_pinned") {
        no_pinned();
    } else if (s == "few_threads") {
        few_threads();
    } else if (s == "ready") {
        ready();
    } else if (s == "released") {
        released();
    } else if (s == "work") {
        work();
    } else if (s == "separate_update") {
        separate_update();
    } else if (s == "update_bytes") {
        update_bytes();
    } else if (s == "slim_tiles") {
        slim_tiles();
    } else if (s == "gather_tiles") {
        gather_tiles();
    } else if (s == "timing") {
        timing();
    } else if (s == "no_host_memory") {
        no_host_memory();
    } else if (s == "failures") {
        failures();
    } else {
        return 2;
    }
    for (const std::string& e : g_errors) std::printf("FAIL %s\n", e.c_str());
    std::printf(g_bad || !g_errors.empty() ? "FAILED\n" : "OK\n");
    std::fflush(stdout);
    _exit(g_bad || !g_errors.empty() ? 1 : 0);   // (the streams' threads never end)
}
