// Kernels that move a member's state between its public blob (the checkpoint of `load` / `free`, Section 2.2:
// layers in order, W then b, convolutions [Cout][Cin][3][3]) and the parameter arenas (rows padded for 16-byte
// loads, convolutions tap-major), and that draw seeded initial weights where they lie.
//
// A checkpoint crosses PCIe once and is laid out on the way: the export kernel gathers arena elements in blob
// order and writes them straight into pinned host memory, the import kernel reads pinned host memory and scatters
// into the arena (and its bf16 operand copy).  What bounds both is the link: 4-byte gathers at 52 GB/s are 13 G
// elements/s, some fifty gathers per compute unit and microsecond, so the index arithmetic is free and no device
// staging copy is needed.  Measured, 16 MB: kernel stores to pinned memory 52.7 GB/s, the DMA engine 55.7 GB/s.
#include "pack_internal.h"
#include "pack_device.h"

namespace packk {

// segment of the blob that holds element e (segments are sorted and cover the blob)
__device__ __forceinline__ int seg_of(const BlobSeg* __restrict__ segs, int n_segs, long long e) {
    int lo = 0, hi = n_segs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].blob_off <= e) lo = mid; else hi = mid - 1;
    }
    return lo;
}
// arena offset (from the member's first element) of element i of segment s
__device__ __forceinline__ long long arena_of(const BlobSeg& s, long long i) {
    long long r;
    unsigned j;
    if (i < 0x100000000ll) {
        const unsigned q = (unsigned)i / (unsigned)s.inner;
        r = q;
        j = (unsigned)i - q * (unsigned)s.inner;
    } else {
        r = i / s.inner;
        j = (unsigned)(i - r * s.inner);
    }
    unsigned a, b;
    if (s.conv) { b = j / 9u; a = j - 9u * b; }              // blob (c, tap)
    else { a = j / (unsigned)s.cin; b = j - a * (unsigned)s.cin; }   // blob (pixel, c)
    return s.arena_off + r * s.ldw + (long long)a * s.cpad + b;
}

// calls f(element, arena offset) for the up to four blob elements of a thread; a thread whose four lie in one
// segment looks the segment up once
template <typename F>
__device__ __forceinline__ void for_four(const BlobSeg* __restrict__ segs, int n_segs, long long e0, int live, F&& f) {
    int k = seg_of(segs, n_segs, e0);
    BlobSeg s = segs[k];
    for (int j = 0; j < live; ++j) {
        while (k + 1 < n_segs && segs[k + 1].blob_off <= e0 + j) s = segs[++k];
        f(j, s, e0 + j - s.blob_off);
    }
}

__global__ __launch_bounds__(256) void export_blob_kernel(const float* __restrict__ arena, const BlobSeg* __restrict__ segs, int n_segs,
                                                          long long e0, int n, float* __restrict__ out) {
    const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (t >= n) return;
    float v[4];
    const int live = min(4, n - t);
    for_four(segs, n_segs, e0 + t, live, [&](int j, const BlobSeg& s, long long i) { v[j] = arena[arena_of(s, i)]; });
    if (live == 4) *reinterpret_cast<f32x4_t*>(out + t) = f32x4_t{v[0], v[1], v[2], v[3]};
    else for (int j = 0; j < live; ++j) out[t + j] = v[j];
}

__global__ __launch_bounds__(256) void import_blob_kernel(float* __restrict__ arena, bf16_t* __restrict__ shadow, const BlobSeg* __restrict__ segs,
                                                          int n_segs, long long e0, int n, const float* __restrict__ in) {
    const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (t >= n) return;
    float v[4];
    const int live = min(4, n - t);
    if (live == 4) {
        const f32x4_t w = *reinterpret_cast<const f32x4_t*>(in + t);
        v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    } else {
        for (int j = 0; j < live; ++j) v[j] = in[t + j];
    }
    for_four(segs, n_segs, e0 + t, live, [&](int j, const BlobSeg& s, long long i) {
        const long long a = arena_of(s, i);
        arena[a] = v[j];
        if (shadow) shadow[a] = f2bf(v[j]);
    });
}

// The seeded initial value of element i of a tensor: a hash of (seed, member, tensor, index) mapped to a uniform
// variable in double precision, so that every value is the one the definition gives whatever computes it.
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}
__global__ __launch_bounds__(256) void seed_blob_kernel(float* __restrict__ arena, bf16_t* __restrict__ shadow, const BlobSeg* __restrict__ segs,
                                                        int n_segs, long long n, unsigned long long seed, unsigned long long member) {
    const long long t = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (t >= n) return;
    const int live = (int)(n - t < 4 ? n - t : 4);
    const unsigned long long hm = splitmix64(seed ^ (member << 32));
    for_four(segs, n_segs, t, live, [&](int, const BlobSeg& s, long long i) {
        const unsigned long long h = splitmix64(splitmix64(hm ^ (unsigned long long)s.tensor) ^ (unsigned long long)i);
        const double u = (double)(h >> 11) * (1.0 / 9007199254740992.0);   // [0, 1)
        float v = (float)((2.0 * u - 1.0) * (double)s.bound);
        const long long a = arena_of(s, i);
        if (shadow) {                       // bf16 packs start from weights that their operand copy holds exactly
            const bf16_t b = f2bf(v);
            v = bf2f(b);
            shadow[a] = b;
        }
        arena[a] = v;
    });
}

__global__ __launch_bounds__(256) void fill_value_kernel(float* __restrict__ dst, long long n, float value) {
    const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;   // n is a multiple of 4 (arena segments of 64)
    if (i < n) *reinterpret_cast<f32x4_t*>(dst + i) = f32x4_t{value, value, value, value};
}

hipError_t launch_export_blob(const float* arena, const BlobSeg* segs, int n_segs, long long e0, int n, float* out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(export_blob_kernel, dim3((n + 1023) / 1024), dim3(256), 0, st, arena, segs, n_segs, e0, n, out);
    return hipGetLastError();
}
hipError_t launch_import_blob(float* arena, void* shadow, const BlobSeg* segs, int n_segs, long long e0, int n, const float* in, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(import_blob_kernel, dim3((n + 1023) / 1024), dim3(256), 0, st, arena, (bf16_t*)shadow, segs, n_segs, e0, n, in);
    return hipGetLastError();
}
hipError_t launch_seed_blob(float* arena, void* shadow, const BlobSeg* segs, int n_segs, long long n, unsigned long long seed, unsigned long long member, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(seed_blob_kernel, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st, arena, (bf16_t*)shadow, segs, n_segs, n, seed, member);
    return hipGetLastError();
}
hipError_t launch_fill_value(float* dst, long long n, float value, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_value_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, st, dst, n, value);
    return hipGetLastError();
}

}  // namespace packk
