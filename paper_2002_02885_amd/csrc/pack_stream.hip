// Streaming kernels of the packed training step between the matrix products: global average pool, shared-input loader
// and loss.  They move each byte once, so what counts is that enough 16-byte loads are in flight and that no element
// costs a division.  As everywhere, one launch handles a list of problems and every sum has a fixed order that depends
// on nothing but the member's own shape.
#include "pack_device.h"

namespace packk {

// ------------------------------------------------------------------------------------------------
// global average pool.  Tensors other than the input hold their channels in groups of 8, so a pixel is whole 16-byte vectors.
// ------------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void unpack(const u32x4_t w, float (&v)[ET<T>::V]) {
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            v[2 * d] = __uint_as_float(w[d] << 16);
            v[2 * d + 1] = __uint_as_float(w[d] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = __uint_as_float(w[d]);
    }
}
template <typename T>
__device__ __forceinline__ u32x4_t pack(const float (&v)[ET<T>::V]) {
    u32x4_t w;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = pack2bf(v[2 * d], v[2 * d + 1]);
    } else {
#pragma unroll
        for (int d = 0; d < 4; ++d) w[d] = __float_as_uint(v[d]);
    }
    return w;
}

// One block pools GAP_VECS vectors of channels (128 bytes of every pixel) of one image: thread (slice, vector) adds the
// pixels slice, slice + 32, ... in order, the slices of a wave are added by a fixed butterfly, the waves in order.
// A thread per channel that walks all pixels, as this was before, has one long chain of 2-byte loads and too few waves:
// five members of 100 x 14 x 14 x 96 bf16 (19 MB) took 53 us, now 8.6 us (the launch itself is about 6).
template <typename T>
__global__ __launch_bounds__(256) void gap_fwd_kernel(const GapProb* __restrict__ probs, const int2* __restrict__ map) {
    constexpr int V = ET<T>::V, SLICES = 256 / GAP_VECS, WAVES = 4;
    const int2 m = map[blockIdx.x];
    const GapProb p = probs[m.x];
    const int vecs = p.c / V, parts = (vecs + GAP_VECS - 1) / GAP_VECS;
    const int n = m.y / parts, part = m.y - n * parts;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lv = threadIdx.x % GAP_VECS, slice = threadIdx.x / GAP_VECS;
    const int vec = part * GAP_VECS + lv;
    float s[V];
#pragma unroll
    for (int e = 0; e < V; ++e) s[e] = 0.f;
    if (vec < vecs) {
        const u32x4_t* const in = (const u32x4_t*)((const T*)p.in + (size_t)n * p.hw * p.c) + vec;
        int i = slice;
        for (; i + 3 * SLICES < p.hw; i += 4 * SLICES) {
            u32x4_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = in[(size_t)(i + j * SLICES) * vecs];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v[V];
                unpack<T>(w[j], v);
#pragma unroll
                for (int e = 0; e < V; ++e) s[e] += v[e];
            }
        }
        for (; i < p.hw; i += SLICES) {
            float v[V];
            unpack<T>(in[(size_t)i * vecs], v);
#pragma unroll
            for (int e = 0; e < V; ++e) s[e] += v[e];
        }
    }
#pragma unroll
    for (int x = GAP_VECS; x < 64; x <<= 1)
#pragma unroll
        for (int e = 0; e < V; ++e) s[e] += __shfl_xor(s[e], x, 64);
    __shared__ float sums[WAVES][GAP_VECS][V];
    if (lane < GAP_VECS)
#pragma unroll
        for (int e = 0; e < V; ++e) sums[wave][lane][e] = s[e];
    __syncthreads();
    if (threadIdx.x < GAP_VECS && vec < vecs) {
        float out[V];
#pragma unroll
        for (int e = 0; e < V; ++e) out[e] = (((sums[0][lv][e] + sums[1][lv][e]) + sums[2][lv][e]) + sums[3][lv][e]) / (float)p.hw;
        *((u32x4_t*)((T*)p.out + (size_t)n * p.c) + vec) = pack<T>(out);
    }
}

// A thread takes whole vectors; the only wide division is the block's own (eight members of 128 x 8 x 8 x 512 bf16, 134 MB: an
// element a thread 77 us, now 31).
template <typename T>
__global__ __launch_bounds__(256) void gap_bwd_kernel(const GapProb* __restrict__ probs, const int2* __restrict__ map) {
    constexpr int V = ET<T>::V, PER_BLOCK = ELEMWISE_PER_BLOCK / V;
    const int2 m = map[blockIdx.x];
    const GapProb p = probs[m.x];
    const unsigned vecs = (unsigned)(p.c / V), image = (unsigned)p.hw * vecs;   // vectors of a pixel, of an image
    const long long total = (long long)p.n * image, first = (long long)m.y * PER_BLOCK;
    const int n0 = (int)(first / image);
    const unsigned rem0 = (unsigned)(first - (long long)n0 * image);
    const float inv = 1.f / (float)p.hw;
    const u32x4_t* const src = (const u32x4_t*)p.in;
    u32x4_t* const dst = (u32x4_t*)p.dz_in;
#pragma unroll
    for (int i = 0; i < PER_BLOCK / 256; ++i) {
        const unsigned t = i * 256 + threadIdx.x;
        const long long idx = first + t;
        if (idx >= total) break;
        const unsigned q = (rem0 + t) / image, at = rem0 + t - q * image;   // (an image may be smaller than a block)
        float g[V];
        unpack<T>(((const u32x4_t*)p.dz_out)[(size_t)(n0 + q) * vecs + at % vecs], g);
#pragma unroll
        for (int e = 0; e < V; ++e) g[e] *= inv;
        if (p.mask) {
            float a[V];
            unpack<T>(src[idx], a);
            if (p.mask == ACT_RELU) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (!(a[e] > 0.f)) g[e] = 0.f;
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) g[e] *= act_deriv(p.mask, a[e]);
            }
        }
        if (p.accum) {
            float old[V];
            unpack<T>(dst[idx], old);
#pragma unroll
            for (int e = 0; e < V; ++e) g[e] += old[e];
        }
        dst[idx] = pack<T>(g);
    }
}

hipError_t launch_gap(bool bf16, bool backward, const GapProb* probs, const int2* map, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (!backward) {
        if (bf16) hipLaunchKernelGGL(gap_fwd_kernel<bf16_t>, dim3(n), dim3(256), 0, st, probs, map);
        else hipLaunchKernelGGL(gap_fwd_kernel<float>, dim3(n), dim3(256), 0, st, probs, map);
    } else {
        if (bf16) hipLaunchKernelGGL(gap_bwd_kernel<bf16_t>, dim3(n), dim3(256), 0, st, probs, map);
        else hipLaunchKernelGGL(gap_bwd_kernel<float>, dim3(n), dim3(256), 0, st, probs, map);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Shared-input loader for packs whose first layer is a convolution over few channels (paper
// Section 3.4: the members read ONE input).  The nine shifted views of the batch are written
// once per step as a dense matrix xcol[(b,i,j), tap*C + c] (zero for taps outside the image and
// for the padding columns up to Kp); every member's first convolution and its weight gradient
// are then plain aligned matrix products over that one buffer, instead of each member gathering
// 3-channel pixels element by element.
// ------------------------------------------------------------------------------------------------
// With one tap the same kernel copies rows whose length is no multiple of 16 bytes into padded rows, so that the
// products over them take aligned loads.  All loaders of a step (strides, or members with data of their own) are one
// launch: an entry of the map is 256 vectors of one loader.  A thread makes one vector; three narrow divisions find its
// pixel and its first tap, the rest are steps (a division per element, as this was before, took longer than the
// memory: eight members of 128 x 64 x 64 pixels, 268 MB out, 183 us, now 135 us).
template <typename T>
__global__ __launch_bounds__(256) void im2col_kernel(const Im2colProb* __restrict__ probs, const int2* __restrict__ map, const char* __restrict__ x_dev) {
    constexpr int V = ET<T>::V;
    const int2 m = map[blockIdx.x];
    const Im2colProb p = probs[m.x];
    const T* const x = (const T*)(x_dev + p.x_off);
    const unsigned groups = (unsigned)(p.Kp / V);
    const long long first = (long long)m.y * 256, rows = (long long)p.B * p.Ho * p.Wo;
    if (first + threadIdx.x >= rows * groups) return;
    const long long r0 = first / groups;   // the block's one wide division
    const unsigned rem = (unsigned)(first - r0 * groups) + threadIdx.x;
    const int g = (int)(rem % groups);
    const long long r = r0 + rem / groups;
    T vals[V];
    if (p.taps == 1) {
        const T* const row = x + r * p.C;
#pragma unroll
        for (int e = 0; e < V; ++e) vals[e] = (g * V + e < p.C) ? row[g * V + e] : (T)0;
    } else {
        const int hw = p.Ho * p.Wo;
        // (r0 is the same in every thread; the rows of a block are at most 256 apart)
        const int b0 = (int)(r0 / hw);
        const unsigned px = (unsigned)(r0 - (long long)b0 * hw) + (unsigned)(r - r0);
        const int b = b0 + (int)(px / (unsigned)hw);
        const int at = (int)(px - (px / (unsigned)hw) * (unsigned)hw);
        const int i = (int)((unsigned)at / (unsigned)p.Wo), j = at - i * p.Wo;
        // tap and channel of the vector's first element; the others by steps
        const unsigned k = (unsigned)(g * V);
        int tap = (int)(k / (unsigned)p.C), c = (int)(k - (unsigned)tap * (unsigned)p.C);
        const T* const img = x + (size_t)b * p.H * p.W * p.C;
        const int y0 = p.stride * i - 1, x0 = p.stride * j - 1;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int u = (tap * 11) >> 5, v = tap - 3 * u;   // tap / 3 for tap < 32
            const int y = y0 + u, xx = x0 + v;
            const bool ok = tap < 9 && (unsigned)y < (unsigned)p.H && (unsigned)xx < (unsigned)p.W;
            vals[e] = ok ? img[(size_t)(y * p.W + xx) * p.C + c] : (T)0;
            if (++c == p.C) {
                c = 0;
                ++tap;
            }
        }
    }
    u32x4_t o;
    __builtin_memcpy(&o, vals, 16);
    *reinterpret_cast<u32x4_t*>((T*)p.out + (size_t)r * p.Kp + g * V) = o;
}

hipError_t launch_im2col(bool bf16, const Im2colProb* probs_dev, const int2* map_dev, int n_blocks, const void* x_dev, hipStream_t st) {
    if (n_blocks <= 0) return hipSuccess;
    if (bf16) hipLaunchKernelGGL(im2col_kernel<bf16_t>, dim3(n_blocks), dim3(256), 0, st, probs_dev, map_dev, (const char*)x_dev);
    else hipLaunchKernelGGL(im2col_kernel<float>, dim3(n_blocks), dim3(256), 0, st, probs_dev, map_dev, (const char*)x_dev);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// softmax cross-entropy, its gradient, and the argmax
// ------------------------------------------------------------------------------------------------
constexpr int CE_PER_LANE = 4;  // classes a lane keeps in registers (fast path: C <= 4 * lanes per row)

// A row is handled by a group of lanes (a power of two, at least min(C, 64)), so a wavefront handles one or more rows at
// once and the logits of a row are read from memory exactly once, into registers.  Row maximum (lowest index among
// equals), sum of exponentials and argmax are combined by a fixed butterfly inside the group.  A row is a chain of a
// load, two butterflies and a store, so a block takes one row per group and a member as many blocks as it has rows
// for: with one block per member, which walked the rows in turn, three members of 256 rows and 100 classes took 43 us, now 6.8.  The blocks leave
// sums of losses, which are added in block order when the loss is read; it depends on nothing but the member's own rows.
template <typename T>
__global__ __launch_bounds__(64 * CE_WAVES) void ce_kernel(const CeProb* __restrict__ probs, const int2* __restrict__ map,
                                                           const int32_t* __restrict__ labels, int* __restrict__ err_flag) {
    const int2 m = map[blockIdx.x];
    const CeProb p = probs[m.x];
    const int lpr = ce_lanes_per_row(p.C);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rpw = 64 / lpr, sub = lane / lpr, sl = lane - sub * lpr;
    const float inv_rows = 1.f / (float)p.rows;
    const bool in_regs = p.C <= CE_PER_LANE * lpr;
    float group_loss = 0.f;
    const int row = m.y * CE_WAVES * rpw + wave * rpw + sub;
    const bool active = row < p.rows;
    const float* z = p.logits + (size_t)(active ? row : 0) * p.ld;
    const int y = active ? labels[p.label_off + row] : 0;
    float zv[CE_PER_LANE];
    float mx = -INFINITY;
    int arg = 0x7fffffff;
    if (in_regs) {
#pragma unroll
        for (int i = 0; i < CE_PER_LANE; ++i) {
            const int c = sl + i * lpr;
            zv[i] = (c < p.C) ? z[c] : -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < CE_PER_LANE; ++i)
            if (zv[i] > mx) { mx = zv[i]; arg = sl + i * lpr; }   // ascending class index
    } else {
        for (int c = sl; c < p.C; c += lpr) {
            const float v = z[c];
            if (v > mx) { mx = v; arg = c; }
        }
    }
    for (int m = lpr >> 1; m > 0; m >>= 1) {
        const float om = __shfl_xor(mx, m, 64);
        const int oa = __shfl_xor(arg, m, 64);
        if (om > mx || (om == mx && oa < arg)) { mx = om; arg = oa; }
    }
    float ev[CE_PER_LANE];
    float s = 0.f;
    if (in_regs) {
#pragma unroll
        for (int i = 0; i < CE_PER_LANE; ++i) {
            ev[i] = (sl + i * lpr < p.C) ? expf(zv[i] - mx) : 0.f;
            s += ev[i];
        }
    } else {
        for (int c = sl; c < p.C; c += lpr) s += expf(z[c] - mx);
    }
    for (int m = lpr >> 1; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
    const bool ok = (y >= 0 && y < p.C);
    if (active && !ok && sl == 0) atomicOr(err_flag, 1);
    // the logit of the label: held by lane y % lpr of the group, slot y / lpr
    float zy = 0.f;
    if (in_regs) {
        const int yy = ok ? y : 0;
        float cand = zv[0];
#pragma unroll
        for (int i = 1; i < CE_PER_LANE; ++i)
            if (yy / lpr == i) cand = zv[i];
        zy = __shfl(cand, sub * lpr + (yy & (lpr - 1)), 64);
    } else if (ok && active) {
        zy = z[y];
    }
    if (active && ok) group_loss += (mx + logf(s)) - zy;
    const float inv_s = 1.f / s;
    T* d = (T*)p.dlogits + (size_t)(active ? row : 0) * p.ldd;
    if (active) {
        if (in_regs) {
#pragma unroll
            for (int i = 0; i < CE_PER_LANE; ++i) {
                const int c = sl + i * lpr;
                if (c < p.C) {
                    const float g = ok ? (ev[i] * inv_s - (c == y ? 1.f : 0.f)) * inv_rows : 0.f;
                    d[c] = ET<T>::from_f(g);
                }
            }
        } else {
            for (int c = sl; c < p.C; c += lpr) {
                const float g = ok ? (expf(z[c] - mx) * inv_s - (c == y ? 1.f : 0.f)) * inv_rows : 0.f;
                d[c] = ET<T>::from_f(g);
            }
        }
        if (sl == 0) p.pred[row] = arg;
    }
    // groups of one wave by a fixed butterfly over the group index, then the waves in order
    float wsum = (sl == 0) ? group_loss : 0.f;
    for (int m = 32; m >= lpr; m >>= 1) wsum += __shfl_xor(wsum, m, 64);
    __shared__ float part[CE_WAVES];
    if (lane == 0) part[wave] = wsum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < CE_WAVES; ++w) t += part[w];
        p.partial[m.y] = t;
    }
}

hipError_t launch_ce(bool bf16, const CeProb* probs, const int2* map, int n, const int32_t* labels, int* err_flag, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (bf16) hipLaunchKernelGGL(ce_kernel<bf16_t>, dim3(n), dim3(64 * CE_WAVES), 0, st, probs, map, labels, err_flag);
    else hipLaunchKernelGGL(ce_kernel<float>, dim3(n), dim3(64 * CE_WAVES), 0, st, probs, map, labels, err_flag);
    return hipGetLastError();
}

// loss of each member = (sum of its blocks' sums, in block order) / rows
template <typename P>
__global__ __launch_bounds__(256) void loss_kernel(const P* __restrict__ probs) {
    const P p = probs[blockIdx.x];
    __shared__ float block_sums[256];
    float total = 0.f;
    for (int b0 = 0; b0 < p.nblk; b0 += 256) {
        const int b = b0 + threadIdx.x;
        block_sums[threadIdx.x] = (b < p.nblk) ? p.partial[b] : 0.f;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < 256 && b0 + i < p.nblk; ++i) total += block_sums[i];
        __syncthreads();
    }
    if (threadIdx.x == 0) *p.loss = total * (1.f / (float)p.rows);
}

hipError_t launch_head_loss(const HeadProb* probs, int n_members, hipStream_t st) {
    if (n_members <= 0) return hipSuccess;
    hipLaunchKernelGGL(loss_kernel<HeadProb>, dim3(n_members), dim3(256), 0, st, probs);
    return hipGetLastError();
}

hipError_t launch_ce_loss(const CeProb* probs, int n_members, hipStream_t st) {
    if (n_members <= 0) return hipSuccess;
    hipLaunchKernelGGL(loss_kernel<CeProb>, dim3(n_members), dim3(256), 0, st, probs);
    return hipGetLastError();
}

}  // namespace packk
