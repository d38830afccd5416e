// Slim form of the dense products for gfx950: forward and input gradient of layers with few outputs (address rules and
// the rule of the dispatch: gemm_slim.h), as a device function.
//
// A staged 64 x 64 tile walks the whole reduction, a round trip and two barriers per chunk, and a small layer has a handful
// of such tiles: two 32 x 128 products over 784 indices are 4 workgroups that take 18.5 us while 252 compute units idle.
// Here a workgroup owns 32 x 32 outputs (64 x 64 where a launch has enough of them) and its eight waves share the chunks of
// the reduction: a wave loads a chunk of 128 bytes of every row, turns it in its own part of LDS, which
// no other wave touches, so that no wave waits for another inside the loop, and adds up its chunks in its own accumulators;
// the eight sums are added in order at the end.  The loads of the next chunk are requested as soon as the registers of
// this one are free.  (Operands straight from memory in the layout of the matrix instructions, without LDS, touch 32 lines
// per load and stop at 30 GB/s per compute unit, against 70 this way.)
// The order of a sum depends on the reduction's length only, whatever the tile, and staged tiles can follow it (gemm_body, SHARES).
#pragma once
#include "gemm_slim.h"
#include "pack_device.h"

namespace packk {

// accumulators of a wave, dealt the steps of its chunks in turn
template <typename T> constexpr int SLIM_SETS = sizeof(T) == 4 ? 2 : 1;

typedef short v4s_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s_t* lds_v4s_ptr;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;

// the tile `tr` of problem `p`, by 64 * SLIM_WAVES threads; lds: SlimCfg::LDS_BYTES
template <int MODE, typename T, int TM, int TN>
__device__ __forceinline__ void slim_body(const GemmProb& p, const TileRef& tr, const void* __restrict__ x, char* const lds) {
    static_assert(MODE == LIN_FWD || MODE == LIN_DX, "dense forward products and input gradients");
    constexpr bool FWD = MODE == LIN_FWD;
    typedef SlimCfg<(int)sizeof(T), !FWD, TM, TN> C;
    constexpr int ESZ = C::ESZ, V = C::V, NA = C::NA, NB = C::NB, NW = SLIM_WAVES;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = tr.tm * C::BM, col0 = tr.tn * C::BN;
    const int R = p.R, Q = p.Q, Kd = p.Kd, lda = p.lda, ldb = p.ldb, flags = p.flags;
    const void* const A = (flags & F_A_INPUT) ? (const char*)x + p.x_off : (const char*)p.A;
    // (both operands span less than 2 GB; an element that does not exist is addressed beyond the window and reads as zero)
    const __amdgpu_buffer_rsrc_t rsa = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)(BUF_RECORDS - 1), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsb = __builtin_amdgcn_make_buffer_rsrc((void*)p.B, 0, (int)(BUF_RECORDS - 1), 0x00020000);

    unsigned va[NA], vb[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) va[i] = slim_a_base<C>(row0, R, lda, lane, i);
#pragma unroll
    for (int i = 0; i < NB; ++i) vb[i] = slim_b_base<C>(col0, Q, ldb, lane, i);

    // fp32: two sums per wave, of the even and the odd steps of its chunks, which halves the rounding
    constexpr int SETS = SLIM_SETS<T>;
    f32x16_t acc[SETS][TM][TN];
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[s][a][b][e] = 0.f;

    char* const la = lds + wave * C::WAVE_BYTES;
    char* const lb = la + C::A_BYTES;
    u32x4_t sa[NA], sb[NB];
    auto request = [&](int c) {   // (chunks beyond the reduction: zeros, no memory access)
        const int k0 = c * C::KC;
#pragma unroll
        for (int i = 0; i < NA; ++i) sa[i] = __builtin_amdgcn_raw_buffer_load_b128(rsa, slim_kc_at<C>(va[i], k0, Kd, lane), 0, 0);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            sb[i] = __builtin_amdgcn_raw_buffer_load_b128(rsb, FWD ? slim_kc_at<C>(vb[i], k0, Kd, lane) : slim_rc_at<C>(vb[i], k0, Kd, ldb, lane, i), 0, 0);
    };
    auto stash = [&]() {
        asm volatile("" ::: "memory");   // (the previous chunk's reads stay in front: LDS operations of a wave keep their order)
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4_t*>(la + slim_kc_lds<C>(lane, i)) = sa[i];
#pragma unroll
        for (int i = 0; i < NB; ++i) *reinterpret_cast<u32x4_t*>(lb + (FWD ? slim_kc_lds<C>(lane, i) : slim_rc_lds<C>(lane, i))) = sb[i];
        asm volatile("" ::: "memory");
    };
    auto multiply = [&]() {
#pragma unroll
        for (int kk = 0; kk < C::KC; kk += 2 * V) {
            f32x16_t(&sum)[TM][TN] = acc[(kk / (2 * V)) % SETS];
            u32x4_t fa[TM], fb[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[a] = *reinterpret_cast<const u32x4_t*>(la + slim_frag_kc<C>(lane, a, kk));
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                if constexpr (FWD) {
                    fb[b] = *reinterpret_cast<const u32x4_t*>(lb + slim_frag_kc<C>(lane, b, kk));
                } else if constexpr (ESZ == 4) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) fb[b][d] = *reinterpret_cast<const unsigned*>(lb + slim_frag_rc32<C>(lane, b, kk, d));
                } else {
                    const v4s_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(lb + slim_frag_rc16<C>(lane, b, kk, 0)));
                    const v4s_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(lb + slim_frag_rc16<C>(lane, b, kk, 1)));
                    fb[b] = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
            if constexpr (ESZ == 2) {
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
                        sum[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fa[a]), __builtin_bit_cast(bf16x8_t, fb[b]), sum[a][b], 0, 0, 0);
            } else {
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b)
                            sum[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa[a][d]), __uint_as_float(fb[b][d]), sum[a][b], 0, 0, 0);
            }
        }
    };
    const int nc = (Kd + C::KC - 1) / C::KC;
    // (every wave a run of neighbouring chunks)
    const int per = (nc + NW - 1) / NW, cend = min(nc, (wave + 1) * per);
    request(wave * per);
    for (int c = wave * per; c < cend; ++c) {
        stash();
        __builtin_amdgcn_sched_barrier(0);
        request(c + 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply();
        __builtin_amdgcn_sched_barrier(0);
    }

    // The eight sums change hands through LDS.  Accumulator register e of a block: row 8*(e/4) + 4*(lane/32) + e%4, column lane%32.
    __syncthreads();
    float(*sum)[C::BM][C::SUM_LD] = reinterpret_cast<float(*)[C::BM][C::SUM_LD]>(lds);
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) sum[wave][a * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)][b * 32 + (lane & 31)] = SETS == 2 ? acc[0][a][b][e] + acc[SETS - 1][a][b][e] : acc[0][a][b][e];
    // what the tail reads from memory comes back under the exchange
    constexpr int G = C::BN / 4, ITEMS = C::BM * G, NIT = (ITEMS + 64 * NW - 1) / (64 * NW);
    const int ldc = p.ldc, cols = stored_cols(p);
    const bool out_f32 = FWD && (flags & F_OUT_F32), whole = ((ldc | cols) & 3) == 0;   // a thread's four columns are stored together
    const T* const aux = (const T*)p.aux;
    f32x4_t extra[NIT];
    float old[NIT][4], msk[NIT][4];
    int rr[NIT], cc[NIT];
#pragma unroll
    for (int n = 0; n < NIT; ++n) {
        const int i = tid + n * 64 * NW;
        rr[n] = row0 + i / G;
        cc[n] = col0 + (i % G) * 4;
        const bool live = i < ITEMS && rr[n] < R && cc[n] < cols;
        if (!live) rr[n] = -1;
        extra[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) { old[n][j] = 0.f; msk[n][j] = 1.f; }
        if (!live) continue;
        if constexpr (FWD) {
            extra[n] = *reinterpret_cast<const f32x4_t*>(p.bias + cc[n]);   // (biases lie on 64-element boundaries, the last four are inside)
        } else {
            const size_t off = (size_t)rr[n] * ldc + cc[n];
            auto four = [&](const T* src, float (&o)[4]) {   // (rows of gradients and activations are whole groups of 8)
                if constexpr (ESZ == 4) {
                    const f32x4_t v = *reinterpret_cast<const f32x4_t*>(src + off);
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[j] = v[j];
                } else {
                    const u32x2_t v = *reinterpret_cast<const u32x2_t*>(src + off);
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[j] = __uint_as_float((j & 1) ? v[j >> 1] & 0xffff0000u : v[j >> 1] << 16);
                }
            };
            if (flags & F_MASK) four(aux, msk[n]);
            if (flags & F_ACCUM) four((const T*)p.C, old[n]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NIT; ++n) {
        if (rr[n] < 0) continue;
        const int r = rr[n] - row0, c = cc[n] - col0;
        f32x4_t part[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) part[w] = *reinterpret_cast<const f32x4_t*>(&sum[w][r][c]);
        f32x4_t v = part[0];
#pragma unroll
        for (int w = 1; w < NW; ++w)   // in order (shares of nothing add zeros)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] += part[w][j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (FWD) {
                v[j] += extra[n][j];
                if (flags & F_RELU) v[j] = fmaxf(v[j], 0.f);
                else if (p.act > ACT_RELU) v[j] = act_apply(p.act, v[j]);
            } else {
                if (flags & F_MASK) {
                    if (p.mask_act == ACT_RELU) { if (!(msk[n][j] > 0.f)) v[j] = 0.f; }
                    else v[j] *= act_deriv(p.mask_act, msk[n][j]);
                }
                if (flags & F_ACCUM) v[j] += old[n][j];
            }
            if (cc[n] + j >= Q) v[j] = 0.f;   // (the padding of a row)
        }
        const size_t off = (size_t)rr[n] * ldc + cc[n];
        if (ESZ == 4 || out_f32) {
            float* const o = (float*)p.C + off;
            if (whole) *reinterpret_cast<f32x4_t*>(o) = v;
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (cc[n] + j < cols) o[j] = v[j];
            }
        } else {
            bf16_t* const o = (bf16_t*)p.C + off;   // (stored in whole groups of 8)
            *reinterpret_cast<u32x2_t*>(o) = u32x2_t{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
        }
    }
}

}  // namespace packk
