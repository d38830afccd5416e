// Address rules of the slim form of the dense products (pack_slim.hip): which vectors of the operands a lane loads, where
// they lie in its wave's part of LDS and which elements a matrix instruction's operands are read from.  Included by the
// kernels and by the host-side walk (gemm_slim_check.h), which holds them against the definition of the products.
#pragma once
#include "pack_internal.h"

#ifndef PACK_HALO_PLANT
#define PACK_HALO_PLANT 0
#endif
#ifndef PACK_HD
#define PACK_HD __host__ __device__
#endif

namespace packk {

// ESZ bytes an element; DX: operand B is contiguous along its row index (the weights of an input gradient), else along the
// reduction.  TM x TN blocks of 32 x 32 outputs.  The chunks of the reduction (128 bytes of
// every row) are shared by SLIM_WAVES waves, each taking neighbouring ones.
constexpr int SLIM_WAVES = 8;
template <int ESZ_, bool DX_, int TM_, int TN_>
struct SlimCfg {
    static constexpr int ESZ = ESZ_, TM = TM_, TN = TN_, V = 16 / ESZ, KC = 128 / ESZ, BM = 32 * TM, BN = 32 * TN;
    static constexpr bool DX = DX_;
    static constexpr int LD_KC = 128 + 16;                        // bytes of a staged row of 128: fragment reads of 16 rows hit 64 banks
    static constexpr int VPR = BN * ESZ / 16, RPL = 64 / VPR;     // DX: vectors of a staged reduction index, indices a load covers
    static constexpr int LD_RC = BN * ESZ + ((BN * ESZ) % 128 == 0 ? 64 : 0);   // DX: odd multiples of 64 bytes
    static constexpr int NA = BM / 8, NB = DX ? KC / RPL : BN / 8;              // loads of 64 lanes x 16 bytes per chunk
    static constexpr int A_BYTES = BM * LD_KC, B_BYTES = DX ? KC * LD_RC : BN * LD_KC, WAVE_BYTES = A_BYTES + B_BYTES;
    static constexpr int SUM_LD = BN + 4;
    static constexpr int SUM_BYTES = SLIM_WAVES * BM * SUM_LD * 4;
    static constexpr int LDS_BYTES = SLIM_WAVES * WAVE_BYTES > SUM_BYTES ? SLIM_WAVES * WAVE_BYTES : SUM_BYTES;
    static_assert(64 % VPR == 0 && KC % RPL == 0, "whole loads");
    static_assert(LDS_BYTES <= 160 * 1024, "local memory");
};

// load i of an operand that is contiguous along the reduction: row (of the tile) and reduction index (of the chunk) of the lane's vector
PACK_HD inline int slim_kc_row(int lane, int i) { return i * 8 + (lane >> 3) + (PACK_HALO_PLANT == 11 && i == 1); }
template <class C> PACK_HD inline int slim_kc_pos(int lane) { return (lane & 7) * C::V; }
template <class C> PACK_HD inline int slim_kc_lds(int lane, int i) { return (i * 8 + (lane >> 3)) * C::LD_KC + (lane & 7) * 16; }
// and of one that is contiguous along its rows
template <class C> PACK_HD inline int slim_rc_pos(int lane, int i) { return i * C::RPL + lane / C::VPR; }
template <class C> PACK_HD inline int slim_rc_row(int lane) { return (lane % C::VPR) * C::V; }
template <class C> PACK_HD inline int slim_rc_lds(int lane, int i) { return slim_rc_pos<C>(lane, i) * C::LD_RC + (lane % C::VPR) * 16; }

// Byte offset of the lane's vector of load i at the start of the reduction (BUF_POISON: the row does not exist), and of the
// chunk that starts at k0.  Both operands span less than 2 GB.
template <class C> PACK_HD inline unsigned slim_a_base(int row0, int R, int lda, int lane, int i) {
    const int r = row0 + slim_kc_row(lane, i);
    return r < R ? (unsigned)(r * lda + slim_kc_pos<C>(lane)) * C::ESZ : BUF_POISON;
}
template <class C> PACK_HD inline unsigned slim_b_base(int col0, int Q, int ldb, int lane, int i) {
    const int q = col0 + (C::DX ? slim_rc_row<C>(lane) : slim_kc_row(lane, i));
    if (q >= Q) return BUF_POISON;
    return (unsigned)(C::DX ? slim_rc_pos<C>(lane, i) * ldb + q : q * ldb + slim_kc_pos<C>(lane)) * C::ESZ;
}
template <class C> PACK_HD inline unsigned slim_kc_at(unsigned base, int k0, int Kd, int lane) {
    return k0 + slim_kc_pos<C>(lane) < Kd ? base + (unsigned)k0 * C::ESZ : BUF_POISON;
}
template <class C> PACK_HD inline unsigned slim_rc_at(unsigned base, int k0, int Kd, int ldb, int lane, int i) {
    return (k0 + slim_rc_pos<C>(lane, i) < Kd && base != BUF_POISON) ? base + (unsigned)(k0 * ldb) * C::ESZ : BUF_POISON;
}

// the lane's operand of the matrix instructions of step kk (2 * V reduction indices; the lane holds the V from kk + (lane / 32) * V on):
// where its row's vector begins,
template <class C> PACK_HD inline int slim_frag_kc(int lane, int block, int kk) { return (block * 32 + (lane & 31)) * C::LD_KC + (kk + (lane >> 5) * C::V) * C::ESZ; }
// where element d of its row lies (float),
template <class C> PACK_HD inline int slim_frag_rc32(int lane, int block, int kk, int d) { return (kk + (lane >> 5) * C::V + d) * C::LD_RC + (block * 32 + (lane & 31)) * 4; }
// and what it addresses in the transposing read of its half h (bfloat16: lane s of a group of 16 addresses four consecutive
// rows of one of four consecutive reduction indices, and receives those four indices of row s of the sixteen)
template <class C> PACK_HD inline int slim_frag_rc16(int lane, int block, int kk, int h) {
    return (kk + (lane >> 5) * C::V + 4 * h + ((lane & 15) >> 2)) * C::LD_RC + (block * 32 + (((lane >> 4) & 1) ^ (PACK_HALO_PLANT == 12)) * 16 + (lane & 3) * 4) * 2;
}

// Which dense products are added up in the order of the slim form: those of at most 32 tiles of 64 x 64 (a batch of 256 rows
// by 512 outputs, say).  The rule looks at the problem's own shape only, since a member's bits must not depend on who else is
// in the pack; whether the slim form itself runs or staged tiles that follow its order is the launch's choice
// (add_gemm_launch).  Alone or with a few others such a product leaves most compute units idle and its time is the chain of
// its chunks.  Measured, slim against plain staged: 2 x (32 x 128 over 784, fp32) 6.6 against 18.5 us, 3 x (200 x 304 over
// 784, fp32) 7.6 / 15, 6 x (64 x 504 over 1032, bf16) 4.9 / 11.7, 8 x (48 x 512 over 3072, bf16) 8.0 / 19.9; beyond the line
// 8 x (256 x 1024 over 3072, bf16) 33 / 28.
constexpr int SLIM_MAX_TILES = 32;
inline bool slim_ok(const GemmProb& g) {
    if (g.flags & (F_RES_ID | F_RES_DOWN | F_SC_ID | F_SC_DOWN | F_ROWMAP)) return false;
    return (long long)((g.R + 63) / 64) * ((g.Q + 63) / 64) <= SLIM_MAX_TILES;
}

}  // namespace packk
