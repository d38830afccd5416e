// Host-side walk of the slim form of the dense products (gemm_slim.h): one tile's loads, chunk by chunk and lane by lane,
// through the waves' parts of LDS to the operands of the matrix instructions, held against the definition of the product
// (OUT[r, q] = sum_k A[r * lda + k] * B(q, k), B(q, k) = B[q * ldb + k] forward, B[k * ldb + q] for an input gradient): a
// load must lie inside the descriptor's window or be cut off, a slot must be written before it is read, and an operand of
// a row that is stored must be the element the definition pairs with it, or zero where there is none.  Part of
// gemm_fetch_check.cpp; nothing here touches a device.
#pragma once
#include "gemm_slim.h"

#include <string>
#include <vector>

namespace packk {
namespace slim_check {

constexpr long long UNWRITTEN = -2, ZERO = -1;

template <class C, class Span>
std::string walk_tile(const GemmProb& p, const TileRef& tr, Span& sa, Span& sb, long long* loads) {
    constexpr int ESZ = C::ESZ, V = C::V;
    const int row0 = tr.tm * C::BM, col0 = tr.tn * C::BN;
    if (row0 < 0 || row0 >= p.R || col0 < 0 || col0 >= p.Q || tr.ks != 0 || p.ksplit < p.Kd) return "the tile lies outside its problem";
    const int nc = (p.Kd + C::KC - 1) / C::KC;
    for (int c = 0; c < nc + SLIM_WAVES; ++c) {   // (a wave requests one chunk beyond its last)
        const int k0 = c * C::KC;
        std::vector<long long> a(C::A_BYTES / ESZ, UNWRITTEN), b(C::B_BYTES / ESZ, UNWRITTEN);   // element offsets from the operands
        for (int which = 0; which < 2; ++which) {
            const bool is_a = which == 0, rc = !is_a && C::DX;
            std::vector<long long>& lds = is_a ? a : b;
            for (int i = 0; i < (is_a ? C::NA : C::NB); ++i)
                for (int lane = 0; lane < 64; ++lane) {
                    const unsigned base = is_a ? slim_a_base<C>(row0, p.R, p.lda, lane, i) : slim_b_base<C>(col0, p.Q, p.ldb, lane, i);
                    const unsigned at = rc ? slim_rc_at<C>(base, k0, p.Kd, p.ldb, lane, i) : slim_kc_at<C>(base, k0, p.Kd, lane);
                    const int slot = (rc ? slim_rc_lds<C>(lane, i) : slim_kc_lds<C>(lane, i));
                    if (slot < 0 || slot % 16 || slot + 16 > (is_a ? C::A_BYTES : C::B_BYTES)) return "a vector is stored outside its wave's part of LDS";
                    const bool cut_off = at >= BUF_POISON;
                    if (!cut_off) {
                        if (c >= nc) return "a chunk beyond the reduction is loaded";
                        if ((unsigned long long)at + 16 > BUF_RECORDS - 1 || at % ESZ) return "a load leaves the descriptor's window";
                        const unsigned long long addr = (unsigned long long)(is_a ? p.A : p.B) + at;
                        if (addr % 16) return "a 16-byte load is not aligned";
                        Span& span = is_a ? sa : sb;
                        span.lo = addr < span.lo ? addr : span.lo;
                        span.hi = addr + 16 > span.hi ? addr + 16 : span.hi;
                        ++*loads;
                    }
                    for (int e = 0; e < V; ++e) {
                        if (lds[slot / ESZ + e] != UNWRITTEN) return "an LDS slot is written twice";
                        lds[slot / ESZ + e] = cut_off ? ZERO : (long long)(at / ESZ) + e;
                    }
                }
        }
        if (c >= nc) continue;
        // a row's element, or zero; beyond the reduction but inside the padded row both operands hold stored zeros
        auto wrong = [&](long long got, bool row_exists, long long row_off, int k, int ld, bool kc) {
            if (!row_exists) return false;   // (never stored)
            if (k < p.Kd) return got != row_off;
            return !(got == ZERO || (kc && k < ld && got == row_off));
        };
        for (int kk = 0; kk < C::KC; kk += 2 * V)
            for (int lane = 0; lane < 64; ++lane)
                for (int e = 0; e < V; ++e) {
                    const int k = k0 + kk + (lane >> 5) * V + e;
                    for (int blk = 0; blk < C::TM; ++blk) {
                        const int r = row0 + blk * 32 + (lane & 31);
                        if (wrong(a[slim_frag_kc<C>(lane, blk, kk) / ESZ + e], r < p.R, (long long)r * p.lda + k, k, p.lda, true)) return "a matrix instruction reads another element of A";
                    }
                    for (int blk = 0; blk < C::TN; ++blk) {
                        const int q = col0 + blk * 32 + (lane & 31);
                        long long got;
                        if (!C::DX) got = b[slim_frag_kc<C>(lane, blk, kk) / ESZ + e];
                        else if (ESZ == 4) got = b[slim_frag_rc32<C>(lane, blk, kk, e) / ESZ];
                        else {
                            // element e of the lane: index e % 4 of half e / 4, from what the lane 4 * (e % 4) + s / 4 of the group addresses
                            const int s = lane & 15, from = (lane & ~15) + 4 * (e & 3) + (s >> 2);
                            got = b[slim_frag_rc16<C>(from, blk, kk, e >> 2) / ESZ + (s & 3)];
                        }
                        const long long want = C::DX ? (long long)k * p.ldb + q : (long long)q * p.ldb + k;
                        if (wrong(got, q < p.Q, want, k, p.ldb, !C::DX)) return "a matrix instruction reads another element of B";
                    }
                }
    }
    return std::string();
}

template <class Span>
std::string walk(bool bf16, int mode, int bm, const GemmProb& p, const TileRef& tr, Span& sa, Span& sb, long long* loads) {
    if (mode == LIN_FWD && bf16 && bm == 64) return walk_tile<SlimCfg<2, false, 2, 2>>(p, tr, sa, sb, loads);
    if (bm != 32 || (mode != LIN_FWD && mode != LIN_DX)) return "no slim form of this product";
    if (mode == LIN_FWD) return bf16 ? walk_tile<SlimCfg<2, false, 1, 1>>(p, tr, sa, sb, loads) : walk_tile<SlimCfg<4, false, 1, 1>>(p, tr, sa, sb, loads);
    return bf16 ? walk_tile<SlimCfg<2, true, 1, 1>>(p, tr, sa, sb, loads) : walk_tile<SlimCfg<4, true, 1, 1>>(p, tr, sa, sb, loads);
}

}  // namespace slim_check
}  // namespace packk
