// Driver of the host-side walk of the slim form of the dense products (csrc/gemm_slim_check.h) for one hand-made problem:
// tests/test_slim_host.py compiles it as it is and once per planted mistake (-DPACK_HALO_PLANT=n).  No GPU code.
#include "pack_internal.h"

#include <cstdio>
#include <cstdlib>
#include <string>

namespace packk {
std::string gemm_fetch_walk(bool bf16, int mode, int bm, int bn, const GemmProb& p, const TileRef& tr, unsigned long long* a_lo,
                            unsigned long long* a_hi, unsigned long long* b_lo, unsigned long long* b_hi, long long* loads);
}

int main(int argc, char** argv) {
    // usage: driver bf16(0|1) dx(0|1) tile R Q Kd
    if (argc != 7) return 2;
    using namespace packk;
    const bool bf16 = std::atoi(argv[1]) != 0, dx = std::atoi(argv[2]) != 0;
    const int tile = std::atoi(argv[3]);
    GemmProb p{};
    p.R = std::atoi(argv[4]); p.Q = std::atoi(argv[5]); p.Kd = p.ksplit = std::atoi(argv[6]);
    auto up = [](int v) { return (v + 7) / 8 * 8; };
    p.lda = up(p.Kd); p.ldb = dx ? up(p.Q) : up(p.Kd); p.ldc = up(p.Q);
    p.flags = F_VEC_A | F_VEC_B | F_SLIM | F_PAD_OUT;
    const unsigned long long esz = bf16 ? 2 : 4, a = 0x100000000ull, b = 0x300000000ull;
    p.A = (const void*)a; p.B = (const void*)b;
    const unsigned long long a_bytes = (unsigned long long)p.R * p.lda * esz, b_bytes = (unsigned long long)(dx ? p.Kd : p.Q) * p.ldb * esz;
    long long loads = 0;
    for (int tm = 0; tm < (p.R + tile - 1) / tile; ++tm)
        for (int tn = 0; tn < (p.Q + tile - 1) / tile; ++tn) {
            unsigned long long alo, ahi, blo, bhi;
            std::string err = gemm_fetch_walk(bf16, dx ? LIN_DX : LIN_FWD, tile, tile, p, TileRef{0, tm, tn, 0}, &alo, &ahi, &blo, &bhi, &loads);
            if (err.empty() && (alo < a || ahi > a + a_bytes || blo < b || bhi > b + b_bytes)) err = "loads leave their operand";
            if (!err.empty()) {
                std::printf("FAIL tile (%d, %d): %s\n", tm, tn, err.c_str());
                return 1;
            }
        }
    std::printf("OK %lld loads\n", loads);
    return 0;
}
