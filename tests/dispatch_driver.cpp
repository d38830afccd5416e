// Driver of tests/test_dispatch_host.py: asks the library for every kind of matrix product on every tile configuration, on a
// machine without a GPU (it ends at once where one is visible), where a launch fails because there is no device and a
// configuration the product has no kernel for is refused before that.  Linked with the library itself.
#include "pack_internal.h"

#include <cstdio>
#include <set>

int main() {
    using namespace packk;
    int devices = 0;
    if (hipGetDeviceCount(&devices) == hipSuccess && devices > 0) { std::printf("a GPU is visible\n"); return 3; }
    (void)hipGetLastError();
    int bad = 0;
    static LrTable lr;
    static OptArgs oa;
    for (int mode = LIN_FWD; mode <= CONV_DW; ++mode)
        for (int bf16 = 0; bf16 < 2; ++bf16)
            for (int opt = 0; opt < 2; ++opt) {
                const bool dense = mode == LIN_FWD || mode == LIN_DX, rows = mode == CONV_FWD || mode == CONV_DX, dw = mode == LIN_DW || mode == CONV_DW;
                if (opt && mode != LIN_DW) continue;   // (the others apply SGD or nothing)
                std::set<int> has = {0, 1, 2, GEMM_CFG_SCALAR};
                if (opt) has.insert(GEMM_CFG_LEAN_OPT);
                else if (dw) has.insert(GEMM_CFG_LEAN);
                else has.insert(GEMM_CFG_LEAN64);
                if (rows || mode == CONV_DW) has.insert({GEMM_CFG_GATHER0, GEMM_CFG_GATHER0 + 1});
                if (rows || (mode == CONV_DW && bf16)) has.insert(GEMM_CFG_GATHER0 + 2);
                if (rows) has.insert({GEMM_CFG_GATHER_LEAN64, GEMM_CFG_ROWS64, GEMM_CFG_ROWS32});
                if (mode == CONV_DW) has.insert({GEMM_CFG_HALO_S1, GEMM_CFG_HALO_S2, GEMM_CFG_HALO32_S1});
                if (mode == CONV_DW && !bf16) has.insert(GEMM_CFG_GATHER_LEAN_DW);
                if (dense) has.insert(GEMM_CFG_SLIM32);
                if (mode == LIN_FWD && bf16) has.insert(GEMM_CFG_SLIM64);
                if (dense) has.insert({GEMM_CFG_SHARES64, GEMM_CFG_SHARES128X64});
                if (dense && bf16) has.insert(GEMM_CFG_SHARES128);
                if (dense && !bf16) has.insert(GEMM_CFG_SLIM_MIXED);
                for (int cfg = -1; cfg <= (int)(sizeof(GEMM_TILE_M) / sizeof(int)); ++cfg) {
                    lr.opt = opt ? &oa : nullptr;
                    const hipError_t e = launch_gemm(mode, bf16 != 0, cfg, nullptr, nullptr, 1, nullptr, nullptr, lr, nullptr);
                    (void)hipGetLastError();
                    const bool want = has.count(cfg) != 0, refused = e == hipErrorInvalidValue, started = !refused && e != hipSuccess;
                    if (want ? !started : !refused) {
                        ++bad;
                        std::printf("FAIL product %d, bf16 %d, optimisers %d, configuration %d: %s\n", mode, bf16, opt, cfg, hipGetErrorName(e));
                    }
                }
            }
    if (!bad) std::printf("OK\n");
    return bad != 0;
}
