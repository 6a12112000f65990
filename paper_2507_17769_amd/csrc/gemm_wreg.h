// Plan and launcher of the weights-in-registers GEMM (gemm_wreg.hip).
#pragma once
#include "ps_common.h"

namespace ps {

constexpr int WREG_MIN_TM = 5, WREG_MAX_TM = 10;

constexpr int WREG_STAGES = 4;   // register sets of weights; a K share is a whole number of rounds through them
// slots of the activation ring: one more than weight sets where LDS holds it (8 / nc K shares of tm KiB per slot)
constexpr int wreg_ring(int tm, int nc) { return 8 / nc * tm * (WREG_STAGES + 1) <= 160 ? WREG_STAGES + 1 : WREG_STAGES; }

struct WregPlan {
    int tm;         // 16-row tiles per block
    int nc;         // 64-column groups per block: 2 or 4 (8 / nc shares of K inside the block)
    int splits;     // K splits over blocks, each with its own fp32 output (1 for the gate/up matrix)
    int row_tiles;  // blocks over the rows: 16 tm row_tiles >= M
};

// true: the kernel computes this product with this plan
bool wreg_valid(const WregPlan& g, int M, int N, int K, int kind);
hipError_t launch_gemm_wreg(const GemmArgs& a, const WregPlan& g, hipStream_t st);

}  // namespace ps
