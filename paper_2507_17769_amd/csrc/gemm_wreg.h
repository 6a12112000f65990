// Launcher of the weights-in-registers GEMM (gemm_wreg.hip).
#pragma once
#include "ps_common.h"

namespace ps {

hipError_t launch_gemm_wreg(const GemmArgs& a, const WregPlan& g, hipStream_t st);

}  // namespace ps
