// Launcher of the HiF4 GEMM (gemm_hif4.hip); launch_gemm (gemm.hip) plans and calls it.
#pragma once

#include <hip/hip_runtime.h>

namespace resq {

struct GemmParams;

// Launches configuration `cfg` (a tile configuration of gemm_geo.h) with ns stages and kg K
// groups; false if RESQ_HIF4_CONFIGS has no such configuration.
bool launch_gemm_hif4(const GemmParams& p, int cfg, int ns, int kg, int n_terms, hipStream_t s);

}  // namespace resq
