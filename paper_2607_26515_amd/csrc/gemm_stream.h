// Launcher of the GEMM for grids of few output tiles (gemm_stream.hip); launch_gemm (gemm.hip)
// plans and calls it.
#pragma once

#include <hip/hip_runtime.h>

namespace resq {

struct GemmParams;

// Configurations, as X(format, column tiles per workgroup, waves, K steps in flight per wave).
#define RESQ_STREAM_CONFIGS(X) \
  X(0, 1, 8, 2) X(0, 2, 8, 2) X(0, 2, 4, 2) X(1, 1, 8, 1) X(1, 2, 8, 1) X(1, 3, 8, 1) X(1, 2, 4, 1)

bool launch_gemm_stream(const GemmParams& p, int fmt, int tn, int waves, int steps, int n_terms, hipStream_t s);

}  // namespace resq
