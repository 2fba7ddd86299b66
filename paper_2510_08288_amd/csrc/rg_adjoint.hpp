// Argument block of the weighted adjoint kernels.
#pragma once

#include "rg_internal.hpp"

namespace rg {

struct AdjArgs {
  int Kc;
  int lmax;                // stride of the SoA scratch (= N)
  int cand;                // candidate index whose v is used
  const int32_t* k_list;
  const float* w_list;
  float* out_m;
  double* out_dv;
  double* out_dth;
  float* ckpt;
  float* seg;
  DevGrad* grad;
};

hipError_t launch_adjoint_fc9(const Problem& pr, const AdjArgs& g, int max_entries,
                              const DevBuffers& b, hipStream_t st);

}  // namespace rg
