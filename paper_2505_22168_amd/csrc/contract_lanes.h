// The one-atom-per-lane contraction kernels and the layout of dE/dG between
// the network and them.
#pragma once

#include "common.h"
#include "contraction.h"

namespace gmnn {

// dE/dG [N][kFP] is stored feature-major inside runs of kDgRun atoms: atom i
// of run r (atoms 64 r .. 64 r + n_r - 1, n_r = 64 but in the last run) has
// feature f at r * 64 * kFP + f * n_r + i % 64.  N * kFP values in all.
constexpr int kDgRun = 64;
__device__ inline int64_t dg_index(int n_atoms, int i, int f) {
  const int r0 = i / kDgRun * kDgRun;
  return (int64_t)r0 * kFP + f * min(kDgRun, n_atoms - r0) + (i - r0);
}

// dE/dG (n_heads arrays one after the other) and psi [N][100] -> dE/dPsi
// (n_heads arrays [N][100])
gmnn_status launch_contract_back(int n_atoms, int n_heads, const float* psi, const float* dG, float* psibar,
                                 hipStream_t s);

}  // namespace gmnn
