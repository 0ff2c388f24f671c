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

// A value and its derivative along one direction.
struct Dual {
  float v, t;
};
__device__ inline Dual operator+(Dual a, Dual b) { return {a.v + b.v, a.t + b.t}; }
__device__ inline Dual operator-(Dual a, Dual b) { return {a.v - b.v, a.t - b.t}; }
__device__ inline Dual operator*(Dual a, Dual b) { return {a.v * b.v, a.v * b.t + a.t * b.v}; }
__device__ inline Dual operator*(float a, Dual b) { return {a * b.v, a * b.t}; }
__device__ inline Dual operator*(Dual a, float b) { return {a.v * b, a.t * b}; }
__device__ inline Dual& operator+=(Dual& a, Dual b) { a.v += b.v; a.t += b.t; return a; }
// c += a b
__device__ inline void mac(float& c, float a, float b) { c += a * b; }
__device__ inline void mac(Dual& c, Dual a, Dual b) {
  c.v += a.v * b.v;
  c.t += a.v * b.t;
  c.t += a.t * b.v;
}

// dE/dG (n_heads arrays one after the other) and psi [N][100] -> dE/dPsi
// (n_heads arrays [N][100])
gmnn_status launch_contract_back(int n_atoms, int n_heads, const float* psi, const float* dG, float* psibar,
                                 hipStream_t s);
// The same in dual numbers along the moments' tangent: the backward is linear
// in dE/dG and polynomial in the moments, so with moments psi + eps psid and
// gradients gv + eps gt its value part is the backward of gv at psi and its
// derivative part the backward of gt plus the derivative of the first along psid.
gmnn_status launch_contract_back_dual(int n_atoms, const float* psi, const float* psid, const float* gv,
                                      const float* gt, float* out_v, float* out_t, hipStream_t s);

}  // namespace gmnn
