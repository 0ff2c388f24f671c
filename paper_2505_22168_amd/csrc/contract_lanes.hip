// Backward of the invariants (Section 2.1, eq. contraction; product rule),
// one atom per lane: dE/dG and the packed moments -> dE/dPsi (packed).
//
// A block is 64 atoms by five waves; wave k owns channel k.  Every index of
// the contractions is a compile-time constant relative to k (channel
// (k + d) mod 5 is "relative channel d"), so a wave runs straight-line FMAs
// on registers: the moments come from LDS and dE/dG from memory with
// wave-uniform addresses, 64 consecutive atoms per load (dE/dG is stored
// feature-major inside runs of 64 atoms, dg_index).  All tensors are kept
// packed: a symmetric rank-3 tensor is 10 values instead of 27, a rank-2 one
// 6 instead of 9.  Work of wave k:
//   Psi3 of channel k       families 4, 7 and 8, complete (one writer)
//   Psi2, Psi1 of every     family 8 with s2 = k; families 5, 6 (with 2) and
//   channel, partial sums   the T7 of family 7 for the pairs (k, k), (k, k+1),
//                           (k, k+2) mod 5, three of the 15 each; family 3
// The partial sums of the other channels go to their owners through LDS,
// added in a fixed order.
#include "common.h"
#include "model.h"
#include "tables.h"

#include "contract_lanes.h"

namespace gmnn {

constexpr int kClWaves = kS;
constexpr int kClThreads = 64 * kClWaves;
constexpr int kClLd = kDgRun + 1;  // LDS stride of a component's 64 atoms (odd: conflict-free transposes)

// packed component of (a, bc) of a symmetric rank-3 tensor and of (a, b) of a
// rank-2 one; number of full entries of a packed rank-2 component
__device__ constexpr int kI3[3][6] = {{0, 1, 2, 3, 4, 5}, {1, 3, 4, 6, 7, 8}, {2, 4, 5, 7, 8, 9}};
__device__ constexpr int kI2[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
__device__ constexpr int kA2[6] = {0, 0, 0, 1, 1, 2}, kB2[6] = {0, 1, 2, 1, 2, 2};
__device__ constexpr float kW2[6] = {1.0f, 2.0f, 2.0f, 1.0f, 2.0f, 1.0f};

// lexicographic index of the triple {a, b, c}, sorted
__device__ inline int tri_idx(int a, int b, int c) {
  const int lo = min(a, min(b, c)), hi = max(a, max(b, c)), mid = a + b + c - lo - hi;
  const int n = kS - lo, q = kS - mid;
  return kS * (kS + 1) * (kS + 2) / 6 - n * (n + 1) * (n + 2) / 6 + n * (n + 1) / 2 - q * (q + 1) / 2 + hi - mid;
}

// The dual-number form (Dual) holds twice the values: it reads Psi1 and Psi2
// from LDS at each use (a barrier to the compiler between steps keeps it from
// holding them) and fetches dE/dG one step ahead instead of two.
template <typename T>
struct ClLds {
  static constexpr int parts = sizeof(T) / 4;
  static constexpr size_t in = 4 * (size_t)kS * kPacked * kClLd;                // moments, later dE/dPsi (one part)
  static constexpr size_t red = sizeof(T) * (kS - 1) * kS * 9 * kDgRun;         // partial sums for other channels
  static constexpr size_t bytes = parts * in > red ? parts * in : red;
};

// psi, dG: the value parts; psid, dGd (Dual): the derivative parts; out, outd
// likewise
template <typename T>
__device__ __forceinline__ void contract_back_run(int n_atoms, const float* __restrict__ psi,
                                                  const float* __restrict__ psid, const float* __restrict__ dG,
                                                  const float* __restrict__ dGd, float* __restrict__ out,
                                                  float* __restrict__ outd, float* __restrict__ sm) {
  constexpr bool DUAL = sizeof(T) == sizeof(Dual);
  constexpr int NP = kS * kPacked, SP = (int)(ClLds<T>::in / 4), AHEAD = DUAL ? 1 : 2;
  const int tid = threadIdx.x, l = tid & 63;
  const int k = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = min(kDgRun, n_atoms);
  // the run's dE/dG as a buffer: feature f of this lane's atom at f * nt + the
  // lane's atom (a scalar offset and one lane offset for every load)
  const auto rg = __builtin_amdgcn_make_buffer_rsrc((void*)dG, 0, 4 * kFP * nt, 0x00027000);
  const auto rgd = __builtin_amdgcn_make_buffer_rsrc((void*)(DUAL ? dGd : dG), 0, 4 * kFP * nt, 0x00027000);
  const int la = 4 * min(l, nt - 1);
  auto G = [&](int f) {
    const float v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, la, 4 * f * nt, 0));
    if constexpr (DUAL)
      return Dual{v, __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rgd, la, 4 * f * nt, 0))};
    else return v;
  };

  // relative channel d is channel ch[d]
  int ch[kS];
#pragma unroll
  for (int d = 0; d < kS; ++d) ch[d] = k + d < kS ? k + d : k + d - kS;
  // dE/dG of step s (families 8, 7 + 4 and the rest, relative channel s % 5
  // each) arrives AHEAD steps before its use
  T gs[3 * kS][13];
  auto fetch = [&](int s) {
    if (s >= 3 * kS) return;
    const int d = s % kS, p = pair_idx(min(k, ch[d]), max(k, ch[d]));
    T(&o)[13] = gs[s];
    if (s < kS) {
#pragma unroll
      for (int e = 0; e < kS; ++e) o[e] = G(kFam8 + ch[e] * 25 + k * 5 + ch[d]);
    } else if (s < 2 * kS) {
#pragma unroll
      for (int e = 0; e < kS; ++e) o[e] = G(kFam7 + ch[e] * 15 + p);
      o[5] = G(kFam4 + p);
    } else {
      o[0] = G(kFam3 + p);
      if (d <= 2) {
        o[1] = G(kFam2 + p);
#pragma unroll
        for (int e = 0; e < kS; ++e) {
          o[2 + e] = G(kFam6 + p * 5 + ch[e]);
          o[7 + e] = G(kFam5 + tri_idx(ch[e], k, ch[d]));
        }
      }
      if (d == 0) o[12] = G(k);
    }
  };
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) fetch(s);

  // packed moments, 16 bytes a load, all in flight; transposed into LDS
  {
    constexpr int NU = kDgRun * NP / 4 / kClThreads;
    static_assert(NU * kClThreads * 4 == kDgRun * NP, "whole float4 rows");
    float4 v[DUAL ? 2 : 1][NU];
#pragma unroll
    for (int h = 0; h < (DUAL ? 2 : 1); ++h)
#pragma unroll
      for (int q = 0; q < NU; ++q) {
        const int t = tid + q * kClThreads;
        v[h][q] = t < nt * (NP / 4) ? ((const float4*)(h ? psid : psi))[t] : float4{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
    for (int h = 0; h < (DUAL ? 2 : 1); ++h)
#pragma unroll
      for (int q = 0; q < NU; ++q) {
        const int t = tid + q * kClThreads;
        float* o = sm + h * SP + (t % (NP / 4)) * 4 * kClLd + t / (NP / 4);
        o[0] = v[h][q].x;
        o[kClLd] = v[h][q].y;
        o[2 * kClLd] = v[h][q].z;
        o[3 * kClLd] = v[h][q].w;
      }
  }
  __syncthreads();

  auto P = [&](int d, int c) {
    const float* p = sm + (ch[d] * kPacked + c) * kClLd + l;
    if constexpr (DUAL) return Dual{p[0], p[SP]};
    else return p[0];
  };
  float r1[DUAL ? 1 : kS][3], r2[DUAL ? 1 : kS][6];
  if constexpr (!DUAL) {
#pragma unroll
    for (int d = 0; d < kS; ++d) {
#pragma unroll
      for (int a = 0; a < 3; ++a) r1[d][a] = P(d, 1 + a);
#pragma unroll
      for (int c = 0; c < 6; ++c) r2[d][c] = P(d, 4 + c);
    }
  }
  auto p1 = [&](int d, int a) {
    if constexpr (DUAL) return P(d, 1 + a);
    else return r1[d][a];
  };
  auto p2 = [&](int d, int c) {
    if constexpr (DUAL) return P(d, 4 + c);
    else return r2[d][c];
  };
  auto step_begins = [&](int s) {
    fetch(s + AHEAD);
    if constexpr (DUAL) asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  const T zero{};
  T p3[10];
#pragma unroll
  for (int c = 0; c < 10; ++c) p3[c] = P(0, 10 + c);
  // gradients: d1 and d3 packed, u of Psi2 per full entry (the packed
  // gradient is kW2 u)
  T d1[kS][3], u[kS][6], d3[10];
#pragma unroll
  for (int d = 0; d < kS; ++d) {
#pragma unroll
    for (int a = 0; a < 3; ++a) d1[d][a] = zero;
#pragma unroll
    for (int c = 0; c < 6; ++c) u[d][c] = zero;
  }
#pragma unroll
  for (int c = 0; c < 10; ++c) d3[c] = zero;

  // family 8: Psi1[s1]_a Psi3[k]_abc Psi2[s3]_bc
#pragma unroll
  for (int d = 0; d < kS; ++d) {
    step_begins(d);
    const T(&ge)[13] = gs[d];
    T pw[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) pw[c] = kW2[c] * p2(d, c);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T v = zero, q = zero;
#pragma unroll
      for (int c = 0; c < 6; ++c) mac(v, p3[kI3[a][c]], pw[c]);
#pragma unroll
      for (int e = 0; e < kS; ++e) {
        mac(d1[e][a], ge[e], v);
        mac(q, ge[e], p1(e, a));
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        mac(d3[kI3[a][c]], q, pw[c]);
        mac(u[d][c], q, p3[kI3[a][c]]);
      }
    }
  }

  // families 7 and 4 of the pair {k, s}: Psi2[x]_ab Psi3[k]_acd Psi3[s]_bcd
  // and Psi3[k]_abc Psi3[s]_abc (the trace of the same product)
#pragma unroll
  for (int d = 0; d < kS; ++d) {
    step_begins(kS + d);
    const T(&ge)[13] = gs[kS + d];
    const T g4 = ge[5];
    T y[6], q3[10];
#pragma unroll
    for (int c = 0; c < 10; ++c) q3[c] = d == 0 ? p3[c] : P(d, 10 + c);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      y[c] = kA2[c] == kB2[c] ? g4 : zero;
#pragma unroll
      for (int e = 0; e < kS; ++e) mac(y[c], ge[e], p2(e, c));
      if (d == 0) y[c] = 2.0f * y[c];
    }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const T qw = kW2[c] * q3[kI3[b][c]];
#pragma unroll
        for (int a = 0; a < 3; ++a) mac(d3[kI3[a][c]], y[kI2[a][b]], qw);
      }
    if (d <= 2) {
#pragma unroll
      for (int ab = 0; ab < 6; ++ab) {
        const int a = kA2[ab], b = kB2[ab];
        T t = zero;
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          mac(t, p3[kI3[a][c]], kW2[c] * q3[kI3[b][c]]);
          if (a != b) mac(t, p3[kI3[b][c]], kW2[c] * q3[kI3[a][c]]);
        }
        if (a != b) t = 0.5f * t;
#pragma unroll
        for (int e = 0; e < kS; ++e) mac(u[e][ab], ge[e], t);
      }
    }
  }

  // families 6 and 2 of the pairs (k, k + d): Psi1[k]_a Psi1[s]_b Psi2[x]_ab
  // and Psi1[k]_a Psi1[s]_a; family 5: tr(Psi2[k] Psi2[s] Psi2[x]); family 3
#pragma unroll
  for (int d = 0; d < kS; ++d) {
    step_begins(2 * kS + d);
    const T(&gr)[13] = gs[2 * kS + d];
    const T g3 = (d == 0 ? 2.0f : 1.0f) * gr[0];
#pragma unroll
    for (int c = 0; c < 6; ++c) mac(u[0][c], g3, p2(d, c));
    if (d > 2) continue;
    const T g2 = gr[1];
    T w[6];
#pragma unroll
    for (int ab = 0; ab < 6; ++ab) {
      const int a = kA2[ab], b = kB2[ab];
      w[ab] = a == b ? g2 : zero;
      T o = p1(0, a) * p1(d, b);
      if (a != b) {
        mac(o, p1(0, b), p1(d, a));
        o = 0.5f * o;
      }
#pragma unroll
      for (int e = 0; e < kS; ++e) {
        mac(w[ab], gr[2 + e], p2(e, ab));
        mac(u[e][ab], gr[2 + e], o);
      }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const T wab = (d == 0 ? 2.0f : 1.0f) * w[kI2[a][b]];
        mac(d1[0][a], wab, p1(d, b));
        if (d != 0) mac(d1[d][a], wab, p1(0, b));
      }
    T m5[6];
#pragma unroll
    for (int ab = 0; ab < 6; ++ab) {
      const int a = kA2[ab], b = kB2[ab];
      m5[ab] = zero;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        mac(m5[ab], p2(0, kI2[a][c]), p2(d, kI2[c][b]));
        if (a != b) mac(m5[ab], p2(0, kI2[b][c]), p2(d, kI2[c][a]));
      }
      if (a != b) m5[ab] = 0.5f * m5[ab];
    }
#pragma unroll
    for (int e = 0; e < kS; ++e) {
      // 3 (2 for two channels) / (distinct orderings of {x, k, s})
      const float mult = (e == 0 && d == 0) ? 1.0f : (e == 0 || e == d || d == 0) ? 3.0f : 6.0f;
      const T g5 = (3.0f * (d != 0 ? 2.0f : 1.0f) / mult) * gr[7 + e];
#pragma unroll
      for (int c = 0; c < 6; ++c) mac(u[e][c], g5, m5[c]);
    }
  }
  const T d0 = gs[2 * kS][12];

  // partial sums to their owners: slot [d - 1][channel][value][atom]
  T* red = (T*)sm;
  __syncthreads();
#pragma unroll
  for (int d = 1; d < kS; ++d) {
    T* o = red + ((d - 1) * kS + ch[d]) * 9 * kDgRun + l;
#pragma unroll
    for (int a = 0; a < 3; ++a) o[a * kDgRun] = d1[d][a];
#pragma unroll
    for (int c = 0; c < 6; ++c) o[(3 + c) * kDgRun] = u[d][c];
  }
  __syncthreads();
#pragma unroll
  for (int d = 1; d < kS; ++d) {
    const T* o = red + ((d - 1) * kS + k) * 9 * kDgRun + l;
#pragma unroll
    for (int a = 0; a < 3; ++a) d1[0][a] = d1[0][a] + o[a * kDgRun];
#pragma unroll
    for (int c = 0; c < 6; ++c) u[0][c] = u[0][c] + o[(3 + c) * kDgRun];
  }
  __syncthreads();
  auto put = [&](int c, T v) {
    float* o = sm + (k * kPacked + c) * kClLd + l;
    if constexpr (DUAL) {
      o[0] = v.v;
      o[SP] = v.t;
    } else {
      o[0] = v;
    }
  };
  put(0, d0);
#pragma unroll
  for (int a = 0; a < 3; ++a) put(1 + a, d1[0][a]);
#pragma unroll
  for (int c = 0; c < 6; ++c) put(4 + c, kW2[c] * u[0][c]);
#pragma unroll
  for (int c = 0; c < 10; ++c) put(10 + c, d3[c]);
  __syncthreads();
#pragma unroll
  for (int h = 0; h < (DUAL ? 2 : 1); ++h)
#pragma unroll
    for (int q = 0; q < kDgRun * NP / 4 / kClThreads; ++q) {
      const int t = tid + q * kClThreads;
      const float* r = sm + h * SP + (t % (NP / 4)) * 4 * kClLd + t / (NP / 4);
      if (t < nt * (NP / 4)) ((float4*)(h ? outd : out))[t] = float4{r[0], r[kClLd], r[2 * kClLd], r[3 * kClLd]};
    }
}

__global__ void __launch_bounds__(kClThreads) __attribute__((amdgpu_waves_per_eu(3)))
    contract_back(int n_atoms, const float* __restrict__ psi, const float* __restrict__ dG,
                  float* __restrict__ psibar) {
  __shared__ __attribute__((aligned(16))) float sm[ClLds<float>::bytes / 4];
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * kDgRun;
  const int64_t head = (int64_t)blockIdx.y * n_atoms;
  contract_back_run<float>(n_atoms - row0, psi + (int64_t)row0 * kS * kPacked, nullptr, dG + (head + row0) * kFP,
                           nullptr, psibar + (head + row0) * kS * kPacked, nullptr, sm);
}

__global__ void __launch_bounds__(kClThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
    contract_back_dual(int n_atoms, const float* __restrict__ psi, const float* __restrict__ psid,
                       const float* __restrict__ gv, const float* __restrict__ gt, float* __restrict__ out_v,
                       float* __restrict__ out_t) {
  extern __shared__ __attribute__((aligned(16))) float sm_dual[];
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * kDgRun;
  const int64_t p = (int64_t)row0 * kS * kPacked, f = (int64_t)row0 * kFP;
  contract_back_run<Dual>(n_atoms - row0, psi + p, psid + p, gv + f, gt + f, out_v + p, out_t + p, sm_dual);
}

gmnn_status launch_contract_back(int n_atoms, int n_heads, const float* psi, const float* dG, float* psibar,
                                 hipStream_t s) {
  if (n_atoms == 0) return GMNN_OK;
  hipLaunchKernelGGL(contract_back, dim3((n_atoms + kDgRun - 1) / kDgRun, n_heads), dim3(kClThreads), 0, s, n_atoms,
                     psi, dG, psibar);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

gmnn_status launch_contract_back_dual(int n_atoms, const float* psi, const float* psid, const float* gv,
                                      const float* gt, float* out_v, float* out_t, hipStream_t s) {
  if (n_atoms == 0) return GMNN_OK;
  const gmnn_status st = ensure_lds_limit((const void*)contract_back_dual, ClLds<Dual>::bytes);
  if (st != GMNN_OK) return st;
  hipLaunchKernelGGL(contract_back_dual, dim3((n_atoms + kDgRun - 1) / kDgRun), dim3(kClThreads),
                     ClLds<Dual>::bytes, s, n_atoms, psi, psid, gv, gt, out_v, out_t);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

}  // namespace gmnn
