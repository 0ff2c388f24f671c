// Training gradients of an energy + force loss (Section 3.4: weighted loss
// terms on energies and forces; Section 3.3: forces are -dE/dx, so the force
// term needs the mixed second derivative of E).
//
// With upstream gradients ebar_b = dL/dEbar_b and lambda = dL/dF, every
// parameter gradient is the gradient of
//     Phi(theta) = sum_i a_i Ebar_i(theta) - D(theta),   a_i = ebar_{b(i)},
//     D = sum_p delta_p . dEbar/dd_p,   delta_p = lambda_j(p) - lambda_i(p),
// i.e. of the energy plus the directional derivative of the energy along
// the position perturbation lambda.  D is evaluated in forward (tangent)
// mode and Phi differentiated in reverse mode:
//   pair_tangent    Psidot_i = sum_p dPsi/dd_p . delta_p
//   train_features  invariants G and their tangent Gdot (in dual numbers: the
//                   product rule on every contraction family, exact since G
//                   is a polynomial), 6 atoms per block
//   train_network   the network forward in dual numbers, a 16-row MFMA block
//                   of primal rows next to one of tangent rows, and its
//                   reverse pass; writes the rows the weight products need
//   contract_back_dual  the invariant backward in dual numbers, one atom per
//                   lane: Psidotbar = J^T Gdotbar and
//                   Psibar = J^T Gbar + (d/dPsi J^T Gdotbar) Psidot
//   pair_beta_grad  dPhi/dbeta per pair, reduced per (Z_i, Z_j) without
//                   atomics on the result
//   weight_grad     W1bar = [G;Gdot]^T [z1bar;z1dotbar],
//                   W2bar = [h1;h1dot]^T [z2bar;z2dotbar] as split-K MFMA
//                   products over all atoms, partials summed in a fixed order
//   reductions      bias, W3, scale and shift gradients (fixed order)
#include <algorithm>
#include <cstdint>

#include "common.h"
#include "contract_lanes.h"
#include "contraction.h"
#include "mfma_rows.h"
#include "model.h"
#include "pair_math.h"

namespace gmnn {

constexpr int kTrainThreads = 512;  // threads of a training network block
constexpr int kTrainWaves = kTrainThreads / 64;
constexpr int kTfAtoms = 6;         // atoms and threads of a training invariant block
constexpr int kTfThreads = 256;

// Rows of the weight products (X1, Y1, X2, Y2): 16 per group of 8 atoms, its
// primal rows and its tangent rows, groups in the order in which blocks of one
// group each would be dispatched (xcd_block's inverse); rows of absent atoms
// are zero.  The order is that of the sums over atoms, which BF16 training
// keeps bit for bit (see train_contract).
constexpr int kRowAtoms = 8;
__device__ __forceinline__ int group_rows(int n_atoms, int group) {
  const int nb = (n_atoms + kRowAtoms - 1) / kRowAtoms, q = nb / kXcds, r = nb % kXcds;
  const int long_runs = r * (q + 1);  // groups of the first r runs, q + 1 each
  const int x = group < long_runs ? group / (q + 1) : r + (group - long_runs) / q;
  const int k = group < long_runs ? group % (q + 1) : (group - long_runs) % q;
  return 16 * (k * kXcds + x);
}

// directional derivative of every monomial at u along v
__device__ inline void dmonomials(float x, float y, float z, float vx, float vy, float vz, float* d) {
  d[0] = 0.0f;
  d[1] = vx; d[2] = vy; d[3] = vz;
  d[4] = 2.0f * x * vx; d[5] = x * vy + y * vx; d[6] = x * vz + z * vx;
  d[7] = 2.0f * y * vy; d[8] = y * vz + z * vy; d[9] = 2.0f * z * vz;
  d[10] = 3.0f * x * x * vx;
  d[11] = 2.0f * x * y * vx + x * x * vy;
  d[12] = 2.0f * x * z * vx + x * x * vz;
  d[13] = y * y * vx + 2.0f * x * y * vy;
  d[14] = y * z * vx + x * z * vy + x * y * vz;
  d[15] = z * z * vx + 2.0f * x * z * vz;
  d[16] = 3.0f * y * y * vy;
  d[17] = 2.0f * y * z * vy + y * y * vz;
  d[18] = z * z * vy + 2.0f * y * z * vz;
  d[19] = 3.0f * z * z * vz;
}

// ---------------------------------------------------------------------------
// Psidot_i = sum_p [ dR_s (u.delta) mono(u) + R_s Dmono(u)[delta_perp / r] ]
template <int LPA>
__global__ void __launch_bounds__(kPairBlock) pair_tangent(DevModel m, DevSystem sys, const float* __restrict__ lambda,
                                                           float* __restrict__ psidot) {
  extern __shared__ float s_beta[];
  stage_beta(m, s_beta);
  __syncthreads();
  const int q = threadIdx.x & (LPA - 1);
  const int i = xcd_block(blockIdx.x, gridDim.x) * (kPairBlock / LPA) + threadIdx.x / LPA;
  const bool live = i < sys.n_atoms;
  float v[128];
#pragma unroll
  for (int k = 0; k < 128; ++k) v[k] = 0.0f;
  if (live) {
    AtomCtx c;
    load_atom(sys, i, c);
    const float* bzi = s_beta + c.zsp * m.n_species * kS * kMaxBasis;
    const float lix = lambda[3 * (int64_t)i], liy = lambda[3 * (int64_t)i + 1], liz = lambda[3 * (int64_t)i + 2];
    for (int64_t p = c.p0 + q; p < c.p1; p += LPA) {
      int j;
      float dx, dy, dz;
      pair_vec(sys, c, p, j, dx, dy, dz);
      const float r2 = dx * dx + dy * dy + dz * dz;
      if (!(r2 < m.rc2) || r2 == 0.0f) continue;
      float r, ir;
      length_of(r2, r, ir);
      const float ux = dx * ir, uy = dy * ir, uz = dz * ir;
      const float ex = lambda[3 * (int64_t)j] - lix, ey = lambda[3 * (int64_t)j + 1] - liy,
                  ez = lambda[3 * (int64_t)j + 2] - liz;
      const float ud = ux * ex + uy * ey + uz * ez;
      Radial rad;
      radial<true>(m, bzi + sys.species[j] * kS * kMaxBasis, r, rad);
      float mo[20], dm[20];
      monomials(ux, uy, uz, mo);
      dmonomials(ux, uy, uz, (ex - ud * ux) * ir, (ey - ud * uy) * ir, (ez - ud * uz) * ir, dm);
#pragma unroll
      for (int s = 0; s < kS; ++s) {
        const float a = rad.dR[s] * ud;
#pragma unroll
        for (int t = 0; t < kPacked; ++t) v[s * kPacked + t] += a * mo[t] + rad.R[s] * dm[t];
      }
    }
  }
  reduce_scatter_128<LPA>(v, q);
  constexpr int OWN = 128 / LPA;
  if (live) {
#pragma unroll
    for (int e = 0; e < OWN; ++e) {
      const int idx = OWN * q + e;
      if (idx < kS * kPacked) psidot[(int64_t)i * (kS * kPacked) + idx] = v[e];
    }
  }
}

// ---------------------------------------------------------------------------
__device__ inline void swish_d2(float z, float& s, float& d1, float& d2) {
  const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-z));  // hardware reciprocal, as swish_parts
  s = z * sg;
  d1 = sg * (1.0f + z * (1.0f - sg));
  d2 = sg * (1.0f - sg) * (2.0f + z * (1.0f - 2.0f * sg));
}

// ---------------------------------------------------------------------------
// Invariants (with PRIMAL) and their tangents into X1, the rows of the first
// weight product.  What bounds it: latency of the short
// contraction tasks between block barriers, as in readout_features, so its
// block size (three blocks per CU at 49 KB of LDS); the sums are those of the
// earlier 8-atom training tile, term by term, which keeps the BF16 network's
// operand roundings where they were.
static constexpr size_t tf_al(size_t x) { return (x + 255) & ~size_t(255); }
struct TrainFeatLds {
  static constexpr size_t psi = tf_al(sizeof(Tables));
  static constexpr size_t psid = psi + tf_al(4 * (size_t)kTfAtoms * PS);
  static constexpr size_t inter = psid + tf_al(4 * (size_t)kTfAtoms * PS);
  static constexpr size_t interd = inter + tf_al(4 * (size_t)kTfAtoms * ISF);
  static constexpr size_t g = interd + tf_al(4 * (size_t)kTfAtoms * ISF);
  static constexpr size_t gd = g + tf_al(4 * (size_t)kTfAtoms * kFP);
  static constexpr size_t bytes = gd + tf_al(4 * (size_t)kTfAtoms * kFP);
};

template <bool PRIMAL>
__global__ void __launch_bounds__(kTfThreads) train_features(int n_atoms, const float* __restrict__ psi,
                                                             const float* __restrict__ psid,
                                                             float* __restrict__ X1) {
  using L = TrainFeatLds;
  constexpr int TA = kTfAtoms, NT = kTfThreads, NP = kS * kPacked;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  Tables& tb = *(Tables*)lds;
  float* sPsi = (float*)(lds + L::psi);
  float* sPd = (float*)(lds + L::psid);
  float* sI = (float*)(lds + L::inter);
  float* sId = (float*)(lds + L::interd);
  float* sG = (float*)(lds + L::g);
  float* sGd = (float*)(lds + L::gd);
  const int tid = threadIdx.x;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * TA;
  const int n_rows = min(TA, n_atoms - row0);
  // packed moments and tangents are contiguous runs: every load issued at
  // once, then expanded into the full tensors
  constexpr int NU = (TA * NP + NT - 1) / NT;
  float v[NU], vd[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int t = tid + u * NT;
    const bool ok = t < n_rows * NP;
    v[u] = ok ? psi[(int64_t)row0 * NP + t] : 0.0f;
    vd[u] = ok ? psid[(int64_t)row0 * NP + t] : 0.0f;
  }
  load_tables(&tb);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int t = tid + u * NT;
    if (t < TA * NP) {
      const int a = t / NP, e = t % NP;
      const int s = e / kPacked, c = e % kPacked;
      const int n = tb.packed_mult[c];
      for (int q = 0; q < n; ++q) {
        sPsi[a * PS + s * kFull + tb.packed_full[c][q]] = v[u];
        sPd[a * PS + s * kFull + tb.packed_full[c][q]] = vd[u];
      }
    }
  }
  __syncthreads();
  constexpr int KSF = 2 * ((TA * 20 + 63) / 64 * 64) <= NT ? 2 : 1;
  contract_forward_a<TA, NT, false, PRIMAL, ISF, KSF>(sPsi, sI, sG, kFP, tb);
  contract_forward_a_dual<TA, NT, ISF, KSF>(sPsi, sPd, sId, sGd, kFP);
  __syncthreads();
  if (PRIMAL) contract_forward_b<TA, NT, false, ISF>(sPsi, sI, sG, kFP, tb);
  contract_forward_b_dual<TA, NT, ISF, ISF>(sPsi, sPd, sI, sId, sGd, kFP, tb);
  __syncthreads();
  // the block of the last atom also clears the rows of its group's absent atoms
  const int n_out = row0 + n_rows < n_atoms ? n_rows : (n_atoms + kRowAtoms - 1) / kRowAtoms * kRowAtoms - row0;
  constexpr int C4 = kFP / 4;
  for (int t = tid; t < n_out * C4; t += NT) {
    const int a = t / C4, i = row0 + a;
    float4* o = (float4*)(X1 + (int64_t)(group_rows(n_atoms, i / kRowAtoms) + i % kRowAtoms) * kFP) + t % C4;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (PRIMAL) o[0] = a < n_rows ? ((const float4*)sG)[t] : zero;
    o[kRowAtoms * C4] = a < n_rows ? ((const float4*)sGd)[t] : zero;
  }
}

// ---------------------------------------------------------------------------
// The network in dual numbers on tiles of 16 AB atoms: row block 2 q holds the
// primal rows of atoms 16 q .. 16 q + 15, row block 2 q + 1 their tangent
// rows, so a lane's accumulators hold both values of the same atom and unit
// (products transposed as in readout_network: four consecutive units of one
// atom per lane).  Rows of the weight products (X1, X2 and Y1, Y2) are read
// and written as 16-byte runs.  BF16: operands
// rounded once as they are stored; FP32: three parts (mfma.h).
//   X1 = [G; Gdot] in; X2 = [h1; h1dot], Y2 = [z2bar; z2dotbar],
//   Y1 = [z1bar; z1dotbar] out; Gbar, Gdbar out (dg_index)
template <int HP, bool BF16, int AB>
struct TrainNetLds {
  static constexpr int TM = 32 * AB, NP = BF16 ? 1 : 3;
  static constexpr int G = kFP + 8, H = HP + 8;  // row strides (bf16)
  static constexpr size_t al(size_t x) { return (x + 255) & ~size_t(255); }
  static constexpr size_t part_g = (size_t)TM * G, part_h = (size_t)TM * H;
  static constexpr size_t rows = 0;                                        // scale, a
  static constexpr size_t ep = rows + al(4 * 2 * 16 * (size_t)AB);         // [waves][TM] partial sums
  static constexpr size_t a = ep + al(4 * (size_t)kTrainWaves * TM);
  static constexpr size_t bytes = a + al(2 * NP * (part_g > part_h ? part_g : part_h));
};

template <int HP, bool BF16, int AB>
__global__ void __launch_bounds__(kTrainThreads)
    train_network(DevModel m, DevSystem sys, const double* __restrict__ ebar, const float* __restrict__ X1,
                  float* __restrict__ Y1, float* __restrict__ X2, float* __restrict__ Y2, float* __restrict__ w3g,
                  float* __restrict__ qsig, float* __restrict__ Gbar, float* __restrict__ Gdbar) {
  using L = TrainNetLds<HP, BF16, AB>;
  constexpr int NP = L::NP, MB = 2 * AB, NW = kTrainWaves;
  constexpr int NBH = HP / 16, NBG = kFP / 16;
  constexpr int TPW = (NBH + NW - 1) / NW, TPW_G = (NBG + NW - 1) / NW;
  constexpr int PG = (int)L::part_g, PH = (int)L::part_h;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  float* sScale = (float*)(lds + L::rows);
  float* sA = sScale + 16 * AB;
  float* sEp = (float*)(lds + L::ep);
  __bf16* sT = (__bf16*)(lds + L::a);
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63;
  const int N = sys.n_atoms;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * 16 * AB;
  const int n_rows = min(16 * AB, N - row0);
  // a lane's accumulator entries j = 0..3: unit uq + j of the column block,
  // atom ar of the row block
  const int ar = l & 15, uq = 4 * (l >> 4);
  RowsRing<NP, TPW> ring;
  RowsRing<NP, TPW_G> ring_g;
  // primal weight-product row of atom a of the tile; its tangent row is kRowAtoms on
  auto group_at = [&](int k) {
    const int g = row0 / kRowAtoms + k;
    return g * kRowAtoms < N ? group_rows(N, g) : 0;
  };
  const int r0 = group_at(0), d1 = group_at(1) - r0;
  const int d2 = AB > 1 ? group_at(2) - d1 - r0 : 0, d3 = AB > 1 ? group_at(3) - d2 - d1 - r0 : 0;
  auto prow = [&](int a) {
    int r = r0 + a % kRowAtoms + (a >= kRowAtoms ? d1 : 0);
    if (AB > 1) r += (a >= 2 * kRowAtoms ? d2 : 0) + (a >= 3 * kRowAtoms ? d3 : 0);
    return (int64_t)r;
  };
  const int n_out = min(16 * AB, (N + kRowAtoms - 1) / kRowAtoms * kRowAtoms - row0);  // with the absent atoms' rows

  {
    constexpr int C4 = kFP / 4;
    constexpr int NU = L::TM * C4 / kTrainThreads;
    static_assert(NU * kTrainThreads == L::TM * C4, "whole rounds of loads");
    floatx4 v[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = tid + u * kTrainThreads;
      const int row = t / C4, a = (row / 32) * 16 + row % 16;
      v[u] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
      if (a < n_rows) v[u] = ((const floatx4*)(X1 + (prow(a) + ((row / 16) & 1) * kRowAtoms) * kFP))[t % C4];
    }
    rows_pre<NP, TPW>(ring, m.w1, kFP / 32, w, NW, NBH);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = tid + u * kTrainThreads;
      st4<NP>(sT, PG, (t / C4) * L::G + (t % C4) * 4, (t % C4) * 4, v[u]);
    }
    for (int a = tid; a < 16 * AB; a += kTrainThreads) {
      sScale[a] = a < n_rows ? m.scale[sys.species[row0 + a]] : 0.0f;
      sA[a] = a < n_rows ? (float)ebar[sys.atom_struct[row0 + a]] : 0.0f;
    }
  }
  lds_barrier();

  // the two rows of atom `a` (in the tile) and unit col of a weight-product array
  auto put = [&](float* X, int a, int col, floatx4 p, floatx4 t) {
    if (a < n_out) {
      const floatx4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
      float* o = X + prow(a) * HP + col;
      *(floatx4*)o = a < n_rows ? p : zero;
      *(floatx4*)(o + kRowAtoms * HP) = a < n_rows ? t : zero;
    }
  };
  // the tile's operands of the next product, once every wave has read this one's
  auto stage = [&](const floatx4 (&acc)[MB][TPW]) {
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if (!has_block(i, w, NW, NBH)) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        const int col = (w + i * NW) * 16 + uq;
        st4<NP>(sT, PH, (r * 16 + ar) * L::H + col, col, acc[r][i]);
      }
    }
    lds_barrier();
  };

  // ---- forward: z1, h1 and their tangents -------------------------------------
  floatx4 s1d[AB][TPW], s1dd[AB][TPW], z1dot[AB][TPW];
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NP>(ring, sT, PG, L::G, m.w1, kFP / 32, w, NW, NBH, acc);
    rows_pre<NP, TPW>(ring, m.w2, HP / 32, w, NW, NBH);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if (!has_block(i, w, NW, NBH)) continue;
      const int col = (w + i * NW) * 16 + uq;
      const floatx4 bias = *(const floatx4*)(m.b1 + col);
#pragma unroll
      for (int q = 0; q < AB; ++q) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float zd = acc[2 * q + 1][i][j];
          float s, d1, d2;
          swish_d2(acc[2 * q][i][j] + bias[j], s, d1, d2);
          s1d[q][i][j] = d1;
          s1dd[q][i][j] = d2;
          z1dot[q][i][j] = zd;
          acc[2 * q][i][j] = s;
          acc[2 * q + 1][i][j] = d1 * zd;
        }
        put(X2, q * 16 + ar, col, acc[2 * q][i], acc[2 * q + 1][i]);
      }
    }
    stage(acc);
  }
  // ---- z2, h2, their tangents, and the adjoints z2bar, z2dotbar ----------------
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NP>(ring, sT, PH, L::H, m.w2, HP / 32, w, NW, NBH, acc);
    rows_pre<NP, TPW>(ring, m.w2t, HP / 32, w, NW, NBH);
    float part[MB][4];  // sums over this wave's units of h2 . w3bar and h2dot . w3bar
#pragma unroll
    for (int r = 0; r < MB; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j) part[r][j] = 0.0f;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if (!has_block(i, w, NW, NBH)) continue;
      const int col = (w + i * NW) * 16 + uq;
      const floatx4 bias = *(const floatx4*)(m.b2 + col);
      const floatx4 wbv = *(const floatx4*)(m.w3bar + col);
#pragma unroll
      for (int q = 0; q < AB; ++q) {
        const int a = q * 16 + ar;
        const float sg = sScale[a], aa = sA[a];
        floatx4 gw;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float wb = wbv[j], zd = acc[2 * q + 1][i][j];
          float h2, d1, dd;
          swish_d2(acc[2 * q][i][j] + bias[j], h2, d1, dd);
          const float h2d = d1 * zd;
          const float hbar = aa * sg * wb;   // dPhi/dh2
          const float hdbar = -sg * wb;      // dPhi/dh2dot
          part[2 * q][j] += h2 * wb;
          part[2 * q + 1][j] += h2d * wb;
          gw[j] = (aa * h2 - h2d) * sg / (float)m.M;
          acc[2 * q][i][j] = __builtin_fmaf(hdbar * dd, zd, hbar * d1);
          acc[2 * q + 1][i][j] = hdbar * d1;
        }
        if (a < n_rows) *(floatx4*)(w3g + (int64_t)(row0 + a) * HP + col) = gw;
        put(Y2, a, col, acc[2 * q][i], acc[2 * q + 1][i]);
      }
    }
    // over the 16 units of a block: bits 3 and 2 across the lane groups, 1
    // and 0 inside the lane
#pragma unroll
    for (int r = 0; r < MB; ++r) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        part[r][j] += __shfl_xor(part[r][j], 32);
        part[r][j] += __shfl_xor(part[r][j], 16);
      }
      const float v = (part[r][0] + part[r][2]) + (part[r][1] + part[r][3]);
      if (l < 16) sEp[w * L::TM + r * 16 + ar] = v;
    }
    stage(acc);
  }
  // scale gradient per atom: a ybar_mean - ydot_mean, with y_mean = h2 . w3bar + mean b3
  if (tid < n_rows) {
    const int r = tid / 16 * 32 + tid % 16;
    float yp = 0.0f, yt = 0.0f, b3m = 0.0f;
    for (int hm = 0; hm < m.M; ++hm) b3m += m.b3[hm];
    b3m /= (float)m.M;
    for (int ww = 0; ww < NW; ++ww) {
      yp += sEp[ww * L::TM + r];
      yt += sEp[ww * L::TM + r + 16];
    }
    qsig[row0 + tid] = sA[tid] * (yp + b3m) - yt;
  }
  // ---- reverse ------------------------------------------------------------------
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NP>(ring, sT, PH, L::H, m.w2t, HP / 32, w, NW, NBH, acc);
    rows_pre<NP, TPW_G>(ring_g, m.w1t, HP / 32, w, NW, NBG);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if (!has_block(i, w, NW, NBH)) continue;
#pragma unroll
      for (int q = 0; q < AB; ++q) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float hbar = acc[2 * q][i][j], hdbar = acc[2 * q + 1][i][j];
          acc[2 * q][i][j] = hbar * s1d[q][i][j] + hdbar * s1dd[q][i][j] * z1dot[q][i][j];
          acc[2 * q + 1][i][j] = hdbar * s1d[q][i][j];
        }
        put(Y1, q * 16 + ar, (w + i * NW) * 16 + uq, acc[2 * q][i], acc[2 * q + 1][i]);
      }
    }
    stage(acc);
  }
  {
    floatx4 acc[MB][TPW_G];
    zero_rows(acc);
    mma_rows<NP, MB, TPW_G, true>(ring_g, sT, PH, L::H, m.w1t, HP / 32, w, NW, NBG, acc);
#pragma unroll
    for (int i = 0; i < TPW_G; ++i) {
      if (!has_block(i, w, NW, NBG)) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        const int a = r / 2 * 16 + uq;  // a lane's four atoms (of one feature)
        if (a >= n_rows) continue;
        float* o = (r & 1 ? Gdbar : Gbar) + dg_index(N, row0 + a, (w + i * NW) * 16 + ar);
        if (N - (row0 + a) / kDgRun * kDgRun >= kDgRun) {
          *(floatx4*)o = acc[r][i];  // a whole run: its rows are 16-byte aligned
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (a + j < n_rows) o[j] = acc[r][i][j];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The invariant backward of the BF16 per-head double backward, 8 atoms a block:
//   Psidotbar = B(Psi; Gdbar),
//   Psibar = B(Psi; Gbar) + [B(Psi + t Psidot; Gdbar) - B(Psi - t Psidot; Gdbar)] / (2 t)
// (exact for B's cubic polynomials, t = |Psi| / |Psidot|).  The one-atom-per-
// lane dual form (contract_lanes) is faster (11,200 atoms: 23 against 320 us) and serves every
// other case, but rounds differently in the last bit: an ensemble's training
// loop in BF16 turns that into 5e-4 of its second step's gradients, by Adam's
// sign-like first step and the operand roundings that it moves, so this path
// keeps its sums.
struct TrainContractLds {
  static constexpr int TA = kRowAtoms, LDGB = kFP + 1;
  static constexpr size_t psi = tf_al(sizeof(Tables));
  static constexpr size_t psid = psi + tf_al(4 * (size_t)TA * PS);
  static constexpr size_t ptmp = psid + tf_al(4 * (size_t)TA * PS);
  static constexpr size_t inter = ptmp + tf_al(4 * (size_t)TA * PS);
  static constexpr size_t gb = inter + tf_al(4 * (size_t)TA * IS);     // [16][LDGB]: Gbar, Gdbar
  static constexpr size_t pba = gb + tf_al(4 * (size_t)16 * LDGB);     // Psibar accumulator, two halves
  static constexpr size_t pbs = pba + tf_al(4 * 2 * (size_t)TA * PS);  // one backward's gradient, two halves
  static constexpr size_t step = pbs + tf_al(4 * 2 * (size_t)TA * PS);
  static constexpr size_t bytes = step + tf_al(4 * (size_t)TA);
};
__global__ void __launch_bounds__(kTrainThreads)
    train_contract(int n_atoms, const float* __restrict__ psi, const float* __restrict__ psidot,
                   const float* __restrict__ gbar, const float* __restrict__ gdbar, float* __restrict__ psibar,
                   float* __restrict__ psidotbar) {
  using L = TrainContractLds;
  constexpr int TA = L::TA, NT = kTrainThreads, NP = kS * kPacked;
  constexpr int KSA = 2 * ((TA * 30 + 63) / 64 * 64) <= NT ? 2 : 1, KSF = 2 * ((TA * 20 + 63) / 64 * 64) <= NT ? 2 : 1;
  static_assert(TA * 29 * 2 <= NT && TA <= kTrainWaves, "threads for both halves of every task");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  Tables& tb = *(Tables*)lds;
  float* sPsi = (float*)(lds + L::psi);
  float* sPd = (float*)(lds + L::psid);
  float* sPt = (float*)(lds + L::ptmp);
  float* sI = (float*)(lds + L::inter);
  float* sGb = (float*)(lds + L::gb);
  float* sPbA = (float*)(lds + L::pba);
  float* sPbA2 = sPbA + TA * PS;
  float* sPbS = (float*)(lds + L::pbs);
  float* sPbS2 = sPbS + TA * PS;
  float* sT = (float*)(lds + L::step);
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * TA;
  const int n_rows = min(TA, n_atoms - row0);
  load_tables(&tb);
  for (int t = tid; t < 16 * kFP; t += NT) {
    const int a = t % TA, f = t / TA % kFP, h = t / (TA * kFP);
    sGb[(h * TA + a) * L::LDGB + f] = a < n_rows ? (h ? gdbar : gbar)[dg_index(n_atoms, row0 + a, f)] : 0.0f;
  }
  __syncthreads();
  for (int t = tid; t < TA * NP; t += NT) {
    const int a = t / NP, e = t % NP, s = e / kPacked, c = e % kPacked;
    const bool ok = a < n_rows;
    const float v = ok ? psi[(int64_t)row0 * NP + t] : 0.0f, vd = ok ? psidot[(int64_t)row0 * NP + t] : 0.0f;
    for (int q = 0; q < tb.packed_mult[c]; ++q) {
      sPsi[a * PS + s * kFull + tb.packed_full[c][q]] = v;
      sPd[a * PS + s * kFull + tb.packed_full[c][q]] = vd;
    }
  }
  __syncthreads();
  if (w < TA) {
    float n0 = 0.0f, n1 = 0.0f;
    for (int e = l; e < kS * kFull; e += 64) {
      n0 += sPsi[w * PS + e] * sPsi[w * PS + e];
      n1 += sPd[w * PS + e] * sPd[w * PS + e];
    }
    n0 = wave_sum(n0);
    n1 = wave_sum(n1);
    if (l == 0) sT[w] = (n1 > 0.0f && n0 > 0.0f) ? sqrtf(n0 / n1) : 1.0f;
  }
  const float* Gbar = sGb;
  const float* Gdbar = sGb + TA * L::LDGB;
  // B(P; G) into pb and its second halves; with_inter: the intermediates of P first
  auto backward = [&](const float* P, const float* G, float* pb, float* pb2, bool with_inter) {
    if (with_inter) {
      contract_forward_a<TA, NT, false, false, IS, KSF>(P, sI, nullptr, 0, tb);
      __syncthreads();
    }
    contract_backward_a<TA, NT, KSA>(P, G, L::LDGB, sI, tb);
    __syncthreads();
    contract_backward_b<TA, NT, 2>(P, G, L::LDGB, sI, pb, tb, pb2);
    __syncthreads();
  };
  backward(sPsi, Gdbar, sPbS, sPbS2, true);
  auto to_psidotbar = [&](int a, int e, float v) {
    if (a < n_rows) psidotbar[(int64_t)(row0 + a) * NP + e] = v;
  };
  fold_packed<TA, NT, decltype(to_psidotbar), true>(sPbS, tb, to_psidotbar, sPbS2);
  backward(sPsi, Gbar, sPbA, sPbA2, false);
  for (int ev = 0; ev < 2; ++ev) {
    const float sgn = ev == 0 ? 1.0f : -1.0f;
    for (int t = tid; t < TA * kS * kFull; t += NT) {
      const int a = t % TA, e = t / TA;
      sPt[a * PS + e] = sPsi[a * PS + e] + sgn * sT[a] * sPd[a * PS + e];
    }
    __syncthreads();
    backward(sPt, Gdbar, sPbS, sPbS2, true);
    for (int t = tid; t < TA * kS * kFull; t += NT) {
      const int a = t % TA, e = t / TA;
      const float d = sPbS[a * PS + e] + sPbS2[a * PS + e];
      sPbA[a * PS + e] += sgn * d / (2.0f * sT[a]);
    }
    __syncthreads();
  }
  auto to_psibar = [&](int a, int e, float v) {
    if (a < n_rows) psibar[(int64_t)(row0 + a) * NP + e] = v;
  };
  fold_packed<TA, NT, decltype(to_psibar), true>(sPbA, tb, to_psibar, sPbA2);
}

// ---------------------------------------------------------------------------
// dPhi/dbeta per pair:
//   c [ f_c g_k (A_s + B_s) + (f_c g_k)' (u.delta) Adot_s ]
// with A_s = Psibar_s . mono(u), Adot_s = Psidotbar_s . mono(u),
// B_s = Psidotbar_s . Dmono(u)[delta_perp / r].  The 35 values of a pair go to
// its (Z_i, Z_j) slot: for each Z_j the wave reduce-scatters the masked
// values, lane k owning slot k, and adds them to the wave's LDS copy of the
// gradient (one writer per slot); per-block copies are summed in wave order
// and written as block partials.
// Blocks of up to 16 waves (four per SIMD hide the per-atom memory round
// trips), as many as the per-wave LDS copies of the gradient allow.
constexpr int kBetaMaxThreads = 1024;
template <int BASIS>
__global__ void __launch_bounds__(kBetaMaxThreads) pair_beta_grad(DevModel m, DevSystem sys, const float* __restrict__ lambda,
                                                             const float* __restrict__ psibar,
                                                             const float* __restrict__ psidotbar,
                                                             float* __restrict__ beta_partial) {
  extern __shared__ float sm[];
  const int nsp = m.n_species;
  const int nslots = nsp * nsp * kS * kMaxBasis;
  float* s_beta = sm;
  float* s_acc = sm + nslots;  // [waves][nslots]
  const int NW = (int)blockDim.x / 64;
  stage_beta(m, s_beta);
  for (int t = threadIdx.x; t < NW * nslots; t += blockDim.x) s_acc[t] = 0.0f;
  __syncthreads();
  const int w = threadIdx.x >> 6, q = threadIdx.x & 63;
  for (int i = blockIdx.x * NW + w; i < sys.n_atoms; i += gridDim.x * NW) {
    AtomCtx c;
    load_atom(sys, i, c);
    const float* bzi = s_beta + c.zsp * nsp * kS * kMaxBasis;
    const float lix = lambda[3 * (int64_t)i], liy = lambda[3 * (int64_t)i + 1], liz = lambda[3 * (int64_t)i + 2];
    for (int64_t p0 = c.p0; p0 < c.p1; p0 += 64) {
      const int64_t p = p0 + q;
      float val[kS * kMaxBasis];
#pragma unroll
      for (int k = 0; k < kS * kMaxBasis; ++k) val[k] = 0.0f;
      int zj = -1;
      if (p < c.p1) {
        int j;
        float dx, dy, dz;
        pair_vec(sys, c, p, j, dx, dy, dz);
        const float r2 = dx * dx + dy * dy + dz * dz;
        if (r2 < m.rc2 && r2 > 0.0f) {
          zj = sys.species[j];
          float r, ir;
          length_of(r2, r, ir);
          const float ux = dx * ir, uy = dy * ir, uz = dz * ir;
          const float ex = lambda[3 * (int64_t)j] - lix, ey = lambda[3 * (int64_t)j + 1] - liy,
                      ez = lambda[3 * (int64_t)j + 2] - liz;
          const float ud = ux * ex + uy * ey + uz * ez;
          float mo[20], dm[20];
          monomials(ux, uy, uz, mo);
          dmonomials(ux, uy, uz, (ex - ud * ux) * ir, (ey - ud * uy) * ir, (ez - ud * uz) * ir, dm);
          // basis: g_k and (f_c g_k)'
          float sn, cs;
          cutoff_cos_sin(m, r, cs, sn);

          const float fc = 0.5f * (cs + 1.0f) * m.psi_scale;
          const float dfc = -0.5f * (3.14159265358979f / m.r_cut) * sn * m.psi_scale;
          const float* pb = psibar + (int64_t)i * (kS * kPacked);
          const float* pd = psidotbar + (int64_t)i * (kS * kPacked);
          const BasisIter<BASIS> b0(m, r, cs, sn);
#pragma unroll
          for (int s = 0; s < kS; ++s) {
            float A = 0.0f, Ad = 0.0f, Bs = 0.0f;
#pragma unroll
            for (int t = 0; t < kPacked; ++t) {
              A += pb[s * kPacked + t] * mo[t];
              Ad += pd[s * kPacked + t] * mo[t];
              Bs += pd[s * kPacked + t] * dm[t];
            }
            BasisIter<BASIS> bi = b0;
#pragma unroll
            for (int k = 0; k < kMaxBasis; ++k) {
              float gk, dgk;
              bi.next(m, k, gk, dgk);
              val[s * kMaxBasis + k] = fc * gk * (A + Bs) + (dfc * gk + fc * dgk) * ud * Ad;
            }
          }
        }
      }
      for (int z = 0; z < nsp; ++z) {
        float vz[64];
#pragma unroll
        for (int k = 0; k < 64; ++k) vz[k] = (k < kS * kMaxBasis && zj == z) ? val[k < kS * kMaxBasis ? k : 0] : 0.0f;
        // 64 values over 64 lanes: lane q ends with slot q
        rs_swap<32, 32>(vz);
        rs_swap<16, 16>(vz);
        rs_step<8, 0>(vz, (q >> 3) & 1);
        rs_step<4, 1>(vz, (q >> 2) & 1);
        rs_step<2, 2>(vz, (q >> 1) & 1);
        rs_step<1, 3>(vz, q & 1);
        if (q < kS * kMaxBasis) s_acc[w * nslots + (c.zsp * nsp + z) * kS * kMaxBasis + q] += vz[0];
      }
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nslots; t += blockDim.x) {
    float v = 0.0f;
    for (int ww = 0; ww < NW; ++ww) v += s_acc[ww * nslots + t];
    beta_partial[(int64_t)blockIdx.x * nslots + t] = v;
  }
}

// ---------------------------------------------------------------------------
// Gradient of Phi in the positions (the loss's dL/dx, Section 3.3).  Phi
// depends on the pair vectors d_p through Psi_i (adjoint Psibar_i) and
// through Psidot_i = sum_p dPsi_i/dd_p . delta_p (adjoint Psidotbar_i), so
//   dPhi/dd_p = grad phi_{Psibar}(d_p) + D_delta grad phi_{Psidotbar}(d_p),
// phi_w(d) = sum_s R_s(|d|) sum_t w[s][t] mono_t(d/|d|) being the pair's
// moment contribution contracted with w.  The first term is the pair
// backward of the energy; the second, a Hessian-vector product, is the
// same gradient evaluated in dual numbers (value, derivative along
// delta_p), which needs R_s'' besides R_s and R_s'.  The positions' gradient
// then gathers these over the reverse index like the forces.
// R_s, dR_s/dr and d^2R_s/dr^2 (the basis and cutoff of radial<true>):
//   Gaussians    g_k'' = (4 gamma^2 (r - mu_k)^2 - 2 gamma) g_k
//   Bessel-like  d^2/dr^2 sinc(k x) = -(k pi / r_c)^2 sinc(k x) - 2 (cos(k x) - sinc(k x)) / r^2
//   cutoff       f_c'' = -(pi / r_c)^2 cos(pi r / r_c) / 2
template <int BASIS>
__device__ inline void radial2(const DevModel& m, const float* __restrict__ bz, float r, float (&R)[kS],
                               float (&dR)[kS], float (&d2R)[kS]) {
  float sn, cs;
  cutoff_cos_sin(m, r, cs, sn);
  const float w = 3.14159265358979f / m.r_cut;
  const float fc = 0.5f * (cs + 1.0f) * m.psi_scale;
  const float dfc = -0.5f * w * sn * m.psi_scale;
  const float d2fc = -0.5f * w * w * cs * m.psi_scale;
  float g[kMaxBasis], dg[kMaxBasis], d2g[kMaxBasis];
  if (BASIS == GMNN_BASIS_BESSEL) {
    const float ir = 1.0f / r;
    const float ix = m.rc_over_pi * ir;
    float sa = sn, ca = cs;
    float sb = 2.0f * cs * sn, cb = 2.0f * cs * cs - 1.0f;
    float sinc_a = sa * ix;
#pragma unroll
    for (int n = 0; n < kMaxBasis; ++n) {
      const float ka = (float)(n + 1) * w, kb = (float)(n + 2) * w;
      const float sinc_b = sb * ix * (1.0f / (float)(n + 2));
      g[n] = m.ck[n] * (sinc_a + sinc_b);
      dg[n] = m.ck[n] * ((ca - sinc_a) + (cb - sinc_b)) * ir;
      d2g[n] = m.ck[n] * (-(ka * ka) * sinc_a - (kb * kb) * sinc_b - 2.0f * ((ca - sinc_a) + (cb - sinc_b)) * ir * ir);
      const float sc = 2.0f * cs * sb - sa, cc = 2.0f * cs * cb - ca;
      sa = sb; ca = cb; sb = sc; cb = cc;
      sinc_a = sinc_b;
    }
  } else {
    const float tau = r - m.r_min;
    const float g0 = __expf(-m.gamma * tau * tau);
    const float a = __expf(2.0f * m.gamma * m.delta * tau);
    float p = g0;
#pragma unroll
    for (int k = 0; k < kMaxBasis; ++k) {
      const float e = tau - (float)k * m.delta;  // r - mu_k
      g[k] = p * m.ck[k];
      dg[k] = -2.0f * m.gamma * e * g[k];
      d2g[k] = (4.0f * m.gamma * m.gamma * e * e - 2.0f * m.gamma) * g[k];
      p *= a;
    }
  }
#pragma unroll
  for (int s = 0; s < kS; ++s) {
    float B = 0.0f, dB = 0.0f, d2B = 0.0f;
#pragma unroll
    for (int k = 0; k < kMaxBasis; ++k) {
      const float bk = bz[s * kMaxBasis + k];
      B += bk * g[k];
      dB += bk * dg[k];
      d2B += bk * d2g[k];
    }
    R[s] = fc * B;
    dR[s] = dfc * B + fc * dB;
    d2R[s] = d2fc * B + 2.0f * dfc * dB + fc * d2B;
  }
}

// grad phi_w at the pair in dual numbers: pair_gradient's formula,
//   g = (sum_s dR_s P_s(u)) u + (grad Q - (grad Q . u) u) / r,
// with u, 1/r, R_s, dR_s carrying their derivatives along delta
__device__ inline void pair_gradient_dual(const float* __restrict__ w, const Dual (&R)[kS], const Dual (&dR)[kS],
                                          Dual x, Dual y, Dual z, Dual ir, Dual& gx, Dual& gy, Dual& gz) {
  Dual mo[kPacked];
  mo[0] = {1.0f, 0.0f};
  mo[1] = x; mo[2] = y; mo[3] = z;
  mo[4] = x * x; mo[5] = x * y; mo[6] = x * z; mo[7] = y * y; mo[8] = y * z; mo[9] = z * z;
  mo[10] = mo[4] * x; mo[11] = mo[4] * y; mo[12] = mo[4] * z; mo[13] = mo[7] * x; mo[14] = mo[5] * z;
  mo[15] = mo[9] * x; mo[16] = mo[7] * y; mo[17] = mo[7] * z; mo[18] = mo[9] * y; mo[19] = mo[9] * z;
  Dual radial_part = {0.0f, 0.0f};
  Dual qc[kPacked];
#pragma unroll
  for (int t = 0; t < kPacked; ++t) qc[t] = {0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < kS; ++s) {
    Dual A = {0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < kPacked; ++t) {
      A += w[s * kPacked + t] * mo[t];
      qc[t] += R[s] * w[s * kPacked + t];
    }
    radial_part += A * dR[s];
  }
  const Dual Gx = qc[1] + 2.0f * qc[4] * x + qc[5] * y + qc[6] * z + 3.0f * qc[10] * x * x + 2.0f * qc[11] * x * y +
                  2.0f * qc[12] * x * z + qc[13] * y * y + qc[14] * y * z + qc[15] * z * z;
  const Dual Gy = qc[2] + qc[5] * x + 2.0f * qc[7] * y + qc[8] * z + qc[11] * x * x + 2.0f * qc[13] * x * y +
                  qc[14] * x * z + 3.0f * qc[16] * y * y + 2.0f * qc[17] * y * z + qc[18] * z * z;
  const Dual Gz = qc[3] + qc[6] * x + qc[8] * y + 2.0f * qc[9] * z + qc[12] * x * x + qc[14] * x * y +
                  2.0f * qc[15] * x * z + qc[17] * y * y + 2.0f * qc[18] * y * z + 3.0f * qc[19] * z * z;
  const Dual gu = Gx * x + Gy * y + Gz * z;
  gx = radial_part * x + (Gx - gu * x) * ir;
  gy = radial_part * y + (Gy - gu * y) * ir;
  gz = radial_part * z + (Gz - gu * z) * ir;
}

constexpr int kPosLanes = 64;  // lanes per atom row of the position-gradient kernels

// dPhi/dd_p for every pair (gpos [P][3]); one 64-lane group per atom
template <int BASIS>
__global__ void __launch_bounds__(kPairBlock) pair_pos_grad(DevModel m, DevSystem sys, const float* __restrict__ lambda,
                                                            const float* __restrict__ psibar,
                                                            const float* __restrict__ psidotbar,
                                                            float* __restrict__ gpos) {
  extern __shared__ float s_beta[];
  stage_beta(m, s_beta);
  __syncthreads();
  const int q = threadIdx.x & (kPosLanes - 1);
  const int i = blockIdx.x * (kPairBlock / kPosLanes) + threadIdx.x / kPosLanes;
  if (i >= sys.n_atoms) return;
  AtomCtx c;
  load_atom(sys, i, c);
  const float* bzi = s_beta + c.zsp * m.n_species * kS * kMaxBasis;
  const float* pb = psibar + (int64_t)i * (kS * kPacked);
  const float* pd = psidotbar + (int64_t)i * (kS * kPacked);
  const float lix = lambda[3 * (int64_t)i], liy = lambda[3 * (int64_t)i + 1], liz = lambda[3 * (int64_t)i + 2];
  for (int64_t p = c.p0 + q; p < c.p1; p += kPosLanes) {
    int j;
    float dx, dy, dz;
    pair_vec(sys, c, p, j, dx, dy, dz);
    const float r2 = dx * dx + dy * dy + dz * dz;
    float gx = 0.0f, gy = 0.0f, gz = 0.0f;
    if (r2 < m.rc2 && r2 > 0.0f) {
      float r, ir;
      length_of(r2, r, ir);
      const float ux = dx * ir, uy = dy * ir, uz = dz * ir;
      const float* bz = bzi + sys.species[j] * kS * kMaxBasis;
      // the energy's pair gradient with Psibar
      Radial rad;
      radial<true>(m, bz, r, rad);
      float mo[20];
      monomials(ux, uy, uz, mo);
      pair_gradient(pb, rad, mo, ux, uy, uz, ir, gx, gy, gz);
      // its derivative along delta_p with Psidotbar
      const float ex = lambda[3 * (int64_t)j] - lix, ey = lambda[3 * (int64_t)j + 1] - liy,
                  ez = lambda[3 * (int64_t)j + 2] - liz;
      const float rdot = ux * ex + uy * ey + uz * ez;  // d|d|/dt
      float R[kS], dR[kS], d2R[kS];
      radial2<BASIS>(m, bz, r, R, dR, d2R);
      Dual Rd[kS], dRd[kS];
#pragma unroll
      for (int s = 0; s < kS; ++s) {
        Rd[s] = {R[s], dR[s] * rdot};
        dRd[s] = {dR[s], d2R[s] * rdot};
      }
      const Dual xd = {ux, (ex - ux * rdot) * ir}, yd = {uy, (ey - uy * rdot) * ir}, zd = {uz, (ez - uz * rdot) * ir};
      const Dual ird = {ir, -rdot * ir * ir};
      Dual hx, hy, hz;
      pair_gradient_dual(pd, Rd, dRd, xd, yd, zd, ird, hx, hy, hz);
      gx += hx.t;
      gy += hy.t;
      gz += hz.t;
    }
    gpos[3 * p] = gx;
    gpos[3 * p + 1] = gy;
    gpos[3 * p + 2] = gz;
  }
}

// dL/dx_i = sum over the row of (gpos[rev p] - gpos[p]) (added to dL_dpos
// with accumulate, for the per-head sum)
__global__ void __launch_bounds__(kPairBlock) pos_gather(DevSystem sys, const float* __restrict__ gpos,
                                                         float* __restrict__ dL_dpos, int accumulate) {
  const int q = threadIdx.x & (kPosLanes - 1);
  const int i = blockIdx.x * (kPairBlock / kPosLanes) + threadIdx.x / kPosLanes;
  const bool live = i < sys.n_atoms;
  float f[3] = {0.0f, 0.0f, 0.0f};
  if (live) {
    const int64_t p0 = sys.row_ptr[i], p1 = sys.row_ptr[i + 1];
    for (int64_t p = p0 + q; p < p1; p += kPosLanes) {
      const int64_t rp = sys.rev[p];
      f[0] += gpos[3 * rp] - gpos[3 * p];
      f[1] += gpos[3 * rp + 1] - gpos[3 * p + 1];
      f[2] += gpos[3 * rp + 2] - gpos[3 * p + 2];
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) f[k] = atom_sum<kPosLanes>(f[k]);
  if (live && q == 0)
#pragma unroll
    for (int k = 0; k < 3; ++k)
      dL_dpos[3 * (int64_t)i + k] = accumulate ? dL_dpos[3 * (int64_t)i + k] + f[k] : f[k];
}

// ---------------------------------------------------------------------------
// C[M][N] = sum_k A[k][M]^T B[k][N] over the rows k of chunk blockIdx.y
// (split-K; partial[chunk][M][N]), every FP32 operand taken in NP bf16 parts
// on BF16 MFMA 16x16x32 with FP32 accumulation:
//   NP = 2 (the BF16 network): hi.hi + hi.lo + lo.hi, about 16 significant
//          bits per product (the dropped lo.lo is below 2^-16 of |a b|);
//   NP = 3 (the FP32 network): the six products of mfma.h's FP32 form.
// Each wave owns a 64 x 64 block of C as 4 x 4 MFMA tiles, so every value
// loaded feeds twelve (24) MFMAs.  M and N are multiples of 64.
constexpr int kWgRows = 1024;    // rows per split-K chunk
constexpr int kWgRowsMin = 256;  // fewest rows per chunk of the FP32 network's staged products

// acc[c] += the NP-part products of one A fragment with four B fragments; NP =
// 3: A carries the k-step's sign (step_sign), which the sum takes out again
template <int NP>
__device__ __forceinline__ void mma_parts(const bf16x8 (&a)[NP], const bf16x8 (&b)[4][NP], float sign,
                                          floatx4 (&acc)[4]) {
  if constexpr (NP == 3) {
    const Split3 x{a[0], a[1], a[2]};
    floatx4 t[4];
    six_products(t, [&](int) -> const Split3& { return x; },
                             [&](int c) { return Split3{b[c][0], b[c][1], b[c][2]}; });
#pragma unroll
    for (int c = 0; c < 4; ++c) add_step(acc[c], t[c], sign);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[c][0], acc[c], 0, 0, 0);
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[c][1], acc[c], 0, 0, 0);
      acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[c][0], acc[c], 0, 0, 0);
    }
  }
}
// the NP parts of eight loaded values as fragments
template <int NP>
__device__ __forceinline__ void put_parts(const float (&v)[8], float sign, bf16x8 (&o)[NP]) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    bf16x2 p[3];
    if constexpr (NP == 3) {
      split3_pair(sign * v[e], sign * v[e + 1], p[0], p[1], p[2]);
    } else {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        p[0][d] = (__bf16)v[e + d];
        p[1][d] = (__bf16)(v[e + d] - (float)p[0][d]);
      }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      o[q][e] = p[q][0];
      o[q][e + 1] = p[q][1];
    }
  }
}

// Both layers' products in one launch: M x HP with M = kFP, then M = HP, so
// that one's last blocks fill up with the other's.
struct WeightProducts {
  const float *A[2], *B[2];  // [K][M], [K][HP]
  float* partial[2];
  int HP;
  int64_t K, kchunk;
};

template <int NP>
__global__ void __launch_bounds__(256) weight_grad(WeightProducts g) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int Ndim = g.HP, tiles_n = Ndim / 64, tiles1 = kFP / 64 * tiles_n;
  int tile = blockIdx.x * 4 + w;
  const bool second = tile >= tiles1;
  if (second) tile -= tiles1;
  const int Mdim = second ? g.HP : kFP;
  if (tile >= (Mdim / 64) * tiles_n) return;
  const float *A = g.A[second], *B = g.B[second];
  float* partial = g.partial[second];
  const int ldA = Mdim, ldB = Ndim;
  const int64_t K = g.K, kchunk = g.kchunk;
  const int m0 = (tile / tiles_n) * 64, n0 = (tile % tiles_n) * 64;
  const int64_t kb = (int64_t)blockIdx.y * kchunk;
  const int64_t ke = min(K, kb + kchunk);
  floatx4 acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  const float* ap = A + m0 + (l & 15);
  const float* bp = B + n0 + (l & 15);
  // lane l supplies A^T[m = l&15][k = 8 (l>>4) + e] and B[k = 8 (l>>4) + e][n = l&15], e < 8
  for (int64_t k = kb; k < ke; k += 32) {
    float a[4][8], b[4][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t kk = k + 8 * (l >> 4) + e;
      const bool ok = kk < ke;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        a[r][e] = ok ? ap[kk * ldA + r * 16] : 0.0f;
        b[r][e] = ok ? bp[kk * ldB + r * 16] : 0.0f;
      }
    }
    const float sign = step_sign((int)((k - kb) / 32));
    bf16x8 bs[4][NP];
#pragma unroll
    for (int c = 0; c < 4; ++c) put_parts<NP>(b[c], 1.0f, bs[c]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bf16x8 as[NP];
      put_parts<NP>(a[r], sign, as);
      mma_parts<NP>(as, bs, sign, acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = m0 + r * 16 + 4 * (l >> 4) + j, col = n0 + c * 16 + (l & 15);
        partial[((int64_t)blockIdx.y * Mdim + row) * Ndim + col] = acc[r][c][j];
      }
}

// The same products for M and N multiples of 128, with the operand rows
// staged through LDS: a block of 4 waves owns a 128 x 128 block of C (2 x 2
// waves of 64 x 64).  Per k-step of 32 rows every thread loads 16 rows of one
// column of A and of B, splits them once for the whole block, and writes them
// to LDS as k-contiguous runs of each part; the next k-step's loads are
// issued before the current step's MFMAs.
constexpr int kWgBlk = 128;  // block tile edge
constexpr int kWgLdk = 40;   // LDS row stride in bf16 (32 k + 8 pad)
template <int NP>
__global__ void __launch_bounds__(256) weight_grad_staged(WeightProducts g) {
  // [A parts, B parts][column][k]
  __shared__ __attribute__((aligned(16))) __bf16 sm[2 * NP][kWgBlk * kWgLdk];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int Ndim = g.HP, tiles_n = Ndim / kWgBlk, tiles1 = kFP / kWgBlk * tiles_n;
  const bool second = (int)blockIdx.x >= tiles1;
  const int tile = blockIdx.x - (second ? tiles1 : 0);
  const int Mdim = second ? g.HP : kFP;
  const float *A = g.A[second], *B = g.B[second];
  float* partial = g.partial[second];
  const int ldA = Mdim, ldB = Ndim;
  const int64_t K = g.K, kchunk = g.kchunk;
  const int mb = (tile / tiles_n) * kWgBlk, nb = (tile % tiles_n) * kWgBlk;
  const int m0 = (w >> 1) * 64, n0 = (w & 1) * 64;  // the wave's block inside the block tile
  const int64_t kb = (int64_t)blockIdx.y * kchunk;
  const int64_t ke = min(K, kb + kchunk);
  floatx4 acc[4][4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[r][c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  // staging: thread tid loads rows 16 h .. 16 h + 15 of column col of the step
  const int col = tid & (kWgBlk - 1), h = tid >> 7;
  const float* ap = A + mb + col;
  const float* bp = B + nb + col;
  float ra[2][8], rb[2][8];
  auto fetch = [&](int64_t k) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int64_t kk = k + 16 * h + e;
      const bool ok = kk < ke;
      ra[e / 8][e % 8] = ok ? ap[kk * ldA] : 0.0f;
      rb[e / 8][e % 8] = ok ? bp[kk * ldB] : 0.0f;
    }
  };
  if (kb < ke) fetch(kb);
  for (int64_t k = kb; k < ke; k += 32) {
    const float sign = step_sign((int)((k - kb) / 32));
    __syncthreads();  // the previous step's fragment reads are done
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      bf16x8 a[NP], b[NP];
      put_parts<NP>(ra[half], sign, a);
      put_parts<NP>(rb[half], 1.0f, b);
      const int o = col * kWgLdk + 16 * h + 8 * half;
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        *(bf16x8*)&sm[q][o] = a[q];
        *(bf16x8*)&sm[NP + q][o] = b[q];
      }
    }
    __syncthreads();
    if (k + 32 < ke) fetch(k + 32);
    // lane l supplies A^T[m = l&15][k = 8 (l>>4) + e] and B[k = 8 (l>>4) + e][n = l&15]
    bf16x8 b[4][NP];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int o = (n0 + 16 * c + (l & 15)) * kWgLdk + 8 * (l >> 4);
#pragma unroll
      for (int q = 0; q < NP; ++q) b[c][q] = *(const bf16x8*)&sm[NP + q][o];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = (m0 + 16 * r + (l & 15)) * kWgLdk + 8 * (l >> 4);
      bf16x8 a[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) a[q] = *(const bf16x8*)&sm[q][o];
      mma_parts<NP>(a, b, sign, acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = mb + m0 + r * 16 + 4 * (l >> 4) + j, cc = nb + n0 + c * 16 + (l & 15);
        partial[((int64_t)blockIdx.y * Mdim + row) * Ndim + cc] = acc[r][c][j];
      }
}

// sum_c partial[c][i], chunks in order (eight loads in flight)
__device__ inline float sum_chunks(const float* __restrict__ partial, int nchunks, int64_t n, int64_t i) {
  float v = 0.0f;
  int c = 0;
  for (; c + 8 <= nchunks; c += 8) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = partial[(int64_t)(c + u) * n + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) v += x[u];
  }
  for (; c < nchunks; ++c) v += partial[(int64_t)c * n + i];
  return v;
}

// Sums over atoms, stage 1, in one launch: the bias gradients (columns of the
// primal rows of Y1 and Y2), the W3 gradient (columns of w3g), and per species
// the sums of qsig and of the energies' weights.
//   blocks [0, 3 nx ny): array b / (nx ny), 64 columns x one chunk of rows
//     (primal: of the weight products' rows, those with (k & 15) < 8); 4 row
//     lanes take rows r, r + 4, ... of the chunk, added in lane order:
//     part[array][chunk][column]
//   blocks beyond: species_partials' chunk of 256 atoms
constexpr int kColChunks = 128;  // at most this many row chunks
struct ColumnSums {
  const float* src[3];
  int ncols[3], chunks[3];
  bool primal[3];
  int64_t nrows[3], rows_per_chunk[3];
};
__device__ inline void column_partials(const float* __restrict__ Y, int ld, int64_t nrows, int64_t rows_per_chunk,
                                       bool primal, int ncols, int bx, int chunk, float* __restrict__ partial,
                                       float (*red)[64]) {
  const int cl = threadIdx.x & 63, r = threadIdx.x >> 6;
  const int c = bx * 64 + cl;
  const int64_t k0 = (int64_t)chunk * rows_per_chunk;
  const int64_t k1 = min(nrows, k0 + rows_per_chunk);
  float v = 0.0f;
  if (c < ncols) {
    int64_t k = k0 + r;
    for (; k + 28 < k1; k += 32) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t kk = k + 4 * u;
        x[u] = !primal || (kk & 15) < kRowAtoms ? Y[kk * ld + c] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v += x[u];
    }
    for (; k < k1; k += 4)
      if (!primal || (k & 15) < kRowAtoms) v += Y[k * ld + c];
  }
  red[r][cl] = v;
  __syncthreads();
  if (r == 0 && c < ncols) partial[(int64_t)chunk * ncols + c] = ((red[0][cl] + red[1][cl]) + red[2][cl]) + red[3][cl];
}

// per-species sums: chunk b takes atoms [b*256, b*256+256) and writes, in
// FP64, sp[b][z][0] = sum qsig_i and sp[b][z][1] = sum ebar_b(i) over its
// atoms of species z, and sp[b][nsp][0] = sum ebar_b(i) sigma_z(i)
// (fixed-shape tree sums: the result does not depend on scheduling)
constexpr int kSpeciesChunk = 256;
__device__ inline void species_partials(const DevModel& m, const DevSystem& sys, const double* __restrict__ ebar,
                                        const float* __restrict__ qsig, int b, double* __restrict__ sp,
                                        double (*red)[kMaxSpecies + 1][2]) {
  const int i = b * kSpeciesChunk + threadIdx.x;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  int z = -1;
  double q = 0.0, e = 0.0;
  if (i < sys.n_atoms) {
    z = sys.species[i];
    q = (double)qsig[i];
    e = ebar[sys.atom_struct[i]];
  }
  const int nsp = m.n_species;
  for (int t = 0; t < nsp; ++t) {
    const double x = wave_sum(z == t ? q : 0.0);
    const double y = wave_sum(z == t ? e : 0.0);
    if (l == 0) {
      red[w][t][0] = x;
      red[w][t][1] = y;
    }
  }
  const double c = wave_sum(z >= 0 ? e * (double)m.scale[z] : 0.0);
  if (l == 0) red[w][nsp][0] = c;
  __syncthreads();
  if (threadIdx.x < 2 * (nsp + 1)) {
    const int t = threadIdx.x >> 1, k = threadIdx.x & 1;
    double v = 0.0;
    for (int ww = 0; ww < kSpeciesChunk / 64; ++ww) v += (t < nsp || k == 0) ? red[ww][t][k] : 0.0;
    sp[((int64_t)b * (kMaxSpecies + 1) + t) * 2 + k] = v;
  }
}

__global__ void __launch_bounds__(kSpeciesChunk)
    train_partials(DevModel m, DevSystem sys, const double* __restrict__ ebar, const float* __restrict__ qsig,
                   ColumnSums cols, int nx, int ny, float* __restrict__ part, int64_t part_stride,
                   double* __restrict__ sp) {
  __shared__ double smem[kSpeciesChunk / 64][kMaxSpecies + 1][2];
  static_assert(sizeof(smem) >= sizeof(float) * 4 * 64, "the column sums' four rows fit");
  const int b = blockIdx.x;
  if (b < 3 * nx * ny) {
    const int k = b / (nx * ny), t = b % (nx * ny);
    if (t / nx >= cols.chunks[k]) return;
    column_partials(cols.src[k], m.HP1, cols.nrows[k], cols.rows_per_chunk[k], cols.primal[k], cols.ncols[k], t % nx,
                    t / nx, part + k * part_stride, (float(*)[64])smem);
  } else {
    species_partials(m, sys, ebar, qsig, b - 3 * nx * ny, sp, smem);
  }
}

// Stage 2, in one launch: every gradient from its partials, added in chunk
// order, into the caller's arrays (unpadded).  Per head of a shallow ensemble
// (head >= 0) the shared arrays are summed over the heads in head order and
// W3 and b3 take the head's column; otherwise every head's column of W3 and
// b3 equals the mean's gradient.
struct GradSums {
  const float *part1, *part2, *cpart, *bpart;
  int64_t cstride;  // between the three column-sum arrays in cpart
  const double* sp;
  int kch, cch_k, cch_n, bch, sp_blocks;  // cch_k, cch_n: row chunks of the bias and the W3 sums
  int HP, H1, H2, heads, head;  // heads: columns of W3
};
__global__ void __launch_bounds__(256) train_sums(DevModel m, GradSums g, gmnn_param_grads out) {
  const int nsp = m.n_species, nslots = nsp * nsp * kS * kMaxBasis;
  const bool add = g.head > 0;
  auto store = [&](float* dst, int64_t i, float v) { dst[i] = add ? dst[i] + v : v; };
  int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t n1 = (int64_t)kF * g.H1, n2 = (int64_t)g.H1 * g.H2;
  if (t < n1) {
    store(out.W1, t, sum_chunks(g.part1, g.kch, (int64_t)kFP * g.HP, t / g.H1 * g.HP + t % g.H1));
    return;
  }
  t -= n1;
  if (t < n2) {
    store(out.W2, t, sum_chunks(g.part2, g.kch, (int64_t)g.HP * g.HP, t / g.H2 * g.HP + t % g.H2));
    return;
  }
  t -= n2;
  if (t < g.H1) {
    store(out.b1, t, sum_chunks(g.cpart, g.cch_k, g.H1, t));
    return;
  }
  t -= g.H1;
  if (t < g.H2) {
    store(out.b2, t, sum_chunks(g.cpart + g.cstride, g.cch_k, g.H2, t));
    return;
  }
  t -= g.H2;
  if (t < g.H2) {
    const float v = sum_chunks(g.cpart + 2 * g.cstride, g.cch_n, g.H2, t);
    if (g.head >= 0) out.W3[t * g.heads + g.head] = v;
    else
      for (int h = 0; h < g.heads; ++h) out.W3[t * g.heads + h] = v;
    return;
  }
  t -= g.H2;
  if (t < (int64_t)nsp * nsp * kS * m.K) {
    store(out.beta, t, sum_chunks(g.bpart, g.bch, nslots, t / m.K * kMaxBasis + t % m.K));
    return;
  }
  t -= (int64_t)nsp * nsp * kS * m.K;
  if (t > nsp) return;
  // scale / shift / b3 from the species sums, added in block order; the loads
  // of 8 blocks are issued before their adds so they overlap
  constexpr int kBatch = 8;
  double s1 = 0.0, s2 = 0.0;
  for (int b0 = 0; b0 < g.sp_blocks; b0 += kBatch) {
    double x[kBatch], y[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int64_t o = ((int64_t)std::min(b0 + j, g.sp_blocks - 1) * (kMaxSpecies + 1) + t) * 2;
      x[j] = g.sp[o];
      y[j] = g.sp[o + 1];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      if (b0 + j < g.sp_blocks) {
        s1 += x[j];
        s2 += y[j];
      }
    }
  }
  if (t < nsp) {
    store(out.scale, t, (float)s1);
    store(out.shift, t, (float)s2);
  } else if (g.head >= 0) {
    out.b3[g.head] = (float)s1;
  } else {
    // dPhi/db3_m = sum_i a_i sigma_i / M (the same for every head)
    for (int h = 0; h < g.heads; ++h) out.b3[h] = (float)(s1 / g.heads);
  }
}

// ---------------------------------------------------------------------------
struct TrainLayout {
  size_t psi, psidot, psibar, psidotbar, X1, Y1, X2, Y2, gbar, gdbar, w3g, qsig, part1, part2, bpart;
  size_t cpart, spart, bytes;
  int64_t cstride;     // between the column-sum arrays in cpart
  int ccK, ccN;        // row chunks of the column sums over weight-product rows / over atoms
  int64_t rcK, rcN;    // rows per chunk
  int sp_blocks;       // blocks of the per-species sums
  int64_t K;           // weight-product rows
  int64_t wg_rows;     // rows per split-K chunk
  int kchunks;         // split-K chunks
  int beta_blocks;
};

// Rows per split-K chunk of the FP32 network's staged products: whole rounds
// of the blocks resident at once (two of 61 KB LDS per compute unit), few
// rounds against few chunks, whose partials train_sums reads back (a chunk
// costs about HP / 80 rows of products: 0.7 us at 2x512, where a row of a
// round takes 0.11).  Against 512 rows always: a step of 7 heads at 1838 atoms
// 2x256 1270 -> 1138 us, of 14 heads at 3633 atoms 2907 -> 2756.
static int64_t weight_rows(int64_t K, int HP) {
  const int tiles = (kFP + HP) / kWgBlk * (HP / kWgBlk), resident = 512;
  int64_t best = kWgRows, best_cost = INT64_MAX;
  for (int64_t rows = kWgRowsMin; rows <= kWgRows; rows += 32) {
    const int64_t kch = (K + rows - 1) / rows, rounds = (tiles * kch + resident - 1) / resident;
    const int64_t cost = rounds * rows + kch * HP / 80;
    if (cost < best_cost) {
      best = rows;
      best_cost = cost;
    }
  }
  return best;
}

// widths that are multiples of the staged kernel's block tile take it; BF16
// products and narrower widths keep whole chunks of kWgRows
static int64_t product_rows(int64_t K, int HP, bool bf16) {
  return HP % kWgBlk == 0 && !bf16 ? weight_rows(K, HP) : kWgRows;
}

TrainLayout train_layout(int n_atoms, int HP, int nsp, bool bf16) {
  TrainLayout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  };
  const size_t N = (size_t)n_atoms;
  L.K = ((int64_t)N + kRowAtoms - 1) / kRowAtoms * 16;
  L.wg_rows = product_rows(L.K, HP, bf16);
  L.kchunks = (int)((L.K + L.wg_rows - 1) / L.wg_rows);
  L.beta_blocks = 256;
  L.psi = take(4 * N * 100);
  L.psidot = take(4 * N * 100);
  L.psibar = take(4 * N * 100);
  L.psidotbar = take(4 * N * 100);
  L.X1 = take(4 * (size_t)L.K * kFP);
  L.Y1 = take(4 * (size_t)L.K * HP);
  L.X2 = take(4 * (size_t)L.K * HP);
  L.Y2 = take(4 * (size_t)L.K * HP);
  L.w3g = take(4 * N * HP);
  L.qsig = take(4 * N);
  // the invariants' adjoints are read before the weight products write their
  // partials: one region for both
  const size_t shared = off;
  L.gbar = take(4 * N * kFP);
  L.gdbar = take(4 * N * kFP);
  const size_t adjoints_end = off;
  off = shared;
  L.part1 = take(4 * (size_t)L.kchunks * kFP * HP);
  L.part2 = take(4 * (size_t)L.kchunks * HP * HP);
  off = std::max(off, adjoints_end);
  const size_t nslots = (size_t)nsp * nsp * kS * kMaxBasis;
  L.bpart = take(4 * (size_t)L.beta_blocks * nslots);
  L.rcN = N > 0 ? ((int64_t)N + kColChunks - 1) / kColChunks : 1;
  L.ccN = (int)(((int64_t)N + L.rcN - 1) / L.rcN);
  L.rcK = L.K > 0 ? (L.K + kColChunks - 1) / kColChunks : 1;
  L.ccK = (int)((L.K + L.rcK - 1) / L.rcK);
  L.cstride = (int64_t)HP * std::max(L.ccK, L.ccN);
  L.cpart = take(4 * 3 * (size_t)L.cstride);
  L.sp_blocks = (int)((N + kSpeciesChunk - 1) / kSpeciesChunk);
  L.spart = take(8 * 2 * (size_t)(kMaxSpecies + 1) * (L.sp_blocks > 0 ? L.sp_blocks : 1));
  L.bytes = off;
  return L;
}

template <int LPA>
__global__ void pair_moments(DevModel m, DevSystem sys, float* psi, int* counters, int n_counters);

bool train_supported(const DevModel& m) {
  return m.n_species <= kMaxSpecies && (m.HP1 == 64 || m.HP1 == 128 || m.HP1 == 256 || m.HP1 == 512);
}

size_t train_workspace_bytes(int n_atoms, int HP, int nsp, bool bf16) {
  return train_layout(n_atoms, HP, nsp, bf16).bytes;
}

struct TrainNetArgs {
  const double* ebar;
  const float* X1;
  float *Y1, *X2, *Y2, *w3g, *qsig, *Gbar, *Gdbar;
};
template <int HP, bool BF16, int AB>
static gmnn_status launch_train_network_t(const DevModel& m, const DevSystem& sys, const TrainNetArgs& t,
                                          hipStream_t s) {
  using L = TrainNetLds<HP, BF16, AB>;
  static_assert(L::bytes <= 160 * 1024, "the tile fits the LDS");
  auto k = train_network<HP, BF16, AB>;
  const gmnn_status st = ensure_lds_limit((const void*)k, L::bytes);
  if (st != GMNN_OK) return st;
  hipLaunchKernelGGL(k, dim3((sys.n_atoms + 16 * AB - 1) / (16 * AB)), dim3(kTrainThreads), L::bytes, s, m, sys,
                     t.ebar, t.X1, t.Y1, t.X2, t.Y2, t.w3g, t.qsig, t.Gbar, t.Gdbar);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}
static gmnn_status launch_train_network(const DevModel& m, const DevSystem& sys, bool bf16, const TrainNetArgs& t,
                                        hipStream_t s) {
  // 32-atom tiles (half the weight traffic) once 16-atom ones would need a
  // second round of the 256 compute units, at 2x256.  At 2x512 the FP32 operands
  // of 32 atoms do not fit the LDS (200 KB); narrower networks gain little or
  // lose (a step of 4900 and of 11,200 atoms, 16- against 32-atom tiles: 2x64 FP32
  // 341 and 427 us against 346 and 439, BF16 306 and 396 against 311 and 393;
  // 2x128 303 and 428 against 307 and 413, 304 and 396 against 306 and 396)
  const bool two = sys.n_atoms > 16 * 256;
#define CASE(HP, AB2)                                                                            \
  if (m.HP1 == HP) {                                                                             \
    if (AB2 > 1 && two)                                                                          \
      return bf16 ? launch_train_network_t<HP, true, AB2>(m, sys, t, s)                          \
                  : launch_train_network_t<HP, false, AB2>(m, sys, t, s);                        \
    return bf16 ? launch_train_network_t<HP, true, 1>(m, sys, t, s)                              \
                : launch_train_network_t<HP, false, 1>(m, sys, t, s);                            \
  }
  CASE(64, 1) CASE(128, 1) CASE(256, 2) CASE(512, 1)
#undef CASE
  return GMNN_ERR_UNSUPPORTED;
}

// head < 0: the head-mean gradient.  head >= 0: head `head` of `heads` (m is
// its one-head view): shared gradients summed in head order, W3 and b3 by
// column; the moments and invariants of the first head serve the others.
gmnn_status train_backward(const DevModel& m, const DevSystem& sys, bool bf16, bool lanes16, int H1, int H2,
                           const double* ebar, const float* lambda, gmnn_param_grads* g, void* ws, size_t ws_bytes,
                           float* dL_dpos, float* gpos, int head, int heads, hipStream_t s) {
  const int HP = m.HP1;
  const int nsp = m.n_species;
  const TrainLayout L = train_layout(sys.n_atoms, HP, nsp, bf16);
  if (ws_bytes < L.bytes) return GMNN_ERR_WORKSPACE;
  char* W = (char*)ws;
  float* psi = (float*)(W + L.psi);
  float* psidot = (float*)(W + L.psidot);
  float* psibar = (float*)(W + L.psibar);
  float* psidotbar = (float*)(W + L.psidotbar);
  float *X1 = (float*)(W + L.X1), *Y1 = (float*)(W + L.Y1), *X2 = (float*)(W + L.X2), *Y2 = (float*)(W + L.Y2);
  float *gbar = (float*)(W + L.gbar), *gdbar = (float*)(W + L.gdbar);
  float* w3g = (float*)(W + L.w3g);
  float* qsig = (float*)(W + L.qsig);
  float* part1 = (float*)(W + L.part1);
  float* part2 = (float*)(W + L.part2);
  float* bpart = (float*)(W + L.bpart);
  float* cpart = (float*)(W + L.cpart);
  double* spart = (double*)(W + L.spart);
  const int N = sys.n_atoms;
  const int nslots = nsp * nsp * kS * kMaxBasis;
  const size_t beta_lds = sizeof(float) * (size_t)nslots;
  const int lpa = (N < 8192 && !lanes16) ? 64 : 16;
  const int nb = (N + kPairBlock / lpa - 1) / (kPairBlock / lpa);
  const bool first = head <= 0;
  gmnn_status st = GMNN_OK;
  if (N > 0) {
    if (lpa == 64) {
      if (first)
        hipLaunchKernelGGL(pair_moments<64>, dim3(nb), dim3(kPairBlock), beta_lds, s, m, sys, psi, (int*)nullptr, 0);
      hipLaunchKernelGGL(pair_tangent<64>, dim3(nb), dim3(kPairBlock), beta_lds, s, m, sys, lambda, psidot);
    } else {
      if (first)
        hipLaunchKernelGGL(pair_moments<16>, dim3(nb), dim3(kPairBlock), beta_lds, s, m, sys, psi, (int*)nullptr, 0);
      hipLaunchKernelGGL(pair_tangent<16>, dim3(nb), dim3(kPairBlock), beta_lds, s, m, sys, lambda, psidot);
    }
    auto kf = first ? train_features<true> : train_features<false>;
    st = ensure_lds_limit((const void*)kf, TrainFeatLds::bytes);
    if (st != GMNN_OK) return st;
    hipLaunchKernelGGL(kf, dim3((N + kTfAtoms - 1) / kTfAtoms), dim3(kTfThreads), TrainFeatLds::bytes, s, N, psi,
                       psidot, X1);
    st = launch_train_network(m, sys, bf16, TrainNetArgs{ebar, X1, Y1, X2, Y2, w3g, qsig, gbar, gdbar}, s);
    if (st == GMNN_OK && bf16 && head >= 0) {
      st = ensure_lds_limit((const void*)train_contract, TrainContractLds::bytes);
      if (st == GMNN_OK)
        hipLaunchKernelGGL(train_contract, dim3((N + kRowAtoms - 1) / kRowAtoms), dim3(kTrainThreads),
                           TrainContractLds::bytes, s, N, psi, psidot, gbar, gdbar, psibar, psidotbar);
    } else if (st == GMNN_OK) {
      st = launch_contract_back_dual(N, psi, psidot, gdbar, gbar, psidotbar, psibar, s);
    }
    if (st != GMNN_OK) return st;
  }
  if (dL_dpos && N > 0) {
    // the positions' gradient from the same adjoints as the beta gradient
    const int nbp = (N + kPairBlock / kPosLanes - 1) / (kPairBlock / kPosLanes);
    auto kp = m.basis == GMNN_BASIS_BESSEL ? pair_pos_grad<GMNN_BASIS_BESSEL> : pair_pos_grad<GMNN_BASIS_GAUSSIAN>;
    st = ensure_lds_limit((const void*)kp, beta_lds);
    if (st != GMNN_OK) return st;
    hipLaunchKernelGGL(kp, dim3(nbp), dim3(kPairBlock), beta_lds, s, m, sys, lambda, psibar, psidotbar, gpos);
    hipLaunchKernelGGL(pos_gather, dim3(nbp), dim3(kPairBlock), 0, s, sys, gpos, dL_dpos, first ? 0 : 1);
  }
  // waves per block: the beta table plus one gradient copy per wave in 160 KB
  const int beta_waves = (int)std::min<size_t>(kBetaMaxThreads / 64, std::max<size_t>(1, 160 * 1024 / beta_lds - 1));
  {
    auto kb = m.basis == GMNN_BASIS_BESSEL ? pair_beta_grad<GMNN_BASIS_BESSEL> : pair_beta_grad<GMNN_BASIS_GAUSSIAN>;
    st = ensure_lds_limit((const void*)kb, beta_lds * (1 + beta_waves));
    if (st != GMNN_OK) return st;
    hipLaunchKernelGGL(kb, dim3(L.beta_blocks), dim3(64 * beta_waves), beta_lds * (1 + beta_waves), s, m, sys, lambda,
                       psibar, psidotbar, bpart);
  }
  // weight products, split over chunks of rows, partials summed in chunk order:
  // two parts per operand on the BF16 path, three on the FP32 path
  const bool staged = HP % kWgBlk == 0;
  const int kch = L.kchunks;
  if (kch > 0) {
    const WeightProducts g{{X1, X2}, {Y1, Y2}, {part1, part2}, HP, L.K, L.wg_rows};
    if (staged)
      hipLaunchKernelGGL(bf16 ? weight_grad_staged<2> : weight_grad_staged<3>,
                         dim3((kFP + HP) / kWgBlk * (HP / kWgBlk), kch), dim3(256), 0, s, g);
    else
      hipLaunchKernelGGL(bf16 ? weight_grad<2> : weight_grad<3>, dim3(((kFP + HP) / 64 * (HP / 64) + 3) / 4, kch),
                         dim3(256), 0, s, g);
  }
  // bias, W3, scale/shift partials, then every gradient from its partials
  // (with no atoms there are no chunks: the sums of zero partials are zero)
  if (N > 0) {
    const int nx = (std::max(H1, H2) + 63) / 64, ny = std::max(L.ccK, L.ccN);
    const ColumnSums cols{{Y1, Y2, w3g}, {H1, H2, H2}, {L.ccK, L.ccK, L.ccN}, {true, true, false},
                          {L.K, L.K, N}, {L.rcK, L.rcK, L.rcN}};
    hipLaunchKernelGGL(train_partials, dim3(3 * nx * ny + L.sp_blocks), dim3(kSpeciesChunk), 0, s, m, sys, ebar, qsig,
                       cols, nx, ny, cpart, L.cstride, spart);
  }
  const GradSums sums{part1, part2, cpart, bpart, L.cstride, spart, kch, L.ccK, L.ccN, L.beta_blocks, L.sp_blocks,
                      HP, H1, H2, heads, head};
  const int64_t total = (int64_t)kF * H1 + (int64_t)H1 * H2 + H1 + 2 * (int64_t)H2 +
                        (int64_t)nsp * nsp * kS * m.K + nsp + 1;
  hipLaunchKernelGGL(train_sums, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, m, sums, *g);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

}  // namespace gmnn
