// Streamed readout for large systems (three launches instead of the tile):
//
//   readout_features  invariants of the moments (Section 2.1, eq.
//                     contraction), 6 atoms per block -> G [N][384] in HBM
//                     (FP32, or for the BF16 network its bf16 high parts
//                     [N][384] followed by the low parts [N][384])
//   readout_network   the network, its scale/shift (eq. scale_shift) and its
//                     input gradient dE/dG, for row tiles of 32 to 64 atoms:
//                     every weight fragment fetched from L2 feeds 2 to 4 MFMA
//                     row blocks, 1/2 to 1/4 of the L2 traffic per atom of
//                     the 16-row tile
//   contract_back     product-rule backward of the invariants, one atom per
//                     lane -> dE/dPsi [N][100] (contract_lanes.hip)
//
// The arithmetic is the tile's, operation for operation (same contraction
// code, same MFMA shapes and k order, same epilogues; the same backward
// kernel follows both), so both give the same result bit for bit.
#include "common.h"
#include "contract_lanes.h"
#include "contraction.h"
#include "mfma.h"
#include "mfma_rows.h"
#include "model.h"

namespace gmnn {

// invariant blocks: 6 atoms and 256 threads (about 25 KB of LDS: six
// blocks per CU, whose load and barrier waits overlap one another; the
// arithmetic of an atom's invariants does not depend on the block size)
constexpr int kRoAtoms = 6;      // atoms per invariant (features) block
constexpr int kFtThreads = 256;  // threads of an invariant block
constexpr int kRoThreads = 512;  // threads of a network block
constexpr int kRoWaves = kRoThreads / 64;

static constexpr size_t ro_al(size_t x) { return (x + 255) & ~size_t(255); }

// ---------------------------------------------------------------------------
// shared: the tile's packed moments (one contiguous run) -> full tensors
__device__ inline void ro_load_moments(const float* __restrict__ psi, int row0, int n_rows, float* __restrict__ sPsi,
                                       const Tables& tb) {
  constexpr int NP = kS * kPacked;
  constexpr int NU = (kRoAtoms * NP + kFtThreads - 1) / kFtThreads;
  const int tid = threadIdx.x;
  float v[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int t = tid + u * kFtThreads;
    v[u] = t < n_rows * NP ? psi[(int64_t)row0 * NP + t] : 0.0f;
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int t = tid + u * kFtThreads;
    if (t < kRoAtoms * NP) {
      const int a = t / NP, e = t % NP;
      const int s = e / kPacked, c = e % kPacked;
      const int n = tb.packed_mult[c];
      for (int q = 0; q < n; ++q) sPsi[a * PS + s * kFull + tb.packed_full[c][q]] = v[u];
    }
  }
}

// ---------------------------------------------------------------------------
// 1. invariants
template <bool BF16>
struct FeatLds {
  static constexpr int ESZ = BF16 ? 2 : 4;
  static constexpr size_t tables = 0;
  static constexpr size_t psi = ro_al(sizeof(Tables));
  static constexpr size_t inter = psi + ro_al(4 * (size_t)kRoAtoms * PS);
  static constexpr size_t g = inter + ro_al(4 * (size_t)kRoAtoms * ISF);
  static constexpr size_t bytes = g + ro_al((BF16 ? 2 : 1) * (size_t)ESZ * kRoAtoms * kFP);
};

template <bool BF16>
__global__ void __launch_bounds__(kFtThreads) readout_features(DevSystem sys, const float* __restrict__ psi,
                                                               void* __restrict__ G) {
  using L = FeatLds<BF16>;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  Tables& tb = *(Tables*)(lds + L::tables);
  float* sPsi = (float*)(lds + L::psi);
  float* sI = (float*)(lds + L::inter);
  char* sG = lds + L::g;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * kRoAtoms;
  const int n_rows = min(kRoAtoms, sys.n_atoms - row0);
  load_tables(&tb);
  __syncthreads();
  ro_load_moments(psi, row0, n_rows, sPsi, tb);
  __syncthreads();
  constexpr int glo = BF16 ? kRoAtoms * kFP : 0;  // low parts after the high ones
  // the first pass runs each task's two independent halves on two threads
  // when the block has threads for both (no change to any arithmetic)
  constexpr int KSF = 2 * ((kRoAtoms * 20 + 63) / 64 * 64) <= kFtThreads ? 2 : 1;
  contract_forward_a<kRoAtoms, kFtThreads, BF16, true, ISF, KSF>(sPsi, sI, sG, kFP, tb, glo);
  __syncthreads();
  contract_forward_b<kRoAtoms, kFtThreads, BF16, ISF>(sPsi, sI, sG, kFP, tb, glo);
  __syncthreads();
  // rows of G are contiguous: 16-byte copies (BF16: the high plane, then the
  // low plane N rows further)
  const int n16 = n_rows * kFP * L::ESZ / 16;
  uint4* dst = (uint4*)((char*)G + (size_t)row0 * kFP * L::ESZ);
  for (int t = threadIdx.x; t < n16; t += kFtThreads) dst[t] = ((const uint4*)sG)[t];
  if (BF16) {
    uint4* dlo = (uint4*)((char*)G + ((size_t)sys.n_atoms + row0) * kFP * L::ESZ);
    const uint4* slo = (const uint4*)(sG + (size_t)glo * L::ESZ);
    for (int t = threadIdx.x; t < n16; t += kFtThreads) dlo[t] = slo[t];
  }
}

// ---------------------------------------------------------------------------
// 2. network on row tiles of TM atoms.  Wave w owns the 16-column blocks
// w, w + 8, ... of every product, for all TM/16 row blocks; each weight
// fragment loaded from L2 feeds TM/16 MFMAs.  Every product runs transposed:
// the weight fragment is the MFMA's A operand and the activation fragment
// its B operand (the two fragment layouts of the 16x16x32 BF16 MFMA coincide,
// so the packed weights and the LDS reads are those of the plain orientation).  A lane's accumulator then holds four
// consecutive hidden units (or features) of one atom, and every epilogue
// store is one 8-byte (BF16) or 16-byte (FP32) write instead of four
// scattered ones.  The block's barriers order LDS only (lds_barrier), so
// the weight fragments prefetched for the next product stay in flight
// through them.
// rows per network block: as many 16-row MFMA blocks as the register file
// (swish'(z1) is kept for the backward; 8 waves, 256 registers each) and,
// with three-part operands, the LDS hold: G at 2x256 or h1 at 2x512 fill it
template <int HP, bool BF16>
constexpr int net_rows() { return HP >= 512 ? 48 : (BF16 || HP >= 256) ? 64 : 32; }

template <int HP, bool BF16>
struct NetLds {
  static constexpr int TM = net_rows<HP, BF16>();
  static constexpr int NF = BF16 ? 2 : 3;  // parts of a forward operand
  static constexpr int NB = BF16 ? 1 : 3;  // parts of a backward operand
  static constexpr int G = kFP + 8, H = HP + 8;  // row strides (bf16)
  static constexpr size_t mx(size_t a, size_t b) { return a > b ? a : b; }
  // region A: G (all parts), then h1 (all parts), then delta1 at its start.
  // BF16: delta2 has a region of its own, and the energy partials of every
  // head [NW][TM][M] follow delta1.  FP32: delta2 takes h1's place, delta1
  // takes delta2's, and the energy partials of up to kEpHeads heads at a
  // time have a region of their own.
  static constexpr int kEpHeads = 4;
  static constexpr size_t part_g = (size_t)TM * G, part_h = (size_t)TM * H;  // elements
  static constexpr size_t b = 0;
  static constexpr size_t rows = b + (BF16 ? ro_al(2 * part_h) : ro_al(4 * (size_t)kRoWaves * TM * kEpHeads));
  static constexpr size_t a = rows + ro_al(4 * 3 * (size_t)TM);  // scale, shift, structure of each row
  static constexpr size_t ep = BF16 ? a + ro_al(2 * part_h) : 0;
  static constexpr size_t a_bytes = ro_al(2 * NF * mx(part_g, part_h));
  static constexpr size_t bytes(int M) {
    return BF16 ? mx(a + a_bytes, ep + ro_al(4 * (size_t)kRoWaves * TM * M)) : a + a_bytes;
  }
};

// DSW: the forward of per-head backwards (energies and swish', no backward)
template <int HP, bool BF16, bool DSW>
__global__ void __launch_bounds__(kRoThreads)
    readout_network(DevModel m, DevSystem sys, const void* __restrict__ G, float* __restrict__ atomic_e,
                    float* __restrict__ dG) {
  using L = NetLds<HP, BF16>;
  constexpr int TM = L::TM, MB = TM / 16, NW = kRoWaves;
  constexpr int NF = L::NF, NBK = L::NB;
  constexpr int NBH = HP / 16, NBG = kFP / 16;
  constexpr int TPW = (NBH + NW - 1) / NW, TPW_G = (NBG + NW - 1) / NW;
  constexpr int PG = (int)L::part_g, PH = (int)L::part_h;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __bf16* sA = (__bf16*)(lds + L::a);
  __bf16* sB = BF16 ? (__bf16*)(lds + L::b) : sA;  // delta2
  float* sEp = (float*)(lds + L::ep);
  float* sScale = (float*)(lds + L::rows);
  float* sShift = sScale + TM;
  int* sStruct = (int*)(sShift + TM);
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * TM;
  const int n_rows = min(TM, sys.n_atoms - row0);
  const int M = m.M;
  // a lane's accumulator entries j = 0..3 of a 16 x 16 block: unit (or
  // feature) uq + j of the column block, atom ar of the row block
  const int ar = l & 15, uq = 4 * (l >> 4);

  // the B fragments of each product's first k-steps are issued one phase
  // ahead (W1's with the tile's G rows, W2's before the first epilogue,
  // W2^T's and W1^T's before the second and third), so their latency
  // overlaps loads, barriers and epilogues instead of the products
  RowsRing<NF, TPW> rf;
  RowsRing<NBK, TPW> rb;
  RowsRing<NBK, TPW_G> rg;

  // G rows (BF16: each part; FP32: split here) -> region A, zero rows beyond
  // the system; every load of the tile is issued before the first store
  {
    constexpr int ESZ = BF16 ? 2 : 4;
    constexpr int NS = BF16 ? 2 : 1;
    constexpr int C16 = kFP * ESZ / 16;  // 16-byte chunks per row
    constexpr int NU = (NS * TM * C16 + kRoThreads - 1) / kRoThreads;
    const char* gbase = (const char*)G;
    uint4 v[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = tid + u * kRoThreads;
      const int part = t / (TM * C16), tt = t % (TM * C16);
      v[u] = uint4{0u, 0u, 0u, 0u};
      if (part < NS && tt < n_rows * C16)
        v[u] = ((const uint4*)(gbase + ((size_t)part * sys.n_atoms + row0) * kFP * ESZ))[tt];
    }
    // W1's first k-steps after the tile's rows: the LDS stores below wait
    // for the rows only
    rows_pre<NF, TPW>(rf, m.w1, kFP / 32, w, NW, NBH);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int t = tid + u * kRoThreads;
      const int part = t / (TM * C16), tt = t % (TM * C16);
      if (part >= NS) continue;
      if constexpr (BF16) *(uint4*)(sA + part * PG + (tt / C16) * L::G + (tt % C16) * 8) = v[u];
      else st4<3>(sA, PG, (tt / C16) * L::G + (tt % C16) * 4, (tt % C16) * 4, __builtin_bit_cast(floatx4, v[u]));
    }
    for (int a = tid; a < TM; a += kRoThreads) {
      float sc = 0.0f, sh = 0.0f;
      int b = 0;
      if (a < n_rows) {
        const int z = sys.species[row0 + a];
        sc = m.scale[z];
        sh = m.shift[z];
        b = sys.atom_struct[row0 + a];
      }
      sScale[a] = sc;
      sShift[a] = sh;
      sStruct[a] = b;
    }
  }
  lds_barrier();

  // z1 = G W1 + b1, h1 = swish(z1) -> region A once every
  // wave is done with G; swish'(z1) stays in registers
  floatx4 dsw1[MB][TPW];
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NF>(rf, sA, PG, L::G, m.w1, kFP / 32, w, NW, NBH, acc);
    rows_pre<NF, TPW>(rf, m.w2, HP / 32, w, NW, NBH);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = w + i * NW;
      if (nb >= NBH) continue;
      const floatx4 bias = *(const floatx4*)(m.b1 + nb * 16 + uq);
#pragma unroll
      for (int r = 0; r < MB; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float d;
          acc[r][i][j] = swish_parts(acc[r][i][j] + bias[j], d);
          dsw1[r][i][j] = d;
        }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = w + i * NW;
      if (nb >= NBH) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r)
        st4<NF>(sA, PH, (r * 16 + ar) * L::H + nb * 16 + uq, nb * 16 + uq, acc[r][i]);
    }
  }
  lds_barrier();

  // z2 = h1 W2 + b2, h2 = swish(z2); delta2 = swish'(z2) sigma wbar -> sB, and
  // per-wave partial sums of h2 . W3[:,m] -> sEp, once every wave is done with h1
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NF>(rf, sA, PH, L::H, m.w2, HP / 32, w, NW, NBH, acc);
    rows_pre<NBK, TPW>(rb, m.w2t, HP / 32, w, NW, NBH);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = w + i * NW;
      if (nb >= NBH) continue;
      const int col = nb * 16 + uq;
      const floatx4 bias = *(const floatx4*)(m.b2 + col);
      const floatx4 wb = *(const floatx4*)(m.w3bar + col);
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        const int row = r * 16 + ar;
        floatx4 d;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float dj;
          acc[r][i][j] = swish_parts(acc[r][i][j] + bias[j], dj);
          d[j] = dj;
        }
        if (m.h2_out && row < n_rows) *(floatx4*)(m.h2_out + (int64_t)(row0 + row) * HP + col) = acc[r][i];
        if (DSW && row < n_rows) {
          float* o = m.dsw_out + (int64_t)(row0 + row) * HP + col;
          *(floatx4*)o = dsw1[r][i];
          *(floatx4*)(o + (int64_t)sys.n_atoms * HP) = d * sScale[row];
        }
        const floatx4 wr = m.head_w ? *(const floatx4*)(m.head_w + (int64_t)sStruct[row] * HP + col) : wb;
        st4<NBK>(sB, PH, row * L::H + col, col, d * sScale[row] * wr);
      }
    }
    // BF16: the partials of all heads at once; FP32: kEpHeads at a time
    const int hstep = BF16 ? M : L::kEpHeads;
    for (int h0 = 0; h0 < M; h0 += hstep) {
      const int nh = min(hstep, M - h0);
      if (h0 > 0) lds_barrier();  // the previous heads' partials are read
      for (int hq = 0; hq < nh; ++hq) {
        const int hm = h0 + hq;
#pragma unroll
        for (int r = 0; r < MB; ++r) {
          // per unit c = uq + j of the 16-column blocks: the sum over the
          // wave's blocks; then an xor butterfly over the 16 units (bits 3 and
          // 2 of c across the lane groups, bits 1 and 0 inside the lane), the
          // tree the tile readout's row sums take, so both readouts agree bit
          // for bit
          float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int i = 0; i < TPW; ++i) {
            const int nb = w + i * NW;
            if (nb >= NBH) continue;
            floatx4 w3;
            if (M == 1) {
              w3 = *(const floatx4*)(m.w3 + nb * 16 + uq);
            } else {
#pragma unroll
              for (int j = 0; j < 4; ++j) w3[j] = m.w3[(nb * 16 + uq + j) * M + hm];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) part[j] += acc[r][i][j] * w3[j];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            part[j] += __shfl_xor(part[j], 32);
            part[j] += __shfl_xor(part[j], 16);
          }
          const float v = (part[0] + part[2]) + (part[1] + part[3]);
          if (l < 16) sEp[(w * TM + r * 16 + ar) * nh + hq] = v;
        }
      }
      lds_barrier();
      for (int t = tid; t < TM * nh; t += kRoThreads) {
        const int a = t / nh, hq = t % nh;
        if (a < n_rows) {
          float y = m.b3[h0 + hq];
#pragma unroll
          for (int ww = 0; ww < NW; ++ww) y += sEp[(ww * TM + a) * nh + hq];
          atomic_e[(int64_t)(row0 + a) * M + h0 + hq] = sScale[a] * y + sShift[a];
        }
      }
    }
  }
  // forward-only pass (the energies an uncertainty bias needs first)
  if (DSW || m.fwd_only) return;

  // delta1 = swish'(z1) (delta2 W2^T) -> region A (h1 is dead)
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NBK>(rb, sB, PH, L::H, m.w2t, HP / 32, w, NW, NBH, acc);
    rows_pre<NBK, TPW_G>(rg, m.w1t, HP / 32, w, NW, NBG);
    if (!BF16) lds_barrier();  // every wave is done with delta2, which delta1 replaces
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = w + i * NW;
      if (nb >= NBH) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r)
        st4<NBK>(sA, PH, (r * 16 + ar) * L::H + nb * 16 + uq, nb * 16 + uq, acc[r][i] * dsw1[r][i]);
    }
  }
  lds_barrier();

  // dE/dG = delta1 W1^T -> HBM (FP32, dg_index).  The activations are the
  // A operand here, so a lane holds one feature of four consecutive atoms:
  // one 16-byte store in the feature-major runs
  {
    floatx4 acc[MB][TPW_G];
    zero_rows(acc);
    mma_rows<NBK, MB, TPW_G, true>(rg, sA, PH, L::H, m.w1t, HP / 32, w, NW, NBG, acc);
#pragma unroll
    for (int i = 0; i < TPW_G; ++i) {
      const int nb = w + i * NW;
      if (nb >= NBG) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        const int row = r * 16 + uq;
        if (row >= n_rows) continue;
        float* o = dG + dg_index(sys.n_atoms, row0 + row, nb * 16 + ar);
        if (sys.n_atoms - (row0 + row) / kDgRun * kDgRun >= kDgRun) {
          *(floatx4*)o = acc[r][i];  // a whole run: its rows are 16-byte aligned
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (row + j < n_rows) o[j] = acc[r][i][j];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The network's backward for several heads (Section 2.2: the heads share
// everything but W3): rows are (head, atom), row block r the 16 atoms of the
// tile under head h0 + r, so swish' of both layers is loaded once for all
// heads and every weight fragment feeds HB row blocks.
//   delta2 = sigma swish'(z2) W3[:, h], delta1 = swish'(z1) (delta2 W2^T),
//   dE/dG = delta1 W1^T -> dG [head][...] (dg_index)
// What bounds it: the latency of the weights from L2 and of W3's column, at
// two blocks a CU (28,160 atoms, 2x256 BF16: 89 us for four heads, four times
// for 16).  With its forward (97 us) and the invariant backward (4 x 68 us)
// it replaces the readout tile, which ran the heads of an atom one after the
// other, the invariant backward between them (1313 us).
template <int HP, bool BF16>
struct HeadsLds {
  static constexpr int NP = BF16 ? 1 : 3;
  static constexpr int HB = 4;  // heads per block
  static constexpr int H = HP + 8;
  static constexpr size_t part = (size_t)16 * HB * H;
  static constexpr size_t bytes = 2 * NP * part;
};

template <int HP, bool BF16>
__global__ void __launch_bounds__(kRoThreads)
    network_heads(DevModel m, int n_atoms, const float* __restrict__ dsw, int head0, int n_heads,
                  float* __restrict__ dG) {
  using L = HeadsLds<HP, BF16>;
  constexpr int NP = L::NP, MB = L::HB, NW = kRoWaves;
  constexpr int NBH = HP / 16, NBG = kFP / 16;
  constexpr int TPW = (NBH + NW - 1) / NW, TPW_G = (NBG + NW - 1) / NW;
  constexpr int PH = (int)L::part;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  __bf16* sT = (__bf16*)lds;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int row0 = xcd_block(blockIdx.x, gridDim.x) * 16;
  const int n_rows = min(16, n_atoms - row0);
  const int hb = blockIdx.y * MB, nh = min(MB, n_heads - hb);  // heads of this block, from head0 + hb
  const int ar = l & 15, uq = 4 * (l >> 4);
  RowsRing<NP, TPW> ring;
  RowsRing<NP, TPW_G> ring_g;
  rows_pre<NP, TPW>(ring, m.w2t, HP / 32, w, NW, NBH);
  floatx4 dsw1[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (!has_block(i, w, NW, NBH)) continue;
    const int col = (w + i * NW) * 16 + uq;
    floatx4 d2 = {0.0f, 0.0f, 0.0f, 0.0f};
    dsw1[i] = d2;
    if (ar < n_rows) {
      const float* p = dsw + (int64_t)(row0 + ar) * HP + col;
      dsw1[i] = *(const floatx4*)p;
      d2 = *(const floatx4*)(p + (int64_t)n_atoms * HP);
    }
#pragma unroll
    for (int r = 0; r < MB; ++r) {
      floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
      if (r < nh)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = d2[j] * m.w3[(col + j) * m.M + head0 + hb + r];
      st4<NP>(sT, PH, (r * 16 + ar) * L::H + col, col, v);
    }
  }
  lds_barrier();
  {
    floatx4 acc[MB][TPW];
    zero_rows(acc);
    mma_rows<NP>(ring, sT, PH, L::H, m.w2t, HP / 32, w, NW, NBH, acc);
    rows_pre<NP, TPW_G>(ring_g, m.w1t, HP / 32, w, NW, NBG);
    lds_barrier();  // every wave is done with delta2, which delta1 replaces
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      if (!has_block(i, w, NW, NBH)) continue;
#pragma unroll
      for (int r = 0; r < MB; ++r)
        st4<NP>(sT, PH, (r * 16 + ar) * L::H + (w + i * NW) * 16 + uq, (w + i * NW) * 16 + uq,
                acc[r][i] * dsw1[i]);
    }
  }
  lds_barrier();
  {
    floatx4 acc[MB][TPW_G];
    zero_rows(acc);
    mma_rows<NP, MB, TPW_G, true>(ring_g, sT, PH, L::H, m.w1t, HP / 32, w, NW, NBG, acc);
    const bool whole = n_atoms - row0 / kDgRun * kDgRun >= kDgRun;  // a whole run: 16-byte aligned rows
#pragma unroll
    for (int i = 0; i < TPW_G; ++i) {
      if (!has_block(i, w, NW, NBG)) continue;
      if (uq >= n_rows) continue;
      const int64_t o = dg_index(n_atoms, row0 + uq, (w + i * NW) * 16 + ar);
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        if (r >= nh) continue;
        float* p = dG + (int64_t)(hb + r) * n_atoms * kFP + o;
        if (whole) {
          *(floatx4*)p = acc[r][i];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (uq + j < n_rows) p[j] = acc[r][i][j];
        }
      }
    }
  }
}

template <int HP, bool BF16>
static gmnn_status launch_heads_t(const DevModel& m, const DevSystem& sys, const float* dsw, int head0, int n_heads,
                                  float* dG, hipStream_t s) {
  using L = HeadsLds<HP, BF16>;
  static_assert(L::bytes <= 160 * 1024, "the tile fits the LDS");
  const gmnn_status st = ensure_lds_limit((const void*)network_heads<HP, BF16>, L::bytes);
  if (st != GMNN_OK) return st;
  hipLaunchKernelGGL((network_heads<HP, BF16>), dim3((sys.n_atoms + 15) / 16, (n_heads + L::HB - 1) / L::HB),
                     dim3(kRoThreads), L::bytes, s, m, sys.n_atoms, dsw, head0, n_heads, dG);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

// dE/dG of heads head0 .. head0 + n_heads - 1 (n_heads arrays, one after the
// other), from the forward's swish' values (DevModel::dsw_out)
gmnn_status launch_network_heads(const DevModel& m, const DevSystem& sys, bool bf16, const float* dsw, int head0,
                                 int n_heads, float* dG, hipStream_t s) {
  if (sys.n_atoms == 0 || n_heads == 0) return GMNN_OK;
#define CASE(HP)                                                                     \
  if (m.HP1 == HP)                                                                   \
    return bf16 ? launch_heads_t<HP, true>(m, sys, dsw, head0, n_heads, dG, s)       \
                : launch_heads_t<HP, false>(m, sys, dsw, head0, n_heads, dG, s);
  CASE(64) CASE(128) CASE(256)
#undef CASE
  // (no plan serves FP32 2x512 with one backward per head)
  if (m.HP1 == 512 && bf16) return launch_heads_t<512, true>(m, sys, dsw, head0, n_heads, dG, s);
  return GMNN_ERR_UNSUPPORTED;
}

// ---------------------------------------------------------------------------
constexpr size_t kLdsMax = 160 * 1024;

// phases: bit 0 invariants, bit 1 network, bit 2 invariant backward
template <int HP, bool BF16>
static gmnn_status launch_stream_t(const DevModel& m, const DevSystem& sys, const float* psi, void* G, float* dG,
                                   float* atomic_e, float* psibar, hipStream_t s, hipEvent_t* ev, int phases) {
  auto mark = [&](int k) {
    if (ev) (void)hipEventRecord(ev[k], s);
  };
  using NL = NetLds<HP, BF16>;
  if (NL::bytes(m.M) > kLdsMax) return GMNN_ERR_UNSUPPORTED;
  gmnn_status st = ensure_lds_limit((const void*)readout_features<BF16>, FeatLds<BF16>::bytes);
  auto network = m.dsw_out ? readout_network<HP, BF16, true> : readout_network<HP, BF16, false>;
  if (st == GMNN_OK) st = ensure_lds_limit((const void*)network, NL::bytes(m.M));
  if (st != GMNN_OK) return st;
  const int N = sys.n_atoms;
  const int g16 = (N + kRoAtoms - 1) / kRoAtoms;
  const int gn = (N + NL::TM - 1) / NL::TM;
  mark(0);
  if (phases & 1)
    hipLaunchKernelGGL(readout_features<BF16>, dim3(g16), dim3(kFtThreads), FeatLds<BF16>::bytes, s, sys, psi, G);
  mark(1);
  mark(2);
  if (phases & 2)
    hipLaunchKernelGGL(network, dim3(gn), dim3(kRoThreads), NL::bytes(m.M), s, m, sys,
                       (const void*)G, atomic_e, dG);
  mark(3);
  mark(4);
  if (phases & 4) {
    st = launch_contract_back(N, 1, psi, dG, psibar, s);
    if (st != GMNN_OK) return st;
  }
  mark(5);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

size_t stream_lds_bytes(int hp, bool bf16, int n_heads) {
  size_t n = 0;
#define SZ(HP) \
  if (hp == HP) n = bf16 ? NetLds<HP, true>::bytes(n_heads) : NetLds<HP, false>::bytes(n_heads);
  SZ(64) SZ(128) SZ(256) SZ(512)
#undef SZ
  if (n == 0) return ~size_t(0);
  size_t f = bf16 ? FeatLds<true>::bytes : FeatLds<false>::bytes;
  if (f > n) n = f;
  return n;
}

// workspace of the streamed readout: G [N][kFP] (FP32, or bf16 high and low
// planes) and dE/dG [N][kFP] FP32
size_t stream_g_bytes(int n_atoms, bool bf16) { return (size_t)n_atoms * kFP * (bf16 ? 2 * 2 : 4); }
size_t stream_dg_bytes(int n_atoms) { return (size_t)n_atoms * kFP * 4; }

// ev (may be null): 6 events recorded around the three kernels; phases:
// which of the three run (bit 0 invariants, bit 1 network, bit 2 invariant
// backward)
gmnn_status launch_stream(const DevModel& m, const DevSystem& sys, bool bf16, const float* psi, void* G, float* dG,
                          float* atomic_e, float* psibar, hipStream_t s, hipEvent_t* ev, int phases) {
  if (sys.n_atoms == 0) return GMNN_OK;
#define CASE(HP)                                                                                          \
  if (m.HP1 == HP)                                                                                        \
    return bf16 ? launch_stream_t<HP, true>(m, sys, psi, G, dG, atomic_e, psibar, s, ev, phases)          \
                : launch_stream_t<HP, false>(m, sys, psi, G, dG, atomic_e, psibar, s, ev, phases);
  CASE(64) CASE(128) CASE(256) CASE(512)
#undef CASE
  return GMNN_ERR_UNSUPPORTED;
}

}  // namespace gmnn
