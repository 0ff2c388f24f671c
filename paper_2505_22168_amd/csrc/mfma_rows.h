// MFMA products on row tiles of several 16-row blocks (the streamed readout's
// network and the training network): a wave owns the 16-column blocks
// w, w + 8, ... of a product for all row blocks, so every weight fragment
// loaded from L2 feeds as many MFMAs as the tile has row blocks.
#pragma once

#include "mfma.h"

namespace gmnn {

// A product is taken from NP parts of both operands: 1 (plain BF16), 2
// (split BF16: hh, hm, mh) or 3 (FP32: six_products), in the order of the tile
// readout's products (mfma.h).
// k-steps of B in flight: measured best on the 2x512 network (100,000 atoms,
// BF16: 433 us with 2 plain and 2 split steps, 453 with 3 and 2, 460 with 1
// and 2, 454 with 2 and 3; FP32: one three-part step, a second one spills)
constexpr int rows_depth(int NP) { return NP == 3 ? 1 : 2; }

template <int NP, int TPW>
struct RowsRing {
  bf16x8 b[rows_depth(NP)][TPW][NP];
};

template <int NP>
__device__ __forceinline__ void frag_parts(bf16x8 (&dst)[NP], const Weights& B, int lane, int inb, int KB, int kb) {
  dst[0] = frag_load(B.h, lane, inb, KB, kb);
  if constexpr (NP > 1) dst[1] = frag_load(B.m, lane, inb, KB, kb);
  if constexpr (NP > 2) dst[2] = frag_load(B.l, lane, inb, KB, kb);
}
template <int NP, int TPW>
__device__ __forceinline__ void rows_load(bf16x8 (&dst)[TPW][NP], const Weights& B, int KB, int kb, int nb0, int nbs,
                                          int NB) {
#pragma unroll
  for (int i = 0; i < TPW; ++i)
    if (has_block(i, nb0, nbs, NB) && kb < KB) frag_parts<NP>(dst[i], B, frag_lane(nb0, KB), i * nbs, KB, kb);
}

// the first k-steps of a product's B fragments, issued ahead of the product
// (their latency then overlaps the previous phase)
template <int NP, int TPW>
__device__ __forceinline__ void rows_pre(RowsRing<NP, TPW>& r, const Weights& B, int KB, int nb0, int nbs, int NB) {
#pragma unroll
  for (int s = 0; s < rows_depth(NP); ++s) rows_load<NP, TPW>(r.b[s], B, KB, s, nb0, nbs, NB);
}

// acc += A B with r holding the first k-steps; part q of A at A + q * apart
// elements.  ATOM_ROWS: the activations are the MFMA's A operand (a lane then
// holds four consecutive atoms of one unit)
template <int NP, int MB, int TPW, bool ATOM_ROWS = false>
__device__ __forceinline__ void mma_rows(RowsRing<NP, TPW>& ring, const __bf16* __restrict__ A, int apart, int lda,
                                         const Weights& B, int KB, int nb0, int nbs, int NB,
                                         floatx4 (&acc)[MB][TPW]) {
  const int l = threadIdx.x & 63;
  const __bf16* abase = A + (l & 15) * lda + (l >> 4) * 8;
  if constexpr (NP == 3) {
    // one k-step in flight: a column block's fragments are replaced by the
    // next step's as soon as its products are issued, three quarters of a
    // step ahead of their use
#pragma unroll 1
    for (int kb = 0; kb < KB; ++kb) {
      Split3 a[MB];
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        const __bf16* p = abase + r * 16 * lda + kb * 32;
        a[r] = Split3{*(const bf16x8*)p, *(const bf16x8*)(p + apart), *(const bf16x8*)(p + 2 * apart)};
      }
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        if (!has_block(i, nb0, nbs, NB)) continue;
        const Split3 b{ring.b[0][i][0], ring.b[0][i][1], ring.b[0][i][2]};
        auto fa = [&](int r) -> const Split3& { return a[r]; };
        auto fb = [&](int) -> const Split3& { return b; };
        floatx4 t[MB];
        six_products<!ATOM_ROWS>(t, fa, fb);
#pragma unroll
        for (int r = 0; r < MB; ++r) add_step(acc[r][i], t[r], step_sign(kb));
        // (past the last step: the same step's fragments again, unused)
        frag_parts<NP>(ring.b[0][i], B, frag_lane(nb0, KB), i * nbs, KB, min(kb + 1, KB - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    constexpr int PF = rows_depth(NP);
    auto step = [&](const bf16x8 (&b)[TPW][NP], int kb) {
      // one row block's A parts at a time (fewer registers live)
#pragma unroll
      for (int r = 0; r < MB; ++r) {
        bf16x8 a[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) a[q] = *(const bf16x8*)(abase + q * apart + r * 16 * lda + kb * 32);
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
          if (!has_block(i, nb0, nbs, NB)) continue;
          auto mma = [&](const bf16x8& x, const bf16x8& y) {
            acc[r][i] = ATOM_ROWS ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc[r][i], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(y, x, acc[r][i], 0, 0, 0);
          };
          mma(a[0], b[i][0]);
          if constexpr (NP == 2) {
            mma(a[0], b[i][1]);
            mma(a[1], b[i][0]);
          }
        }
      }
    };
    pipeline<PF>(
        KB, [&](int slot, int kb) { step(ring.b[slot], kb); },
        [&](int slot, int kb) { rows_load<NP, TPW>(ring.b[slot], B, KB, kb, nb0, nbs, NB); });
  }
}

template <int MB, int TPW>
__device__ inline void zero_rows(floatx4 (&acc)[MB][TPW]) {
#pragma unroll
  for (int r = 0; r < MB; ++r)
#pragma unroll
    for (int i = 0; i < TPW; ++i) acc[r][i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
}

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

// four consecutive activations of one row, columns col .. col + 3, in NP parts,
// part q at base + q * part elements (three parts: with their k-step's sign)
template <int NP>
__device__ __forceinline__ void st4(__bf16* base, int part, int idx, int col, floatx4 v) {
  bf16x4 o[3];
  if constexpr (NP == 3) {
    v = v * step_sign(col / 32);
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      bf16x2 h, m, l;
      split3_pair(v[j], v[j + 1], h, m, l);
      o[0][j] = h[0]; o[0][j + 1] = h[1];
      o[1][j] = m[0]; o[1][j + 1] = m[1];
      o[2][j] = l[0]; o[2][j + 1] = l[1];
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[0][j] = (__bf16)v[j];
      if constexpr (NP == 2) o[1][j] = (__bf16)split_low(v[j], o[0][j]);
    }
  }
#pragma unroll
  for (int q = 0; q < NP; ++q) *(bf16x4*)(base + q * part + idx) = o[q];
}

}  // namespace gmnn
