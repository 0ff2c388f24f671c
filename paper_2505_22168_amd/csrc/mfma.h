// MFMA tile products and the network stage of a tile (gfx950).
//
// Weight layout (filled by gmnn_model_prepare), for B = W of shape K x N:
//   16x16x32 BF16 MFMA: fragment (nb, kb) is 64 lanes x 8 bf16, lane l holding
//     B[32 kb + 8 (l>>4) + e][16 nb + (l&15)], e = 0..7     -> one 16-byte load
//   in three parts h + m + l = w (model.h).
// A tiles live in LDS, row-major, rows padded so 16-byte reads stay aligned.
//
// FP32 products.  The FP32 MFMA (16x16x4) issues 256 FLOP per cycle and CU,
// the BF16 one 4096.  An FP32 product is therefore taken from three-part
// operands, x = h + m + l exactly with 8 significant bits per part, as the six
// BF16 products hh, hm, mh, mm, hl, lh, with FP32 accumulation: 96 cycles per
// 16x16x32 block instead of 256, and K/32 roundings of the sum instead of K.
// The dropped ml, lm and ll are at most 2^-24 of a term together, half an ulp
// (|m| <= 2^-8, |l| <= 2^-17 of a value near 1).  Measured against 64 bits:
// atomic energies 0.79 and forces 0.91 times the FP32 MFMA's errors (150
// structures, 2x256, rms of 20 sets of inputs), the nine gradients of a training
// step 0.92 to 1.02 (two structures, likewise) and 0.97 in the mean (11,200 atoms,
// 2x512, six sets; single gradients of a set 0.65 to 1.06).
#pragma once

#include "common.h"
#include "model.h"
#include "tables.h"

namespace gmnn {

// Each wave owns one 16-row block rb and the 16-column blocks nb0 + i*nbs
// (i < TPW, nb < NB).  B fragments stream from L2 through a ring of register
// buffers, PF k-steps ahead of the MFMAs: 16 BF16 fragments (64 registers) in
// flight per wave whatever the width, 6 to 8 three-part ones (72 to 96) for
// FP32.  The ring of a product can be filled ahead of it (ring_fill), e.g.
// before the epilogue and barrier of the previous product, so its first
// fragments arrive during them.
template <int TPW>
constexpr int prefetch_depth() { return TPW >= 4 ? 4 : 16 / TPW > 8 ? 8 : 16 / TPW; }
// ... of three-part fragments where BF16 ones would go `depth` deep
constexpr int prefetch_depth3(int tpw, int depth) {
  return depth < 4 ? (tpw >= 2 ? 1 : 2) : tpw >= 4 ? 2 : tpw >= 2 ? 3 : 6;
}

// the parts of a three-part fragment
struct Split3 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ Split3 split3x8(floatx4 a, floatx4 b) {
  Split3 s;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const floatx4 v = e < 4 ? a : b;
    bf16x2 h, m, l;
    split3_pair(v[e & 3], v[(e & 3) + 1], h, m, l);
    s.h[e] = h[0]; s.h[e + 1] = h[1];
    s.m[e] = m[0]; s.m[e + 1] = m[1];
    s.l[e] = l[0]; s.l[e + 1] = l[1];
  }
  return s;
}

// one k-step of N FP32 products, t[n] = x(n) y(n), smallest part products first
// from zero, to be added to the sum in FP32.  An MFMA aligns the sum it adds to
// with its products and drops what falls below, towards minus infinity: a long
// sum kept in it drifts by 1e-6 of a force, and a step's six products still by
// 2e-9 of their terms, which doubles the error of a solid's stress.  So x is
// negated in every other k-step (step_sign; exact) and those steps' products
// are subtracted: the drift cancels.  The N chains are interleaved: an MFMA
// waits for the one before it in its own chain.  SWAP: y is the MFMA's A
// operand (the order of the part products stays, so both orientations agree
// bit for bit).
template <bool SWAP = false, int N, typename X, typename Y>
__device__ __forceinline__ void six_products(floatx4 (&t)[N], X x, Y y) {
#define GMNN_PART(PX, PY, FROM)                                                                           \
  _Pragma("unroll") for (int n = 0; n < N; ++n)                                                           \
      t[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(SWAP ? y(n).PY : x(n).PX, SWAP ? x(n).PX : y(n).PY, \
                                                     FROM, 0, 0, 0)
  GMNN_PART(l, h, (floatx4{0.0f, 0.0f, 0.0f, 0.0f}));
  GMNN_PART(h, l, t[n]);
  GMNN_PART(m, m, t[n]);
  GMNN_PART(m, h, t[n]);
  GMNN_PART(h, m, t[n]);
  GMNN_PART(h, h, t[n]);
#undef GMNN_PART
}
// the sign of k-step kb's x, and a signed step's products into the sum
__device__ __forceinline__ float step_sign(int kb) { return kb & 1 ? -1.0f : 1.0f; }
__device__ __forceinline__ void add_step(floatx4& sum, const floatx4& t, float sign) {
#pragma unroll
  for (int j = 0; j < 4; ++j) sum[j] = __builtin_fmaf(sign, t[j], sum[j]);
}

// k-steps 0 .. KB - 1 of a product whose fragments come through a ring of PF
// slots, the first PF of them already issued: step(slot, kb), then
// load(slot, kb + PF).  The last steps are peeled, so no branch guards a load
// (a guarded one would put the ring in scratch memory).  The 64-wide BF16
// tile, where half the waves have no column block, takes the loop unrolled
// (582 atoms: 31.9 us against 32.3; 2x128 33.2 against 33.0, 2x512 52.3 against 51.9).
template <int PF, int UNROLL = 1, typename Step, typename Load>
__device__ __forceinline__ void pipeline(int KB, Step step, Load load) {
  const int full = KB > PF ? (KB - PF) / PF * PF : 0;
#pragma unroll UNROLL
  for (int kb = 0; kb < full; kb += PF) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      step(s, kb + s);
      load(s, kb + s + PF);
    }
  }
#pragma unroll
  for (int s = 0; s < 2 * PF; ++s) {
    if (full + s >= KB) continue;
    step(s % PF, full + s);
    if (full + s + PF < KB) load(s % PF, full + s + PF);
  }
}

template <bool BF16>
struct FragT { using type = bf16x8; };
template <>
struct FragT<false> { using type = Split3; };

template <bool BF16, int TPW, int DEPTH = prefetch_depth<TPW>()>
struct BRing {
  static constexpr int PF = BF16 ? DEPTH : prefetch_depth3(TPW, DEPTH);
  typename FragT<BF16>::type b[PF][TPW];
};

// Fragment (nb0 + i nbs, kb) of one part of B, as a buffer load: the wave's
// block and the lane in one 32-bit offset (frag_lane), i and kb in a scalar
// one, so a product's loads share a single address register.  Three-part
// fragments and four column blocks a wave need the registers (FP32 2x256 tile,
// 48 atoms: 45.8 us, 47.0 with plain addresses; BF16 2x512: 49.0 and 49.4);
// fewer BF16 fragments take plain addresses (frag_plain: 2x64 at 582 atoms 32.2
// us against 32.5, 2x256 at 1400 39.5 against 39.9).
__device__ __forceinline__ int frag_lane(int nb0, int KB) { return (nb0 * KB * 64 + (threadIdx.x & 63)) * 16; }
__device__ __forceinline__ bf16x8 frag_load(const bf16x8* part, int lane, int inb, int KB, int kb) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc((void*)part, 0, 0x7fffffff, 0x00027000);
  return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane, (inb * KB + kb) * 1024, 0));
}

__device__ __forceinline__ bf16x8 frag_plain(const bf16x8* part, int lane, int inb, int KB, int kb) {
  return *(const bf16x8*)((const char*)part + lane + (size_t)((inb * KB + kb) * 1024));
}
template <int TPW>
__device__ __forceinline__ bf16x8 frag_bf16(const bf16x8* part, int lane, int inb, int KB, int kb) {
  if constexpr (TPW < 4) return frag_plain(part, lane, inb, KB, kb);
  else return frag_load(part, lane, inb, KB, kb);
}

// whether a wave has an i-th column block (known at compile time where the
// blocks divide evenly, so that no branch guards the ring's registers)
__device__ __forceinline__ bool has_block(int i, int nb0, int nbs, int NB) {
  return NB >= (i + 1) * nbs || nb0 + i * nbs < NB;
}

template <bool BF16, int TPW, int DEPTH>
__device__ __forceinline__ void ring_load(BRing<BF16, TPW, DEPTH>& r, int slot, const Weights& B, int KB, int kb,
                                          int nb0, int nbs, int NB) {
  const int lane = frag_lane(nb0, KB);
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (has_block(i, nb0, nbs, NB) && kb < KB) {
      auto part = [&](const bf16x8* p) { return frag_load(p, lane, i * nbs, KB, kb); };
      if constexpr (BF16) r.b[slot][i] = frag_bf16<TPW>(B.h, lane, i * nbs, KB, kb);
      else r.b[slot][i] = Split3{part(B.h), part(B.m), part(B.l)};
    }
  }
}

// issue the first PF k-steps of the product with B of K rows
template <bool BF16, int TPW, int DEPTH>
__device__ __forceinline__ void ring_fill(BRing<BF16, TPW, DEPTH>& r, const Weights& B, int K, int nb0, int nbs,
                                          int NB) {
#pragma unroll
  for (int s = 0; s < BRing<BF16, TPW, DEPTH>::PF; ++s) ring_load(r, s, B, K / 32, s, nb0, nbs, NB);
}

// acc += A[rb rows] B over K, with the ring already holding k-steps 0..PF-1.
// A: bf16 (BF16), or FP32 split into its parts as it is read (the same parts,
// and the same order of products, as the streamed readout's)
template <bool BF16, int TPW, int DEPTH>
__device__ __forceinline__ void mma_ring(BRing<BF16, TPW, DEPTH>& r, const void* A, int lda, int rb, const Weights& B,
                                         int K, int nb0, int nbs, int NB, floatx4 (&acc)[TPW]) {
  constexpr int PF = BRing<BF16, TPW, DEPTH>::PF;
  const int l = threadIdx.x & 63;
  const int KB = K / 32;
  const int row = (rb * 16 + (l & 15)) * lda + (l >> 4) * 8;
  if constexpr (BF16) {
    auto step = [&](int slot, int kb) {
      const bf16x8 a = *(const bf16x8*)((const __bf16*)A + row + kb * 32);
#pragma unroll
      for (int i = 0; i < TPW; ++i)
        if (has_block(i, nb0, nbs, NB))
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, r.b[slot][i], acc[i], 0, 0, 0);
    };
    auto load = [&](int slot, int kb) { ring_load(r, slot, B, KB, kb, nb0, nbs, NB); };
    if (NB < nbs) pipeline<PF, 4>(KB, step, load);
    else pipeline<PF>(KB, step, load);
  } else {
    // a wave with one column block runs two k-steps at once: one chain of six
    // dependent MFMAs would leave the pipe waiting (every K here is a multiple
    // of 64)
    constexpr int U = TPW == 1 ? 2 : 1;
    static_assert(PF % U == 0, "whole groups of k-steps in the ring");
    pipeline<PF / U>(
        KB / U,
        [&](int slot, int g) {
          // only a product narrower than the waves leaves some without a block
          // (one column block per wave there)
          if (TPW == 1 && !has_block(0, nb0, nbs, NB)) return;
          Split3 a[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float* p = (const float*)A + row + (g * U + u) * 32;
            const float sign = step_sign(g * U + u);
            a[u] = split3x8(sign * *(const floatx4*)p, sign * *(const floatx4*)(p + 4));
          }
          floatx4 t[U * TPW];
          six_products(t, [&](int n) -> const Split3& { return a[n / TPW]; },
                       [&](int n) -> const Split3& { return r.b[slot * U + n / TPW][n % TPW]; });
#pragma unroll
          for (int n = 0; n < U * TPW; ++n) add_step(acc[n % TPW], t[n], step_sign(g * U + n / TPW));
        },
        [&](int slot, int g) {
#pragma unroll
          for (int u = 0; u < U; ++u) ring_load(r, slot * U + u, B, KB, g * U + u, nb0, nbs, NB);
        });
  }
}

// ---------------------------------------------------------------------------
// Split-BF16 products (the network's forward products in BF16 mode).  Each
// FP32 operand x is held as two bf16 parts, hi = bf16(x) and lo = bf16(x - hi)
// (x - hi is exact in FP32), and
//   acc += Ahi Bhi + Ahi Blo + Alo Bhi        (per k-step, in this order)
// keeps about 16 significant bits of every operand; the dropped Alo Blo term
// is 2^-16 relative.  Three BF16 MFMAs per k-step instead of one, FP32
// accumulation.  The A parts live in LDS (high and low parts in two arrays
// of the same layout); the B fragments stream through a ring whose slot i < TPW
// holds the high fragment of column block nb0 + i nbs and slot TPW + i its
// low fragment (same fragment layout, separate arrays).
template <bool BF16, int TPW, int DEPTH>
struct FwdRingT {
  using type = BRing<false, TPW, DEPTH>;
};
template <int TPW, int DEPTH>
struct FwdRingT<true, TPW, DEPTH> {
  using type = BRing<true, 2 * TPW, (DEPTH / 2 > 0 ? DEPTH / 2 : 1)>;
};
template <bool BF16, int TPW, int DEPTH>
using FwdRing = typename FwdRingT<BF16, TPW, DEPTH>::type;

template <int TPW, int SD>
__device__ __forceinline__ void split_ring_load(BRing<true, 2 * TPW, SD>& r, int slot, const Weights& B, int KB,
                                                int kb, int nb0, int nbs, int NB) {
  const int lane = frag_lane(nb0, KB);
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (has_block(i, nb0, nbs, NB) && kb < KB) {
      r.b[slot][i] = frag_bf16<TPW>(B.h, lane, i * nbs, KB, kb);
      r.b[slot][TPW + i] = frag_bf16<TPW>(B.m, lane, i * nbs, KB, kb);
    }
  }
}

// first k-steps of a forward product: two-part fragments (BF16) or three-part ones
template <bool BF16, int TPW, int DEPTH>
__device__ __forceinline__ void fwd_ring_fill(FwdRing<BF16, TPW, DEPTH>& r, const Weights& B, int K, int nb0, int nbs,
                                              int NB) {
  if constexpr (BF16) {
    constexpr int SD = DEPTH / 2 > 0 ? DEPTH / 2 : 1;
#pragma unroll
    for (int s = 0; s < SD; ++s) split_ring_load<TPW, SD>(r, s, B, K / 32, s, nb0, nbs, NB);
  } else {
    ring_fill(r, B, K, nb0, nbs, NB);
  }
}

// acc += A B for a forward product: split-BF16 (bf16 parts of A at A and
// Alo) or FP32 (A; Alo unused)
template <bool BF16, int TPW, int DEPTH>
__device__ __forceinline__ void fwd_mma(FwdRing<BF16, TPW, DEPTH>& r, const void* A, const void* Alo, int lda, int rb,
                                        const Weights& B, int K, int nb0, int nbs, int NB,
                                        floatx4 (&acc)[TPW]) {
  if constexpr (BF16) {
    constexpr int SD = DEPTH / 2 > 0 ? DEPTH / 2 : 1;
    const int l = threadIdx.x & 63;
    const int KB = K / 32;
    const int aoff = (rb * 16 + (l & 15)) * lda + (l >> 4) * 8;
    const __bf16* ahi = (const __bf16*)A + aoff;
    const __bf16* alo_p = (const __bf16*)Alo + aoff;
    auto step = [&](int slot, int kb) {
      const bf16x8 ah = *(const bf16x8*)(ahi + kb * 32);
      const bf16x8 al = *(const bf16x8*)(alo_p + kb * 32);
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        if (!has_block(i, nb0, nbs, NB)) continue;
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, r.b[slot][i], acc[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, r.b[slot][TPW + i], acc[i], 0, 0, 0);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, r.b[slot][i], acc[i], 0, 0, 0);
      }
    };
    auto load = [&](int slot, int kb) { split_ring_load<TPW, SD>(r, slot, B, KB, kb, nb0, nbs, NB); };
    if (NB < nbs) pipeline<SD, 4>(KB, step, load);
    else pipeline<SD>(KB, step, load);
  } else {
    mma_ring(r, A, lda, rb, B, K, nb0, nbs, NB, acc);
  }
}

// store of a forward activation: FP32 (base), or its bf16 high part (base)
// and low part (lo, same layout)
template <bool BF16>
__device__ inline void st_split(void* base, void* lo, int idx, float v) {
  if constexpr (BF16) {
    const __bf16 h = (__bf16)v;
    ((__bf16*)base)[idx] = h;
    ((__bf16*)lo)[idx] = (__bf16)split_low(v, h);
  } else {
    ((float*)base)[idx] = v;
  }
}

template <int TPW>
__device__ inline void zero_acc(floatx4 (&acc)[TPW]) {
#pragma unroll
  for (int i = 0; i < TPW; ++i) acc[i] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
}

// swish(z) = z sigmoid(z) and its derivative; the sigmoid takes the hardware
// reciprocal (1 ulp) instead of a correctly rounded division, a ten-
// instruction sequence per activation in the VALU-bound network epilogues
__device__ inline float swish_parts(float z, float& dsw) {
  const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-z));
  dsw = s * (1.0f + z * (1.0f - s));
  return z * s;
}

template <bool BF16>
__device__ inline void st_act(void* base, int idx, float v) {
  if (BF16) ((__bf16*)base)[idx] = (__bf16)v;
  else ((float*)base)[idx] = v;
}

// LDS row strides of the network tiles (elements)
template <int HP, bool BF16>
struct NetStrides {
  static constexpr int G = BF16 ? (kFP + 8) : (kFP + 4);   // invariants (A of the first product)
  static constexpr int H = BF16 ? (HP + 8) : (HP + 4);     // h1 / delta2 / delta1
  static constexpr int GB = kFP + 1;                       // dE/dG (FP32)
};

template <int TM, int HP, int NW>
struct NetShape {
  static constexpr int MB = TM / 16;                 // 16-row blocks
  static constexpr int WPR = NW / MB;                // waves per row block
  static constexpr int NBH = HP / 16;                // 16-column blocks of a hidden layer
  static constexpr int NBG = kFP / 16;               // ... of the invariants
  static constexpr int TPW = (NBH + WPR - 1) / WPR;  // column blocks per wave (hidden)
  static constexpr int TPW_G = (NBG + WPR - 1) / WPR;
};

// Network forward for the TM rows of a tile (all NW waves):
//   z1 = G W1 + b1, h1 = swish(z1); z2 = h1 W2 + b2, h2 = swish(z2);
//   y_m = h2 . W3[:,m] + b3[m], E_m = sigma y_m + mu  (written for rows < n_rows,
//   also to sEa[row][m] in LDS when sEa is not null)
// sG: invariants (read).  sH: h1 out.  swish'(z1) is returned in dsw1 (the
// backward product hands each wave exactly these output fragments again).
// MEAN: delta2 = swish'(z2) sigma mean_m W3[:,m] -> sD2 (the head-mean
// backward); otherwise swish'(z2) -> sDsw2 (FP32, row stride HP + 1) for
// per-head backwards.  sEp: [NW][16][kMaxHeads] partial sums.
// BF16 mode: both forward products are split-BF16 (fwd_mma), with the low
// parts of G at sGlo and of h1 at sHlo; fring holds the first k-steps of W1
// on entry.  sHlo may overlap sG and sD2 (the tile keeps h1's low part where
// G was and delta2 goes): barriers after each forward product's MFMAs keep
// those stores behind every wave's reads.  The backward products stay plain
// BF16: the first k-steps of W2^T are issued into `ring` before the second
// epilogue.
template <int TM, int HP, bool BF16, int NW, bool MEAN, int DEPTH>
__device__ __forceinline__ void network_forward(const DevModel& m, const void* sG, const void* sGlo, void* sH,
                                       void* sHlo, void* sD2, float* sDsw2,
                                       float* sEp, const float* sScale, const float* sShift, const int* sStruct,
                                       int row0, int n_rows,
                                       float* __restrict__ atomic_e, float* sEa,
                                       floatx4 (&dsw1)[NetShape<TM, HP, NW>::TPW],
                                       FwdRing<BF16, NetShape<TM, HP, NW>::TPW, DEPTH>& fring,
                                       BRing<BF16, NetShape<TM, HP, NW>::TPW, DEPTH>& ring) {
  using St = NetStrides<HP, BF16>;
  using Sh = NetShape<TM, HP, NW>;
  constexpr int MB = Sh::MB, WPR = Sh::WPR, NBH = Sh::NBH, TPW = Sh::TPW;
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63;
  const int rb = w % MB, cw = w / MB;
  const int M = m.M;
  // per-column epilogue constants of this wave, loaded ahead of the products
  float b1v[TPW], b2v[TPW], wbv[TPW], w30[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int nb = cw + i * WPR;
    const int col = (nb < NBH ? nb : 0) * 16 + (l & 15);
    b1v[i] = m.b1[col];
    b2v[i] = m.b2[col];
    wbv[i] = m.w3bar[col];
    w30[i] = m.w3[col * M];
  }
  {
    floatx4 acc[TPW];
    zero_acc(acc);
    fwd_mma<BF16, TPW, DEPTH>(fring, sG, sGlo, St::G, rb, m.w1, kFP, cw, WPR, NBH, acc);
    fwd_ring_fill<BF16, TPW, DEPTH>(fring, m.w2, HP, cw, WPR, NBH);
    if (BF16) __syncthreads();  // every wave is done with G before h1's low part is stored
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = cw + i * WPR;
      if (nb >= NBH) continue;
      const int col = nb * 16 + (l & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (l >> 4) + j;
        float d;
        const float hv = swish_parts(acc[i][j] + b1v[i], d);
        dsw1[i][j] = d;
        st_split<BF16>(sH, sHlo, row * St::H + col, hv);
      }
    }
  }
  __syncthreads();
  {
    floatx4 acc[TPW];
    zero_acc(acc);
    fwd_mma<BF16, TPW, DEPTH>(fring, sH, sHlo, St::H, rb, m.w2, HP, cw, WPR, NBH, acc);
    // the backward's first product (W2^T) starts loading now
    ring_fill(ring, m.w2t, HP, cw, WPR, NBH);
    if (BF16) __syncthreads();  // every wave is done with h1's low part before delta2 is stored
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = cw + i * WPR;
      if (nb >= NBH) continue;
      const int col = nb * 16 + (l & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (l >> 4) + j;
        float d;
        const float hv = swish_parts(acc[i][j] + b2v[i], d);
        acc[i][j] = hv;
        if (m.h2_out && row < n_rows) m.h2_out[(int64_t)(row0 + row) * HP + col] = hv;
        if (MEAN)
          st_act<BF16>(sD2, row * St::H + col,
                       d * sScale[row] * (m.head_w ? m.head_w[(int64_t)sStruct[row] * HP + col] : wbv[i]));
        else sDsw2[row * (HP + 1) + col] = d;
      }
    }
    for (int hm = 0; hm < M; ++hm) {
      float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int i = 0; i < TPW; ++i) {
        const int nb = cw + i * WPR;
        if (nb >= NBH) continue;
        const float w3 = hm == 0 ? w30[i] : m.w3[(nb * 16 + (l & 15)) * M + hm];
#pragma unroll
        for (int j = 0; j < 4; ++j) part[j] += acc[i][j] * w3;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float v = part[j];
        v = row16_rot_sum(v);  // lane 0 of the row: the xor-butterfly sum
        if ((l & 15) == 0) sEp[(w * 16 + 4 * (l >> 4) + j) * kMaxHeads + hm] = v;
      }
    }
  }
  __syncthreads();
  for (int t = tid; t < TM * M; t += NW * 64) {
    const int a = t / M, hm = t % M;
    if (a < n_rows) {
      float y = m.b3[hm];
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
        if (ww % MB == a / 16) y += sEp[(ww * 16 + a % 16) * kMaxHeads + hm];
      const float e = sScale[a] * y + sShift[a];
      atomic_e[(int64_t)(row0 + a) * M + hm] = e;
      if (sEa) sEa[a * M + hm] = e;
    }
  }
}

// delta2 of head `hm`: swish'(z2) sigma W3[:,hm] -> sD2
template <int TM, int HP, bool BF16, int NW>
__device__ __forceinline__ void network_delta2_head(const DevModel& m, const float* sDsw2, const float* sScale, void* sD2,
                                           int hm) {
  using St = NetStrides<HP, BF16>;
  for (int t = threadIdx.x; t < TM * HP; t += NW * 64) {
    const int row = t / HP, col = t % HP;
    st_act<BF16>(sD2, row * St::H + col, sDsw2[row * (HP + 1) + col] * sScale[row] * m.w3[col * m.M + hm]);
  }
}

// Network backward given delta2 in sD2 and the ring holding the first k-steps
// of W2^T: delta1 = swish'(z1) (delta2 W2^T) -> sH, dE/dG = delta1 W1^T ->
// sGb (FP32).  Ends with a barrier.
template <int TM, int HP, bool BF16, int NW, int DEPTH>
__device__ __forceinline__ void network_backward(const DevModel& m, const void* sD2, void* sH, float* sGb,
                                        const floatx4 (&dsw1)[NetShape<TM, HP, NW>::TPW],
                                        BRing<BF16, NetShape<TM, HP, NW>::TPW, DEPTH>& ring) {
  using St = NetStrides<HP, BF16>;
  using Sh = NetShape<TM, HP, NW>;
  constexpr int MB = Sh::MB, WPR = Sh::WPR, NBH = Sh::NBH, NBG = Sh::NBG, TPW = Sh::TPW, TPW_G = Sh::TPW_G;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int rb = w % MB, cw = w / MB;
  BRing<BF16, TPW_G, (DEPTH < prefetch_depth<TPW_G>() ? DEPTH : prefetch_depth<TPW_G>())> ring_g;
  {
    floatx4 acc[TPW];
    zero_acc(acc);
    mma_ring(ring, sD2, St::H, rb, m.w2t, HP, cw, WPR, NBH, acc);
    ring_fill(ring_g, m.w1t, HP, cw, WPR, NBG);
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      const int nb = cw + i * WPR;
      if (nb >= NBH) continue;
      const int col = nb * 16 + (l & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (l >> 4) + j;
        st_act<BF16>(sH, row * St::H + col, acc[i][j] * dsw1[i][j]);
      }
    }
  }
  __syncthreads();
  {
    floatx4 acc[TPW_G];
    zero_acc(acc);
    mma_ring(ring_g, sH, St::H, rb, m.w1t, HP, cw, WPR, NBG, acc);
#pragma unroll
    for (int i = 0; i < TPW_G; ++i) {
      const int nb = cw + i * WPR;
      if (nb >= NBG) continue;
      const int col = nb * 16 + (l & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + 4 * (l >> 4) + j;
        sGb[row * St::GB + col] = acc[i][j];
      }
    }
  }
  __syncthreads();
}

}  // namespace gmnn
