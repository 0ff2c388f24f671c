// Batch selection by last-layer gradient features (Section 2.4):
//
//   ll_features     phi(S) = gradient of the structure's head-mean energy
//                   w.r.t. one head's last-layer weights and bias (eq.
//                   lastlayer): (1/M) [sum_i sigma_Zi h2_i ; sum_i sigma_Zi],
//                   summed per structure in FP64 in atom order (the other
//                   heads' blocks of the full gradient are equal copies)
//   selection       greedy maximum-distance selection (eq. maxdist): each
//                   step picks the pool structure whose smallest distance to
//                   the training set and the structures picked so far is
//                   largest; distances in FP64, ties to the smallest index,
//                   entries without a distance (NaN) last.
//                   One launch per pick: every block finds the pick from the
//                   previous launch's block maxima, takes the distances of
//                   its rows to it, and leaves its own maximum.
//
// What bounds a pick: the launch and one round trip of the rows (a distance
// is one FP64 chain over the features, in feature order, so that picks do not
// depend on the launch shape; 257 features take 0.9 us).  Rows go through LDS
// in coalesced loads, all in flight.  300 rows of 257: 42 us in three
// launches before, 9 us now.
#include "common.h"
#include "model.h"

namespace gmnn {

// block b: structure b; thread c <= H2: column c of h2, or the bias entry at
// c = H2 -- columns H2 .. HP2 of h2 are padding and skipped.  Atoms are added
// in order; eight of them are loaded at a time.
__global__ void __launch_bounds__(1024) ll_features(DevModel m, DevSystem sys, int H2, const float* __restrict__ h2,
                                                    double* __restrict__ phi) {
  const int b = blockIdx.x;
  const int64_t a0 = sys.atom_ptr[b], a1 = sys.atom_ptr[b + 1];
  const double invM = 1.0 / (double)m.M;
  for (int c = threadIdx.x; c <= H2; c += blockDim.x) {
    double acc = 0.0;
    const float* col = h2 + (c < H2 ? c : 0);
    int64_t i = a0;
    for (; i + 8 <= a1; i += 8) {
      float v[8], sg[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sg[u] = m.scale[sys.species[i + u]];
        v[u] = col[(i + u) * m.HP2];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += c < H2 ? (double)sg[u] * (double)v[u] : (double)sg[u];
    }
    for (; i < a1; ++i) {
      const double sg = (double)m.scale[sys.species[i]];
      acc += c < H2 ? sg * (double)col[i * m.HP2] : sg;
    }
    phi[(int64_t)b * (H2 + 1) + c] = acc * invM;
  }
}

constexpr int kSelBlock = 256;   // threads
constexpr int kSelRows = 16;     // pool rows staged at a time
constexpr int kSelDims = 288;    // features staged at a time (257 of a 2x256 network in one go, 513 of 2x512 in two)
constexpr int kSelLd = kSelDims + 1;
constexpr int kSelPer = kSelRows * kSelDims / kSelBlock;  // values a thread stages
constexpr int kSelMaxBlocks = 512;

static int64_t sel_blocks(int64_t n) {
  const int64_t nb = (n + kSelRows - 1) / kSelRows;
  return nb < kSelMaxBlocks ? nb : kSelMaxBlocks;
}

// rows [r0, r0 + nr) x features [k0, k0 + nk) of a row-major array: every load
// in flight, then into LDS
struct SelTile {
  double v[kSelPer];
  __device__ inline void load(const double* __restrict__ x, int64_t r0, int nr, int D, int k0, int nk) {
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
      const int t = threadIdx.x + u * kSelBlock, r = t / kSelDims, k = t % kSelDims;
      v[u] = r < nr && k < nk ? x[(r0 + r) * D + k0 + k] : 0.0;
    }
  }
  __device__ inline void store(double* __restrict__ dst) const {
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
      const int t = threadIdx.x + u * kSelBlock;
      dst[t / kSelDims * kSelLd + t % kSelDims] = v[u];
    }
  }
};

struct Best {
  double v;
  int64_t i;
};
__device__ inline Best better(Best a, Best b) { return b.v > a.v || (b.v == a.v && b.i < a.i) ? b : a; }
// the block's best entry (ties to the smallest index), for every thread
__device__ inline Best block_best(Best x, Best* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = better(x, Best{__shfl_xor(x.v, o), __shfl_xor(x.i, o)});
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  x = red[0];
  for (int w = 1; w < kSelBlock / 64; ++w) x = better(x, red[w]);
  return x;
}

// INIT: mind[i], the smallest squared distance of pool entry i to the training
// set (or its squared norm when the training set is empty: the first pick is
// then the entry farthest from the origin).  Otherwise step `step`: the pick
// from the previous launch's block maxima, which leaves the pool (-1), and
// every minimum now covers it (replace: the first pick without a training set;
// the norms that chose it are no distances to a selected entry).  Both leave
// the block maxima of mind.
template <bool INIT>
__global__ void __launch_bounds__(kSelBlock) sel_step(const double* __restrict__ pool, int64_t n, int D,
                                                      const double* __restrict__ train, int64_t nt,
                                                      const Best* __restrict__ prev, Best* __restrict__ next,
                                                      int step, int replace, int32_t* __restrict__ selected,
                                                      double* __restrict__ mind) {
  __shared__ double s_rows[kSelRows * kSelLd];
  __shared__ double s_tgt[(INIT ? kSelRows : 1) * kSelLd];
  __shared__ double s_min[INIT ? kSelRows * kSelRows : 1];
  __shared__ Best s_red[kSelBlock / 64];
  const int tid = threadIdx.x;
  int64_t pick = -1;
  // the first rows are under way while the pick is found
  SelTile rows, tgt;
  const int64_t first = (int64_t)blockIdx.x * kSelRows;
  rows.load(pool, first, (int)(n - first < kSelRows ? n - first : kSelRows), D, 0, min(kSelDims, D));
  if (!INIT) {
    Best x{-3.0, INT64_MAX};
    for (int p = tid; p < (int)gridDim.x; p += kSelBlock) x = better(x, prev[p]);
    pick = block_best(x, s_red).i;
    if (blockIdx.x == 0 && tid == 0) selected[step] = (int32_t)pick;
  }
  // INIT with a training set: thread (row r, target q) of 16 x 16; else one
  // thread per row
  const bool grid2 = INIT && nt > 0;
  const int r = tid % kSelRows, q = tid / kSelRows;
  Best best{-2.0, INT64_MAX};
  for (int64_t r0 = (int64_t)blockIdx.x * kSelRows; r0 < n; r0 += (int64_t)gridDim.x * kSelRows) {
    const int nr = (int)(n - r0 < kSelRows ? n - r0 : kSelRows);
    const bool mine = r < nr && (grid2 || q == 0);
    double low = 0.0;
    bool have = false;
    for (int64_t t0 = 0; t0 < (grid2 ? nt : 1); t0 += kSelRows) {
      const int nq = grid2 ? (int)(nt - t0 < kSelRows ? nt - t0 : kSelRows) : 1;
      double s = 0.0;
      for (int k0 = 0; k0 < D; k0 += kSelDims) {
        const int nk = min(kSelDims, D - k0);
        if (r0 != first || t0 > 0 || k0 > 0) rows.load(pool, r0, nr, D, k0, nk);
        if (grid2) tgt.load(train, t0, nq, D, k0, nk);
        double pv[2];
        if (!INIT)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int k = tid + u * kSelBlock;
            pv[u] = k < nk ? pool[pick * D + k0 + k] : 0.0;
          }
        __syncthreads();  // the previous use of the staged rows is over
        rows.store(s_rows);
        if (grid2) tgt.store(s_tgt);
        if (!INIT)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (tid + u * kSelBlock < kSelDims) s_tgt[tid + u * kSelBlock] = pv[u];
        __syncthreads();
        if (mine && q < nq) {
          const double* a = s_rows + r * kSelLd;
          const double* b = s_tgt + q * kSelLd;
          if (INIT && !grid2) {
#pragma unroll 8
            for (int k = 0; k < nk; ++k) s += a[k] * a[k];
          } else {
#pragma unroll 8
            for (int k = 0; k < nk; ++k) {
              const double d = a[k] - b[k];
              s += d * d;
            }
          }
        }
      }
      if (q < nq) {
        low = have ? fmin(low, s) : s;
        have = true;
      }
    }
    if (INIT && grid2) {
      // over the targets of each row (fmin is exact in any order)
      __syncthreads();
      s_min[q * kSelRows + r] = low;
      __syncthreads();
      if (q == 0)
        for (int p = 1; p < (int)(nt < kSelRows ? nt : kSelRows); ++p) low = fmin(low, s_min[p * kSelRows + r]);
    }
    if (q == 0 && r < nr) {
      const int64_t i = r0 + r;
      double v = low;
      if (!INIT) {
        const double m = mind[i];
        v = m < 0.0 ? m : i == pick ? -1.0 : replace ? low : fmin(m, low);
      }
      mind[i] = v;
      // a NaN compares with nothing, which would leave a pool of them without a
      // valid pick: it counts below every distance (the larger of it and a
      // number is the number)
      if (!(v < 0.0)) best = better(best, Best{fmax(v, -0.5), i});
    }
  }
  best = block_best(best, s_red);
  if (tid == 0) next[blockIdx.x] = best;
}

}  // namespace gmnn

using namespace gmnn;

extern "C" {

size_t gmnn_select_workspace_bytes(int64_t n_pool) {
  if (n_pool < 1) return 0;
  // minima, and the block maxima of two launches
  return (size_t)(8 * n_pool + 2 * (int64_t)sizeof(Best) * sel_blocks(n_pool) + 64 + 255) & ~size_t(255);
}

gmnn_status gmnn_select_max_distance(const double* pool, int64_t n_pool, int32_t dim, const double* train,
                                     int64_t n_train, int32_t n_select, int32_t* selected, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  if (!pool || n_pool < 1 || dim < 1 || n_train < 0 || (n_train > 0 && !train) || n_select < 0 ||
      n_select > n_pool || (n_select > 0 && !selected) || !workspace)
    return GMNN_ERR_INVALID_ARG;
  if (workspace_bytes < gmnn_select_workspace_bytes(n_pool)) return GMNN_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const int64_t nb = sel_blocks(n_pool);
  double* mind = (double*)workspace;
  Best* part[2] = {(Best*)(mind + n_pool), (Best*)(mind + n_pool) + nb};
  const dim3 grid((unsigned)nb), block(kSelBlock);
  hipLaunchKernelGGL(sel_step<true>, grid, block, 0, s, pool, n_pool, dim, train, n_train, (const Best*)nullptr,
                     part[0], 0, 0, (int32_t*)nullptr, mind);
  for (int k = 0; k < n_select; ++k)
    hipLaunchKernelGGL(sel_step<false>, grid, block, 0, s, pool, n_pool, dim, (const double*)nullptr, (int64_t)0,
                       (const Best*)part[k & 1], part[(k + 1) & 1], k, (k == 0 && n_train == 0) ? 1 : 0, selected,
                       mind);
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

}  // extern "C"
