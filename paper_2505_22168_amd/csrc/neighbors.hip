// Periodic cell-list neighbour search (gfx950).
//
// The potential sums over every neighbour j != i of atom i inside the cutoff
// (Section 2.1, eq. basis_fn); periodic cells narrower than twice the cutoff
// hold several images of one neighbour (Section 3.5), so the search enumerates
// as many cell images as the cell width requires instead of the minimum
// image.  The list is canonical (rows by i, inside a row by (j, Sx, Sy, Sz)),
// so it is bit-identical whatever order the atoms land in their cells.
//
// Kernels (one build = 8 launches, 2 more above kScanOne elements a scan, all
// on the caller's stream):
//   nl_setup     one block: per-structure cell grid, cell offsets, clears
//   nl_bin       thread/atom: fractional coords, image, cell, cell counts
//   scan         cell counts -> cell starts
//   nl_cellfill  thread/atom: positions and images into cell order
//   nl_rows<0>   wave/atom: count neighbours (FP64 inclusion test)
//   scan         row counts -> row_ptr, n_pairs
//   nl_rows<1>   wave/atom: collect, rank-sort in LDS, write the row
//   nl_reverse   wave/atom: index of the reverse pair, guessed, then searched
//
// What bounds it.  The 11.0M pairs of the 100k solid are 135 MB of output,
// about 30 us; the build is bound by its candidates (instructions per tested
// pair, dependent loads) and by the lanes' scattered loads of the reverse
// search.  Cells of half the list radius (125 of them hold 430 candidates per
// atom at that density, 27 whole ones 740) and candidates stored in cell
// order, so that a run of cells along the third axis is one contiguous read,
// took the two row passes from 433 and 622 us to 207 and 323 us (with the
// 32-bit rank sort); the mirrored first guess of the reverse search (45% of
// the pairs of a jittered lattice) took it from 456 to 255 us, the scans from
// 94 to 9 us.  The build: 1.77 -> 0.85 ms.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "neighbors.h"

namespace gmnn {

// ---------------------------------------------------------------------------
// per-structure grid (device)
// ---------------------------------------------------------------------------
__host__ __device__ inline int cells_on_axis(double x) {
  const double f = floor(x);
  return f < 1.0 ? 1 : f > (double)kMaxCellsPerAxis ? kMaxCellsPerAxis : (int)f;
}
// a structure takes the fine grid while its cells stay within a few per atom
// (clearing and scanning the cells of a mostly empty box would cost more than
// the candidates saved)
__host__ __device__ inline long long max_fine_cells(int64_t n_atoms) { return 8 * (long long)n_atoms + 1024; }

__device__ inline void grid_of_structure(const double* h, const uint8_t* pbc, double rbin, int64_t n_atoms,
                                         StructGrid& g) {
  for (int k = 0; k < 9; ++k) g.h[k] = h[k];
  // inverse of the row-vector lattice: frac_k = sum_c x_c inv[c][k]
  const double a00 = h[0], a01 = h[1], a02 = h[2];
  const double a10 = h[3], a11 = h[4], a12 = h[5];
  const double a20 = h[6], a21 = h[7], a22 = h[8];
  const double c00 = a11 * a22 - a12 * a21, c01 = a12 * a20 - a10 * a22, c02 = a10 * a21 - a11 * a20;
  const double c10 = a02 * a21 - a01 * a22, c11 = a00 * a22 - a02 * a20, c12 = a01 * a20 - a00 * a21;
  const double c20 = a01 * a12 - a02 * a11, c21 = a02 * a10 - a00 * a12, c22 = a00 * a11 - a01 * a10;
  const double det = a00 * c00 + a01 * c01 + a02 * c02;
  const double id = 1.0 / det;
  // inv = adj / det with adj[c][k] = cofactor[k][c]
  g.inv[0] = c00 * id; g.inv[1] = c10 * id; g.inv[2] = c20 * id;
  g.inv[3] = c01 * id; g.inv[4] = c11 * id; g.inv[5] = c21 * id;
  g.inv[6] = c02 * id; g.inv[7] = c12 * id; g.inv[8] = c22 * id;
  const double vol = fabs(det);
  const double cr[3][3] = {{c00, c01, c02}, {c10, c11, c12}, {c20, c21, c22}};
  double width[3];
  for (int k = 0; k < 3; ++k) {
    // |h_{k+1} x h_{k+2}| = |cofactor row k|; width = vol / that
    const double nrm = sqrt(cr[k][0] * cr[k][0] + cr[k][1] * cr[k][1] + cr[k][2] * cr[k][2]);
    width[k] = vol / nrm;
  }
  long long cells = 1;
  for (int k = 0; k < 3; ++k) cells *= cells_on_axis(kCellsPerRadius * width[k] / rbin);
  const double fine = cells <= max_fine_cells(n_atoms) ? kCellsPerRadius : 1.0;
  cells = 1;
  for (int k = 0; k < 3; ++k) {
    const int nc = cells_on_axis(fine * width[k] / rbin);
    int m = (int)ceil(rbin * (double)nc / width[k]);
    if (m < 1) m = 1;
    g.nc[k] = nc;
    g.m[k] = m;
    g.pbc[k] = pbc[k] ? 1 : 0;
    cells *= nc;
  }
  g.n_cells = (int)cells;
}

// disp_bits (optional): the largest squared displacement since the last
// build (float bits); the build runs only if it exceeds thresh2 (the go flag
// every later kernel of the build checks)
__global__ void __launch_bounds__(1024) nl_setup(const double* __restrict__ cell, const uint8_t* __restrict__ pbc,
                                                 const int64_t* __restrict__ atom_ptr, int n_structs, double rbin, StructGrid* __restrict__ grids,
                                                 int64_t cell_capacity, int32_t* __restrict__ cell_count,
                                                 int32_t* __restrict__ cell_fill, int64_t* __restrict__ n_cells_total,
                                                 uint32_t* __restrict__ status, const uint32_t* __restrict__ disp_bits,
                                                 float thresh2, int* __restrict__ go) {
  __shared__ int64_t run;
  __shared__ int64_t part[1024];
  __shared__ int s_go;
  const int t = threadIdx.x;
  if (t == 0) {
    const int g = disp_bits ? (__uint_as_float(*disp_bits) > thresh2 ? 1 : 0) : 1;
    *go = g;
    s_go = g;
    run = 0;
    if (g) *status = 0u;
  }
  __syncthreads();
  if (!s_go) return;
  for (int b0 = 0; b0 < n_structs; b0 += 1024) {
    const int b = b0 + t;
    StructGrid g;
    int64_t nc = 0;
    if (b < n_structs) {
      grid_of_structure(cell + 9 * (int64_t)b, pbc + 3 * (int64_t)b, rbin, atom_ptr[b + 1] - atom_ptr[b], g);
      nc = g.n_cells;
    }
    part[t] = nc;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      int64_t v = (t >= o) ? part[t - o] : 0;
      __syncthreads();
      part[t] += v;
      __syncthreads();
    }
    if (b < n_structs) {
      g.cell_offset = run + part[t] - nc;
      grids[b] = g;
    }
    __syncthreads();
    if (t == 1023) run += part[1023];
    __syncthreads();
  }
  const int64_t total = run;
  if (t == 0) {
    *n_cells_total = total;
    if (total > cell_capacity) raise_flag(status, GMNN_FLAG_CAPACITY);
  }
  const int64_t lim = total < cell_capacity ? total : cell_capacity;
  for (int64_t c = t; c < lim; c += 1024) {
    cell_count[c] = 0;
    cell_fill[c] = 0;
  }
}

__device__ inline int find_struct(const int64_t* __restrict__ atom_ptr, int n_structs, int64_t i) {
  int lo = 0, hi = n_structs - 1;  // largest b with atom_ptr[b] <= i
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (atom_ptr[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ void nl_bin(const float* __restrict__ pos, const int64_t* __restrict__ atom_ptr, int n_structs,
                       int n_atoms, const StructGrid* __restrict__ grids, const int64_t* __restrict__ n_cells_total,
                       int64_t cell_capacity, int32_t* __restrict__ atom_struct, int32_t* __restrict__ atom_cell,
                       int4* __restrict__ atom_img, int32_t* __restrict__ cell_count, uint32_t* __restrict__ status,
                       const int* __restrict__ go, float* __restrict__ ref_pos) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_atoms) return;
  if (!*go) return;
  if (ref_pos) {
    ref_pos[3 * (int64_t)i] = pos[3 * (int64_t)i];
    ref_pos[3 * (int64_t)i + 1] = pos[3 * (int64_t)i + 1];
    ref_pos[3 * (int64_t)i + 2] = pos[3 * (int64_t)i + 2];
  }
  if (*n_cells_total > cell_capacity) return;
  const int b = find_struct(atom_ptr, n_structs, i);
  atom_struct[i] = b;
  const StructGrid& g = grids[b];
  const double x[3] = {(double)pos[3 * (int64_t)i], (double)pos[3 * (int64_t)i + 1], (double)pos[3 * (int64_t)i + 2]};
  int img[3], cc[3];
  bool bad = false;
  for (int k = 0; k < 3; ++k) {
    const double f = x[0] * g.inv[0 * 3 + k] + x[1] * g.inv[1 * 3 + k] + x[2] * g.inv[2 * 3 + k];
    if (!isfinite(f) || fabs(f) > 1.0e6) {
      bad = true;
      img[k] = 0;
      cc[k] = 0;
      continue;
    }
    double w = f;
    int n = 0;
    if (g.pbc[k]) {
      const double fl = floor(f);
      n = (int)fl;
      w = f - fl;
    }
    int c = (int)floor(w * (double)g.nc[k]);
    c = c < 0 ? 0 : (c >= g.nc[k] ? g.nc[k] - 1 : c);
    img[k] = n;
    cc[k] = c;
  }
  if (bad) raise_flag(status, GMNN_FLAG_NONFINITE);
  const int cid = g.cell_offset + (cc[0] * g.nc[1] + cc[1]) * g.nc[2] + cc[2];
  atom_cell[i] = cid;
  atom_img[i] = make_int4(img[0], img[1], img[2], (cc[0] << 20) | (cc[1] << 10) | cc[2]);
  atomicAdd(&cell_count[cid], 1);
}

// ---------------------------------------------------------------------------
// Exclusive scans of int32 counts into int64 offsets (n + 1 entries).  n_dev
// (if given) is clamped to n_host, the length of `in`.  cap >= 0: offsets
// beyond the pair capacity would send the pair kernels past the list arrays,
// so an overflowing list is left empty (the total still reports the size
// needed, and the capacity flag is raised later).  Up to kScanOne elements
// one block walks over them (a launch less); above, every block of
// kScanTile elements is summed first, and then scanned behind the sum of the
// blocks before it.
constexpr int kScanThreads = 1024;
constexpr int kScanTile = 4 * kScanThreads;
constexpr int64_t kScanOne = 4 * kScanTile;

__device__ inline int64_t scan_length(const int64_t* n_dev, int64_t n_host) {
  return n_dev && *n_dev < n_host ? *n_dev : n_host;
}
__device__ inline int4 scan_load(const int32_t* __restrict__ in, int64_t e, int64_t n) {
  int4 v = {0, 0, 0, 0};
  if (e + 4 <= n) return *(const int4*)(in + e);
  if (e < n) v.x = in[e];
  if (e + 1 < n) v.y = in[e + 1];
  if (e + 2 < n) v.z = in[e + 2];
  return v;
}
// exclusive prefix of v over the block's threads; total: the block's sum
__device__ inline int block_prefix(int v, int* sums, int& total) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int incl = wave_incl_scan(v);
  __syncthreads();  // the previous use of sums is read
  if (l == 63) sums[w] = incl;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int k = 0; k < kScanThreads / 64; ++k) {
    if (k < w) before += sums[k];
    total += sums[k];
  }
  return before + incl - v;
}
__device__ inline void scan_store(int64_t* __restrict__ out, int64_t e, int64_t n, int64_t base, int4 v, bool zero) {
  const int64_t o[4] = {base, base + v.x, base + v.x + v.y, base + v.x + v.y + v.z};
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (e + k < n) out[e + k] = zero ? 0 : o[k];
}

__global__ void __launch_bounds__(kScanThreads) scan_one(const int32_t* __restrict__ in, int64_t* __restrict__ out,
                                                         const int64_t* __restrict__ n_dev, int64_t n_host,
                                                         int64_t* __restrict__ total, const int* __restrict__ go,
                                                         int64_t cap) {
  if (!*go) return;
  __shared__ int sums[kScanThreads / 64];
  const int64_t n = scan_length(n_dev, n_host);
  int64_t base = 0;
  for (int64_t t0 = 0; t0 < n; t0 += kScanTile) {
    const int64_t e = t0 + 4 * (int64_t)threadIdx.x;
    const int4 v = scan_load(in, e, n);
    int sum;
    const int before = block_prefix(v.x + v.y + v.z + v.w, sums, sum);
    scan_store(out, e, n, base + before, v, false);
    base += sum;
  }
  const bool over = cap >= 0 && base > cap;
  if (over) {
    __syncthreads();
    for (int64_t k = threadIdx.x; k < n; k += kScanThreads) out[k] = 0;
  }
  if (threadIdx.x == 0) {
    out[n] = over ? 0 : base;
    if (total) *total = base;
  }
}

__global__ void __launch_bounds__(kScanThreads) scan_sums(const int32_t* __restrict__ in,
                                                          const int64_t* __restrict__ n_dev, int64_t n_host,
                                                          int32_t* __restrict__ part, const int* __restrict__ go) {
  if (!*go) return;
  __shared__ int sums[kScanThreads / 64];
  const int64_t n = scan_length(n_dev, n_host);
  const int4 v = scan_load(in, (int64_t)blockIdx.x * kScanTile + 4 * (int64_t)threadIdx.x, n);
  int sum;
  (void)block_prefix(v.x + v.y + v.z + v.w, sums, sum);
  if (threadIdx.x == 0) part[blockIdx.x] = sum;
}

__global__ void __launch_bounds__(kScanThreads) scan_write(const int32_t* __restrict__ in, int64_t* __restrict__ out,
                                                           const int64_t* __restrict__ n_dev, int64_t n_host,
                                                           const int32_t* __restrict__ part,
                                                           int64_t* __restrict__ total, const int* __restrict__ go,
                                                           int64_t cap) {
  if (!*go) return;
  __shared__ int sums[kScanThreads / 64];
  __shared__ int64_t wide[2][kScanThreads / 64];
  const int64_t n = scan_length(n_dev, n_host);
  const int nb = gridDim.x;
  // the sums of the blocks before this one, and of all
  int64_t mine = 0, all = 0;
  for (int k = threadIdx.x; k < nb; k += kScanThreads) {
    const int64_t x = part[k];
    all += x;
    if (k < (int)blockIdx.x) mine += x;
  }
  mine = wave_sum(mine);
  all = wave_sum(all);
  if ((threadIdx.x & 63) == 0) {
    wide[0][threadIdx.x >> 6] = mine;
    wide[1][threadIdx.x >> 6] = all;
  }
  __syncthreads();
  int64_t base = 0, sum_all = 0;
  for (int k = 0; k < kScanThreads / 64; ++k) {
    base += wide[0][k];
    sum_all += wide[1][k];
  }
  const bool over = cap >= 0 && sum_all > cap;
  const int64_t e = (int64_t)blockIdx.x * kScanTile + 4 * (int64_t)threadIdx.x;
  const int4 v = scan_load(in, e, n);
  int sum;
  const int before = block_prefix(v.x + v.y + v.z + v.w, sums, sum);
  scan_store(out, e, n, base + before, v, over);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    out[n] = over ? 0 : sum_all;
    if (total) *total = sum_all;
  }
}

// positions and images of the atoms in cell order: {x, y, z, atom} and the
// image (three ints); the order inside a cell is arbitrary (rows are sorted)
struct CellAtom {
  float x, y, z;
  int j;
};
__global__ void nl_cellfill(int n_atoms, const float* __restrict__ pos, const int32_t* __restrict__ atom_cell,
                            const int4* __restrict__ atom_img, const int64_t* __restrict__ cell_start,
                            const int64_t* __restrict__ n_cells_total, int64_t cell_capacity,
                            int32_t* __restrict__ cell_fill, CellAtom* __restrict__ cell_atoms,
                            int4* __restrict__ cell_img, const int* __restrict__ go) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_atoms) return;
  if (!*go) return;
  if (*n_cells_total > cell_capacity) return;
  const int c = atom_cell[i];
  const int64_t slot = cell_start[c] + atomicAdd(&cell_fill[c], 1);
  cell_atoms[slot] = CellAtom{pos[3 * (int64_t)i], pos[3 * (int64_t)i + 1], pos[3 * (int64_t)i + 2], i};
  cell_img[slot] = atom_img[i];
}

__device__ inline int floor_div(int a, int b) {
  int q = a / b;
  if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
  return q;
}

// FP64 inclusion test, every operation rounded once (no contraction), the
// same expression as the reference definition of the list.
__device__ inline double pair_d2(const double xi[3], const double xj[3], const double h[9], int sx, int sy, int sz) {
#pragma clang fp contract(off)
  const double fx = (double)sx, fy = (double)sy, fz = (double)sz;
  const double dx = (xj[0] - xi[0]) + ((fx * h[0] + fy * h[3]) + fz * h[6]);
  const double dy = (xj[1] - xi[1]) + ((fx * h[1] + fy * h[4]) + fz * h[7]);
  const double dz = (xj[2] - xi[2]) + ((fx * h[2] + fy * h[5]) + fz * h[8]);
  return (dx * dx + dy * dy) + dz * dz;
}

// the same without a shift: adding the zero shift to the separation rounds
// to the separation itself
__device__ inline double pair_d2_home(const double xi[3], const double xj[3]) {
#pragma clang fp contract(off)
  const double dx = xj[0] - xi[0], dy = xj[1] - xi[1], dz = xj[2] - xi[2];
  return (dx * dx + dy * dy) + dz * dz;
}

constexpr int kRowsWaves = 4;    // waves per block in nl_rows / nl_reverse
constexpr int kRowKeys = 512;    // keys of a row sorted in LDS; longer rows are sorted from the output arrays

// The candidates of atom i: runs of cells along the third axis, contiguous in
// cell order.  Run t of (2 m0 + 1)(2 m1 + 1) K: the column (o0, o1), and of
// the cells c2 - m2 .. c2 + m2 those in image s2_lo + t % K.
//
// MODE 0: count neighbours of every atom; MODE 1: collect, sort, write.
template <int MODE>
__global__ void __launch_bounds__(64 * kRowsWaves) __attribute__((amdgpu_waves_per_eu(5))) nl_rows(
    const float* __restrict__ pos, int n_atoms, const StructGrid* __restrict__ grids,
    const int32_t* __restrict__ atom_struct, const int4* __restrict__ atom_img,
    const int64_t* __restrict__ cell_start, const CellAtom* __restrict__ cell_atoms,
    const int4* __restrict__ cell_img, const int64_t* __restrict__ n_cells_total, int64_t cell_capacity, double rc2,
    int32_t* __restrict__ row_count, const int64_t* __restrict__ row_ptr, const int64_t* __restrict__ n_pairs,
    int64_t capacity, int32_t* __restrict__ out_j, int32_t* __restrict__ out_shift, uint32_t* __restrict__ status,
    const int* __restrict__ go) {
  __shared__ int s_excl[kRowsWaves][64];
  __shared__ int s_start[kRowsWaves][64];
  __shared__ int s_sw[kRowsWaves][64];
  __shared__ __attribute__((aligned(16))) uint64_t s_keys[MODE ? kRowsWaves : 1][MODE ? kRowKeys : 1];
  const int w = threadIdx.x >> 6;
  const int l = threadIdx.x & 63;
  const int i = xcd_block(blockIdx.x, gridDim.x) * kRowsWaves + w;
  if (i >= n_atoms) return;
  if (!*go) return;
  if (*n_cells_total > cell_capacity) return;
  if (MODE == 1 && *n_pairs > capacity) {
    if (i == 0 && l == 0) raise_flag(status, GMNN_FLAG_CAPACITY);
    return;
  }
  const int b = atom_struct[i];
  const StructGrid& g = grids[b];
  const int4 ii = atom_img[i];
  const int ci[3] = {(ii.w >> 20) & 1023, (ii.w >> 10) & 1023, ii.w & 1023};
  const double xi[3] = {(double)pos[3 * (int64_t)i], (double)pos[3 * (int64_t)i + 1], (double)pos[3 * (int64_t)i + 2]};
  const int w1 = 2 * g.m[1] + 1;
  const int lo2 = ci[2] - g.m[2], hi2 = ci[2] + g.m[2];
  const int s2_lo = g.pbc[2] ? floor_div(lo2, g.nc[2]) : 0;
  const int K = (g.pbc[2] ? floor_div(hi2, g.nc[2]) : 0) - s2_lo + 1;
  const int T = (2 * g.m[0] + 1) * w1 * K;
  const float inv_k = (1.0f - 0x1p-21f) / (float)K, inv_w = 1.0f / (float)w1;
  int count = 0;
  int base = 0;         // MODE 1: keys collected so far
  int n = 0;            // MODE 1: the row's length
  int64_t r0 = 0;
  bool coincident = false;
  bool shift_range = false;
  bool wide = false;    // a key that does not fit the 32-bit form
  if (MODE == 1) {
    r0 = row_ptr[i];
    n = row_count[i];
  }
  const bool in_lds = n <= kRowKeys;
  for (int t0 = 0; t0 < T; t0 += 64) {
    const int t = t0 + l;
    int cnt = 0, start = 0, swp = 0;
    if (t < T) {
      // t = (o0 * w1 + o1) * K + o2.  inv_k is low by 2^-21, more than the
      // roundings of t, 1 / K and the product together, so q0 comes out right
      // or one short (images have 8 bits: q0 < 2^16).  q1: the reciprocal and
      // the product are off by 2^-24 each, less than half a step of q0 + 0.5.
      // (Divisions raise the registers past 96 and cost the list of 100,000
      // atoms 5%; so did this until five waves a SIMD were asked for.)
      int q0 = (int)((float)t * inv_k), o2 = t - q0 * K;
      if (o2 >= K) {
        ++q0;
        o2 -= K;
      }
      const int q1 = (int)(((float)q0 + 0.5f) * inv_w), o1 = q0 - q1 * w1;
      const int cell[2] = {ci[0] + q1 - g.m[0], ci[1] + o1 - g.m[1]};
      int cc[2], sw[3];
      bool ok = true;
      for (int k = 0; k < 2; ++k) {
        if (g.pbc[k]) {
          // at most one image away while the stencil is narrower than the grid
          sw[k] = g.m[k] <= g.nc[k] ? (cell[k] < 0 ? -1 : cell[k] >= g.nc[k] ? 1 : 0) : floor_div(cell[k], g.nc[k]);
          cc[k] = cell[k] - sw[k] * g.nc[k];
        } else {
          sw[k] = 0;
          cc[k] = cell[k];
          if (cell[k] < 0 || cell[k] >= g.nc[k]) ok = false;
        }
      }
      sw[2] = s2_lo + o2;
      const int c_lo = max(lo2 - sw[2] * g.nc[2], 0), c_hi = min(hi2 - sw[2] * g.nc[2], g.nc[2] - 1);
      if (ok && c_lo <= c_hi) {
        const int64_t cid = g.cell_offset + (int64_t)(cc[0] * g.nc[1] + cc[1]) * g.nc[2];
        start = (int)cell_start[cid + c_lo];
        cnt = (int)cell_start[cid + c_hi + 1] - start;
        swp = pack_shift(sw[0], sw[1], sw[2]);
      }
    }
    const int incl = wave_incl_scan(cnt);
    const int total = __shfl(incl, 63, 64);
    s_excl[w][l] = incl - cnt;
    s_start[w][l] = start - (incl - cnt);
    s_sw[w][l] = swp;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // a lane's candidate: last run k with excl[k] <= c; the next step's
    // candidate is loaded before this one is tested
    auto fetch = [&](int c, CellAtom& a, int4& img, int& sw) {
      int lo = 0;
#pragma unroll
      for (int h = 32; h > 0; h >>= 1)
        if (s_excl[w][lo + h] <= c) lo += h;
      const int slot = s_start[w][lo] + c;
      a = cell_atoms[slot];
      img = cell_img[slot];
      sw = s_sw[w][lo];
    };
    CellAtom na;
    int4 nimg;
    int nsw = 0;
    if (l < total) fetch(l, na, nimg, nsw);
    for (int c0 = 0; c0 < total; c0 += 64) {
      const CellAtom ca = na;
      const int4 jj = nimg;
      const int csw = nsw;
      if (c0 + 64 + l < total) fetch(c0 + 64 + l, na, nimg, nsw);
      bool acc = false;
      uint64_t key = 0;
      if (c0 + l < total) {
        int swx, swy, swz;
        unpack_shift(csw, swx, swy, swz);
        const int j = ca.j;
        const int sx = swx - jj.x + ii.x, sy = swy - jj.y + ii.y, sz = swz - jj.z + ii.z;
        if (!(j == i && sx == 0 && sy == 0 && sz == 0)) {
          const double xj[3] = {(double)ca.x, (double)ca.y, (double)ca.z};
          const double d2 = (sx | sy | sz) == 0 ? pair_d2_home(xi, xj) : pair_d2(xi, xj, g.h, sx, sy, sz);
          if (d2 < rc2) {
            if (d2 == 0.0) {
              coincident = true;
            } else {
              acc = true;
              if (sx < -127 || sx > 127 || sy < -127 || sy > 127 || sz < -127 || sz > 127) {
                shift_range = true;
                acc = false;
              } else if (MODE == 1) {
                key = pair_key(j, sx, sy, sz);
                wide |= sx < -2 || sx > 1 || sy < -2 || sy > 1 || sz < -2 || sz > 1;
              }
            }
          }
        }
      }
      if (MODE == 0) {
        count += acc ? 1 : 0;
      } else {
        const uint64_t bal = __ballot(acc);
        const int slot = base + __popcll(bal & ((1ull << l) - 1ull));
        // (a row past the limit was truncated by the count pass)
        if (acc && slot < n) {
          if (in_lds) s_keys[w][slot] = key;
          else {
            out_j[r0 + slot] = (int)(key >> 24);
            out_shift[r0 + slot] = (int)(key & 0xffffff);
          }
        }
        base += __popcll(bal);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  if (coincident) raise_flag(status, GMNN_FLAG_COINCIDENT);
  if (shift_range) raise_flag(status, GMNN_FLAG_SHIFT_RANGE);
  if (MODE == 0) {
    count = wave_sum(count);
    if (l == 0) {
      // a row past the limit is truncated (and flagged): its slots are exactly
      // the ones the collect pass fills, so the list stays well formed
      row_count[i] = count < GMNN_MAX_ROW ? count : GMNN_MAX_ROW;
      if (count > GMNN_MAX_ROW) raise_flag(status, GMNN_FLAG_ROW_TOO_LONG);
    }
    return;
  }
  auto put = [&](uint64_t k, int rank) {
    out_j[r0 + rank] = (int)(k >> 24);
    out_shift[r0 + rank] = pack_shift((int)((k >> 16) & 0xff) - 128, (int)((k >> 8) & 0xff) - 128,
                                      (int)(k & 0xff) - 128);
  };
  // rank sort (keys are unique inside a row)
  if (!in_lds) {
    // a long row: its keys back from the output arrays, all of a lane's in
    // registers before the first one is overwritten
    __threadfence_block();
    constexpr int Q = GMNN_MAX_ROW / 64;
    uint64_t k[Q];
    int rank[Q];
    auto at = [&](int e) {
      return ((uint64_t)(uint32_t)__builtin_nontemporal_load(out_j + r0 + e) << 24) |
             (uint32_t)__builtin_nontemporal_load(out_shift + r0 + e);
    };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      k[q] = l + 64 * q < n ? at(l + 64 * q) : 0;
      rank[q] = 0;
    }
    for (int e = 0; e < n; ++e) {
      const uint64_t x = at(e);
#pragma unroll
      for (int q = 0; q < Q; ++q) rank[q] += x < k[q] ? 1 : 0;
    }
    __threadfence_block();
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (l + 64 * q < n) put(k[q], rank[q]);
    return;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (__ballot(wide) == 0ull && n_atoms < (1 << 25)) {
    // images within [-2, 1] and fewer than 2^25 atoms: the order is that of
    // 32-bit keys (j, and two bits per image component), half the work per
    // comparison; four keys a read, the row padded with the largest
    uint32_t* s32 = (uint32_t*)s_keys[w];
    uint64_t k[kRowKeys / 64];
    uint32_t k32[kRowKeys / 64];
#pragma unroll
    for (int q = 0; q < kRowKeys / 64; ++q)
      if (l + 64 * q < n) k[q] = s_keys[w][l + 64 * q];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < kRowKeys / 64; ++q) {
      const int e = l + 64 * q;
      if (64 * q >= n + 3) break;
      const uint64_t x = k[q];
      k32[q] = ((uint32_t)(x >> 24) << 6) | ((uint32_t)((x >> 16) & 0xff) - 126) << 4 |
               ((uint32_t)((x >> 8) & 0xff) - 126) << 2 | ((uint32_t)(x & 0xff) - 126);
      if (e >= n) k32[q] = 0xffffffffu;
      s32[e] = k32[q];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    auto ranks = [&](auto QN) {
      constexpr int Q = decltype(QN)::value;
      int rank[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) rank[q] = 0;
      for (int e = 0; e < n; e += 4) {
        const uint4 x = *(const uint4*)(s32 + e);
#pragma unroll
        for (int q = 0; q < Q; ++q)
          rank[q] += (x.x < k32[q] ? 1 : 0) + (x.y < k32[q] ? 1 : 0) + (x.z < k32[q] ? 1 : 0) + (x.w < k32[q] ? 1 : 0);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (l + 64 * q < n) put(k[q], rank[q]);
    };
    if (n <= 64) ranks(std::integral_constant<int, 1>());
    else if (n <= 128) ranks(std::integral_constant<int, 2>());
    else if (n <= 256) ranks(std::integral_constant<int, 4>());
    else ranks(std::integral_constant<int, kRowKeys / 64>());
    return;
  }
  for (int e = l; e < n; e += 64) {
    const uint64_t k = s_keys[w][e];
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += (s_keys[w][q] < k) ? 1 : 0;
    put(k, rank);
  }
}

struct __attribute__((packed, aligned(4))) Int4u {
  int x, y, z, w;
};
struct __attribute__((packed, aligned(8))) Ptr2 {
  int64_t x, y;
};
__global__ void __launch_bounds__(64 * kRowsWaves) nl_reverse(int n_atoms, const int64_t* __restrict__ row_ptr,
                                                             const int32_t* __restrict__ nj,
                                                             const int32_t* __restrict__ nshift,
                                                             const int64_t* __restrict__ n_pairs, int64_t capacity,
                                                             int32_t* __restrict__ rev, uint32_t* __restrict__ status,
                                                             const int* __restrict__ go) {
  const int w = threadIdx.x >> 6;
  const int l = threadIdx.x & 63;
  const int i = xcd_block(blockIdx.x, gridDim.x) * kRowsWaves + w;
  if (i >= n_atoms) return;
  if (!*go) return;
  if (*n_pairs > capacity) return;
  const int64_t p0 = row_ptr[i], p1 = row_ptr[i + 1];
  const int ni = (int)(p1 - p0);
  for (int64_t p = p0 + l; p < p1; p += 64) {
    const int j = nj[p];
    const Ptr2 rp = *(const Ptr2*)(row_ptr + j);
    const int64_t r0 = rp.x;
    const int n = (int)(rp.y - r0);
    const int32_t* __restrict__ row = nj + r0;
    // first slot of row j that holds atom i or a later one.  In a spatially
    // ordered system the rows mirror each other (j early in row i puts i late
    // in row j), so eight slots around the mirrored place (two 16-byte loads)
    // are looked at first; where they miss, the rest is halved as usual
    int lo = 0, hi = n;
    bool sole = false;  // the window shows that no second image of i follows
    if (n >= 8) {
      const int guess = n - 1 - (int)((float)(int)(p - p0) * (float)n / (float)ni);
      const int g0 = max(0, min(guess - 3, n - 8));
      const Int4u a = *(const Int4u*)(row + g0), b = *(const Int4u*)(row + g0 + 4);
      const int v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      int below = 0, equal = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        below += v[e] < i ? 1 : 0;
        equal += v[e] == i ? 1 : 0;
      }
      if (below == 8) {
        lo = g0 + 8;
      } else if (below > 0 || g0 == 0) {
        lo = hi = g0 + below;
        sole = equal == 1 && below < 7;
      } else {
        hi = g0;
      }
    }
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (row[mid] < i) lo = mid + 1; else hi = mid;
    }
    int64_t found = sole ? r0 + lo : -1;
    if (!sole) {
      // several images of i: the one with the opposite shift
      int sx, sy, sz;
      unpack_shift(nshift[p], sx, sy, sz);
      const int32_t want = pack_shift(-sx, -sy, -sz);
      for (int e = lo; e < n && row[e] == i; ++e)
        if (nshift[r0 + e] == want) {
          found = r0 + e;
          break;
        }
    }
    if (found < 0) {
      raise_flag(status, GMNN_FLAG_ROW_TOO_LONG);
      found = p;
    }
    rev[p] = (int32_t)found;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// at least the cells the device's grid has, whichever way its roundings fall
static int host_cells_bound(const double* h, double rbin, int64_t n_atoms) {
  const double a[3][3] = {{h[0], h[1], h[2]}, {h[3], h[4], h[5]}, {h[6], h[7], h[8]}};
  double cr[3][3];
  for (int k = 0; k < 3; ++k) {
    const double* u = a[(k + 1) % 3];
    const double* v = a[(k + 2) % 3];
    cr[k][0] = u[1] * v[2] - u[2] * v[1];
    cr[k][1] = u[2] * v[0] - u[0] * v[2];
    cr[k][2] = u[0] * v[1] - u[1] * v[0];
  }
  const double det = a[0][0] * cr[0][0] + a[0][1] * cr[0][1] + a[0][2] * cr[0][2];
  const double vol = fabs(det);
  long long fewest = 1, fine = 1, coarse = 1;
  for (int k = 0; k < 3; ++k) {
    const double nrm = sqrt(cr[k][0] * cr[k][0] + cr[k][1] * cr[k][1] + cr[k][2] * cr[k][2]);
    const int nf = cells_on_axis(kCellsPerRadius * (vol / nrm) / rbin);
    fewest *= std::max(nf - 1, 1);
    // +1 per axis absorbs any rounding difference between host and device
    fine *= nf + 1;
    coarse *= cells_on_axis(vol / nrm / rbin) + 1;
  }
  const long long cells = fewest <= max_fine_cells(n_atoms) ? std::max(fine, coarse) : coarse;
  return (int)(cells > (1LL << 30) ? (1LL << 30) : cells);
}

NlLayout nl_layout(const gmnn_system* sys, double rbin) {
  NlLayout L;
  int64_t cells = 0;
  for (int b = 0; b < sys->n_structs; ++b)
    cells += host_cells_bound(sys->cell_host + 9 * (int64_t)b, rbin,
                              sys->atom_ptr_host[b + 1] - sys->atom_ptr_host[b]);
  L.cell_capacity = cells;
  const int64_t N = sys->n_atoms;
  const int64_t B = sys->n_structs;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  };
  L.off_grids = take(sizeof(StructGrid) * (size_t)B);
  L.off_cell_count = take(4 * (size_t)cells);
  L.off_cell_fill = take(4 * (size_t)cells);
  L.off_cell_start = take(8 * (size_t)(cells + 1));
  L.off_cells_total = take(8 * 2);
  L.off_atom_cell = take(4 * (size_t)N);
  L.off_atom_img = take(16 * (size_t)N);
  L.off_cell_atoms = take(sizeof(CellAtom) * (size_t)N);
  L.off_cell_img = take(16 * (size_t)N);
  L.off_scan = take(4 * (size_t)((std::max<int64_t>(cells, N) + kScanTile - 1) / kScanTile));
  L.off_row_count = take(4 * (size_t)N + 4);
  L.off_go = take(4);
  L.bytes = off;
  return L;
}

gmnn_status nl_build(const gmnn_system* sys, float cutoff, float skin, gmnn_neighbors* nl, void* ws,
                     size_t ws_bytes, hipStream_t stream, const uint32_t* disp_bits, float thresh2, float* ref_pos) {
  const double rl = (double)(cutoff + skin);
  const double rbin = rl + 1.0e-4;
  NlLayout L = nl_layout(sys, rbin);
  if (ws_bytes < L.bytes) return GMNN_ERR_WORKSPACE;
  char* w = (char*)ws;
  StructGrid* grids = (StructGrid*)(w + L.off_grids);
  int32_t* cell_count = (int32_t*)(w + L.off_cell_count);
  int32_t* cell_fill = (int32_t*)(w + L.off_cell_fill);
  int64_t* cell_start = (int64_t*)(w + L.off_cell_start);
  int64_t* cells_total = (int64_t*)(w + L.off_cells_total);
  int32_t* atom_cell = (int32_t*)(w + L.off_atom_cell);
  int4* atom_img = (int4*)(w + L.off_atom_img);
  CellAtom* cell_atoms = (CellAtom*)(w + L.off_cell_atoms);
  int4* cell_img = (int4*)(w + L.off_cell_img);
  int32_t* part = (int32_t*)(w + L.off_scan);
  int32_t* row_count = (int32_t*)(w + L.off_row_count);
  int* go = (int*)(w + L.off_go);
  const int N = sys->n_atoms;
  const int B = sys->n_structs;
  const float rlf = cutoff + skin;
  const double rc2 = (double)rlf * (double)rlf;
  nl->cutoff = rlf;

  hipLaunchKernelGGL(nl_setup, dim3(1), dim3(1024), 0, stream, sys->cell, sys->pbc, sys->atom_ptr, B, rbin, grids,
                     L.cell_capacity, cell_count, cell_fill, cells_total, nl->status, disp_bits, thresh2, go);
  const int tb = 256;
  const int nb_atoms = (N + tb - 1) / tb;
  if (N > 0) {
    hipLaunchKernelGGL(nl_bin, dim3(nb_atoms), dim3(tb), 0, stream, sys->pos, sys->atom_ptr, B, N, grids,
                       cells_total, L.cell_capacity, nl->atom_struct, atom_cell, atom_img, cell_count, nl->status, go,
                       ref_pos);
  }
  auto scan = [&](const int32_t* in, int64_t* out, const int64_t* n_dev, int64_t n, int64_t* total, int64_t cap) {
    if (n <= kScanOne) {
      hipLaunchKernelGGL(scan_one, dim3(1), dim3(kScanThreads), 0, stream, in, out, n_dev, n, total, (const int*)go,
                         cap);
      return;
    }
    const dim3 grid((unsigned)((n + kScanTile - 1) / kScanTile));
    hipLaunchKernelGGL(scan_sums, grid, dim3(kScanThreads), 0, stream, in, n_dev, n, part, (const int*)go);
    hipLaunchKernelGGL(scan_write, grid, dim3(kScanThreads), 0, stream, in, out, n_dev, n, (const int32_t*)part, total,
                       (const int*)go, cap);
  };
  scan(cell_count, cell_start, cells_total, L.cell_capacity, nullptr, -1);
  if (N > 0) {
    hipLaunchKernelGGL(nl_cellfill, dim3(nb_atoms), dim3(tb), 0, stream, N, sys->pos, atom_cell, atom_img, cell_start,
                       cells_total, L.cell_capacity, cell_fill, cell_atoms, cell_img, (const int*)go);
    const int nb_rows = (N + kRowsWaves - 1) / kRowsWaves;
    hipLaunchKernelGGL(nl_rows<0>, dim3(nb_rows), dim3(64 * kRowsWaves), 0, stream, sys->pos, N, grids,
                       nl->atom_struct, atom_img, cell_start, cell_atoms, cell_img, cells_total, L.cell_capacity, rc2, row_count,
                       (const int64_t*)nullptr, (const int64_t*)nullptr, nl->capacity, (int32_t*)nullptr,
                       (int32_t*)nullptr, nl->status, (const int*)go);
    scan(row_count, nl->row_ptr, nullptr, N, nl->n_pairs, nl->capacity);
    hipLaunchKernelGGL(nl_rows<1>, dim3(nb_rows), dim3(64 * kRowsWaves), 0, stream, sys->pos, N, grids,
                       nl->atom_struct, atom_img, cell_start, cell_atoms, cell_img, cells_total, L.cell_capacity, rc2, row_count,
                       nl->row_ptr, nl->n_pairs, nl->capacity, nl->j, nl->shift, nl->status, (const int*)go);
    hipLaunchKernelGGL(nl_reverse, dim3(nb_rows), dim3(64 * kRowsWaves), 0, stream, N, nl->row_ptr, nl->j, nl->shift,
                       nl->n_pairs, nl->capacity, nl->rev, nl->status, (const int*)go);
  } else {
    scan(row_count, nl->row_ptr, nullptr, 0, nl->n_pairs, nl->capacity);
  }
  return hipGetLastError() == hipSuccess ? GMNN_OK : GMNN_ERR_HIP;
}

}  // namespace gmnn
