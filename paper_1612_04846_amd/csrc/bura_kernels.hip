// HIP kernels (gfx950) for the k+1 shifted SPD solves of the BURA method
// (Section 2.2, eq. (16)): matrix-free 5/7-point stencils of the scaled operator
// A + s I (Section 1.4, eq. (10); Section 5.3), weighted-Jacobi smoothing,
// full-weighting restriction, multilinear prolongation, an in-LDS V-cycle for
// the coarse levels, the PCG vector updates with FP64 block reductions, the
// FP64 residual of the refinement loop and the FP64 combine of eq. (16).
//
// Every launch processes a batch of independent systems: blockIdx.z (stencil
// launches) or blockIdx.y (flat kernels) selects the system; a system whose `active` flag
// is 0 is skipped by whole blocks.  Reductions are deterministic: each block
// writes one FP64 partial per system and a per-system kernel adds the partials
// in a fixed order, so a system's result does not depend on what else is in
// the batch.
#include "bura_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace bura {

// --------------------------------------------------------------------------
// small helpers
// --------------------------------------------------------------------------

// Tile coordinates of a stencil workgroup: (x tile, y tile, system), in launch
// order.  Workgroups are dealt to the 8 XCDs round-robin, so vertically
// adjacent tiles sit on different L2s and their common halo rows are fetched
// twice; those second fetches hit the on-package last-level cache.  Renumbering
// the workgroups so that an XCD takes contiguous tiles removed them but made
// every stencil kernel slower (it concentrates each XCD on one address range),
// so launch order is kept.
struct Tile {
  int x, y, z;
};

__device__ __forceinline__ Tile block_tile() {
  Tile r;
  r.x = blockIdx.x;
  r.y = blockIdx.y;
  r.z = blockIdx.z;
  return r;
}

// The tile of a launch whose systems share more than the L2s hold (the face
// weights of a 3D variable-coefficient level, the FP64 right-hand side): the
// systems of a tile run side by side on one XCD (workgroups are dealt to the 8
// XCDs round-robin), which reads the shared values once, and an XCD has a
// contiguous range of tiles.  127^3, 9 systems, whose weights (25 MB in FP32)
// were read from memory once per system: a solve of 7513 us takes 7377.  (FP64
// sweeps, whose vectors are twice as long, take the launch order: 127^3, 8
// systems 11.1 ms, by tiles 11.7.)
__device__ __forceinline__ Tile block_tile_shared() {
  const unsigned lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const unsigned total = gridDim.x * gridDim.y * gridDim.z, x = lin & 7;
  const unsigned idx = x * (total >> 3) + min(x, total & 7) + (lin >> 3);
  const unsigned tile = idx / gridDim.z;
  Tile r;
  r.x = tile % gridDim.x;
  r.y = tile / gridDim.x;
  r.z = idx - tile * gridDim.z;
  return r;
}

template <int DIM>
__device__ __forceinline__ void tile_ijk(const Tile& tl, int n, int& i, int& j, int& k) {
  i = tl.x * kTileX + threadIdx.x;
  const int ytiles = (n + kTileY - 1) / kTileY;
  int by = tl.y;
  if (DIM == 3) {
    k = by / ytiles;
    by -= k * ytiles;
  } else {
    k = 0;
  }
  j = by * kTileY + threadIdx.y;
}

// 3D launches that march along z (the stencil product, the smoothing sweeps
// and the FP64 residual): a workgroup of march_x(n) x (256 / march_x(n))
// threads owns that
// block of columns over kMarchZ consecutive planes, and each thread carries
// its column's values at planes k-1, k, k+1 in registers from one plane to the
// next, so the points above and below are not loaded again (a
// one-point-per-thread launch reads them from the last-level caches).
constexpr int kMarchZ = 8;
// rows per thread of the marching kernels that write per-block partials (the
// rows above and below a thread's interior rows come from its own registers;
// a workgroup covers march_x(n) x ((256 / march_x(n)) kMarchRows) columns)
// (4 since the workgroups are up to 256 columns wide and so only a few rows
// high: 255^3 mixed went from 35.8 ms with 2 rows to 34.5 ms; 8 rows gained
// another 0.5 % but halves the workgroups of small grids)
constexpr int kMarchRows = 4;

struct Column {
  int i, j, k0, k1;   // the thread's first column (i, j) (rows j .. j + rows - 1) and its planes [k0, k1)
};

__device__ __forceinline__ Column march_column(const Tile& tl, int n, int rows, int planes = kMarchZ) {
  Column c;
  // the workgroup's shape is chosen per grid (march_x on the host)
  const int my = blockDim.y;
  const int yt = (n + my * rows - 1) / (my * rows);
  const int kc = tl.y / yt;
  c.i = tl.x * blockDim.x + threadIdx.x;
  c.j = ((tl.y - kc * yt) * my + threadIdx.y) * rows;
  c.k0 = kc * planes;
  c.k1 = min(c.k0 + planes, n);
  return c;
}

// A thread's R rows in a marching kernel: row r is j0 + r; rows at or beyond n
// are not computed (their loads read row n - 1).  Offsets of the rows and of
// the halo rows j0 - 1 and j0 + R within a plane.
template <int R>
struct Rows {
  long long col[R];   // in-plane offset of row r (clamped)
  bool valid[R];
  bool has_d, has_u;  // rows j0 - 1 and j0 + R inside the grid
  long long col_d, col_u;
  int il, ir;         // x-neighbour offsets (0 at the boundary)
  __device__ __forceinline__ Rows(int i, int j0, int n) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      valid[r] = j0 + r < n;
      col[r] = (long long)min(j0 + r, n - 1) * n + i;
    }
    has_d = j0 > 0;
    has_u = j0 + R < n;
    col_d = (long long)(has_d ? j0 - 1 : j0) * n + i;
    col_u = (long long)(has_u ? j0 + R : n - 1) * n + i;
    il = i > 0 ? -1 : 0;
    ir = i < n - 1 ? 1 : 0;
  }
  // the row-below / row-above neighbours of row r from the rows' centre values
  // and the halo values (0 outside the grid)
  template <typename T>
  __device__ __forceinline__ T down(int r, const T* centre, T halo_d) const {
    return r == 0 ? (has_d ? halo_d : T(0)) : centre[r - 1];
  }
  template <typename T>
  __device__ __forceinline__ T up(int r, const T* centre, T halo_u) const {
    return r == R - 1 ? (has_u ? halo_u : T(0)) : (valid[r + 1] ? centre[r + 1] : T(0));
  }
};

// FP64 block sum; the result is valid in thread 0 only.  Fixed order.
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double sh[16];   // one value per wave, up to 1024 threads
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  if ((tid & 63) == 0) sh[tid >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (tid == 0) {
    const int nw = (blockDim.x * blockDim.y + 63) >> 6;
    for (int w = 0; w < nw; ++w) r += sh[w];
  }
  return r;
}

// Stencil launches: the block's (x, y) tile index; flat launches: blockIdx.x.
__device__ __forceinline__ void write_partial(double* partial, int sys, double v, int blk, int nblk) {
  const double s = block_sum(v);
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  if (tid == 0) partial[(size_t)sys * nblk + blk] = s;
}

__device__ __forceinline__ void write_partial_tile(const Tile& tl, double* partial, int sys, double v) {
  write_partial(partial, sys, v, tl.y * gridDim.x + tl.x, gridDim.x * gridDim.y);
}

__device__ __forceinline__ void write_partial_flat(double* partial, int sys, double v) {
  write_partial(partial, sys, v, blockIdx.x, gridDim.x);
}

__device__ void apply_op(int op, double tot, const SysState& S, int sys, double tol, int max_iter);

// The last block of `sys` (after every block has written its partial) sums
// the partials in the same fixed order as k_scalars and applies fin.op.
__device__ __forceinline__ void finish(const Fin& fin, const double* partial, int sys, int blk_count) {
  if (fin.op < 0) return;
  __shared__ int s_last;
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  const int nthr = blockDim.x * blockDim.y;
  if (tid == 0) {
    __threadfence();
    const unsigned prev = atomicAdd(fin.cnt + sys, 1u);
    s_last = prev == (unsigned)(blk_count - 1);
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  double v = 0.0;
  for (int b = tid; b < blk_count; b += nthr) v += partial[(size_t)sys * blk_count + b];
  const double tot = block_sum(v);
  if (tid == 0) {
    atomicExch(fin.cnt + sys, 0u);
    apply_op(fin.op, tot, fin.st, sys, fin.tol, fin.max_iter);
  }
}

// Profiling: the first block of each system adds that system's algorithmic
// bytes for the whole launch (each vector element read or written once) to a
// per-kernel-class counter -- one atomic per system per launch.
// Stencil launches: grid (x tiles, y tiles, system); element-wise launches:
// grid (chunks, system); the coarse solve: one block per system.
enum CountKind { COUNT_TILE, COUNT_FLAT, COUNT_ONE };

template <CountKind K>
__device__ __forceinline__ void count_bytes(unsigned long long* ctr, unsigned long long b) {
  if (ctr == nullptr || threadIdx.x != 0 || threadIdx.y != 0) return;
  const bool first = K == COUNT_ONE ? true : (K == COUNT_FLAT ? blockIdx.x == 0 : (blockIdx.x == 0 && blockIdx.y == 0));
  if (first) atomicAdd(ctr, b);
}

// stencil launches: the workgroup holding tile (0, 0) of the system counts
__device__ __forceinline__ void count_bytes_tile(const Tile& tl, unsigned long long* ctr, unsigned long long b) {
  if (ctr == nullptr || threadIdx.x != 0 || threadIdx.y != 0) return;
  if (tl.x == 0 && tl.y == 0) atomicAdd(ctr, b);
}


// (A_l + s I) x at interior point (i,j,k), flux form sum_f w_f (x_c - x_nb) + s x_c.
// Also returns the diagonal through *dg when dg != nullptr.
template <typename T, int DIM, bool VAR>
__device__ __forceinline__ T apply_pt(const LevelDev<T>& L, const T* __restrict__ x, int i, int j, int k,
                                      long long p, T s, T* dg) {
  const int n = L.n;
  const long long nn = (long long)n * n;
  // neighbour loads are unconditional (a boundary neighbour reads the centre
  // instead) so that they are all in flight together; the value is selected after
  const T xc = x[p];
  const T xl0 = x[i > 0 ? p - 1 : p], xr0 = x[i < n - 1 ? p + 1 : p];
  const T xd0 = x[j > 0 ? p - n : p], xu0 = x[j < n - 1 ? p + n : p];
  T xb0 = T(0), xf0 = T(0);
  if (DIM == 3) {
    xb0 = x[k > 0 ? p - nn : p];
    xf0 = x[k < n - 1 ? p + nn : p];
  }
  const T xl = i > 0 ? xl0 : T(0), xr = i < n - 1 ? xr0 : T(0);
  const T xd = j > 0 ? xd0 : T(0), xu = j < n - 1 ? xu0 : T(0);
  const T xb = DIM == 3 && k > 0 ? xb0 : T(0), xf = DIM == 3 && k < n - 1 ? xf0 : T(0);
  if (!VAR) {
    const T w = L.wc;
    T sum = (xc - xl) + (xc - xr) + (xc - xd) + (xc - xu);
    if (DIM == 3) sum += (xc - xb) + (xc - xf);
    if (dg) *dg = w * T(2 * DIM) + s;
    return w * sum + s * xc;
  } else {
    const long long fx = ((long long)k * n + j) * (n + 1) + i;
    const T wl = L.wf0[fx], wr = L.wf0[fx + 1];
    const long long fy = ((long long)k * (n + 1) + j) * n + i;
    const T wd = L.wf1[fy], wu = L.wf1[fy + n];
    T acc = wl * (xc - xl) + wr * (xc - xr) + wd * (xc - xd) + wu * (xc - xu);
    T d = wl + wr + wd + wu;
    if (DIM == 3) {
      const long long fz = ((long long)k * n + j) * n + i;
      const T wb = L.wf2[fz], wf = L.wf2[fz + nn];
      acc += wb * (xc - xb) + wf * (xc - xf);
      d += wb + wf;
    }
    if (dg) *dg = d + s;
    return acc + s * xc;
  }
}

template <typename T, int DIM, bool VAR>
__device__ __forceinline__ T diag_pt(const LevelDev<T>& L, int i, int j, int k, T s) {
  if (!VAR) return L.wc * T(2 * DIM) + s;
  const int n = L.n;
  const long long fx = ((long long)k * n + j) * (n + 1) + i;
  const long long fy = ((long long)k * (n + 1) + j) * n + i;
  T d = L.wf0[fx] + L.wf0[fx + 1] + L.wf1[fy] + L.wf1[fy + n];
  if (DIM == 3) {
    const long long fz = ((long long)k * n + j) * n + i;
    d += L.wf2[fz] + L.wf2[fz + (long long)n * n];
  }
  return d + s;
}

// value o of a plane whose address is the same for the workgroup: a scalar base
// and a 32-bit offset, not a 64-bit address per lane
template <typename T>
__device__ __forceinline__ T plane_at(const T* __restrict__ plane, unsigned o) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(plane) + o * (unsigned)sizeof(T));
}

// The face weights of a marching thread's R rows at one plane: left, right,
// below in y (d[R]: above the last row), below and above in z.  All of them
// are loaded with the plane's other values, before any is used (loaded where
// each row used them, behind the row's bounds test, every row waited for
// memory again); the face between two rows or planes is loaded once.  127^3
// mixed, 9 systems: 7377 -> 6524 us a solve.  FP64 sweeps would hold 160 - 280
// registers that way and ran 5 - 8 % slower (47^3 - 127^3): they load a row's
// weights at the row (EARLY false), the FP64 residual all at once (155 -> 151 us).
template <typename T, bool VAR, int R, bool EARLY = sizeof(T) == 4>
struct ColFaces {
  T l[R], r[R], d[R + 1], b[R], f[R];
  __device__ __forceinline__ void start(const LevelDev<T>& L, const Rows<R>& w, int k0) {
    if (!VAR || !EARLY) return;
#pragma unroll
    for (int q = 0; q < R; ++q) f[q] = L.wf2[(long long)k0 * L.n * L.n + w.col[q]];
  }
  // the weights of row q of the grid (EARLY false)
  __device__ __forceinline__ void row(const LevelDev<T>& L, const Rows<R>& w, int i, int j0, int k, int q) {
    if (!VAR || EARLY) return;
    const int n = L.n;
    const long long fx = ((long long)k * n + j0 + q) * (n + 1) + i, fy = ((long long)k * (n + 1) + j0 + q) * n + i;
    const long long p = (long long)k * n * n + w.col[q];
    l[q] = L.wf0[fx];
    r[q] = L.wf0[fx + 1];
    d[q] = L.wf1[fy];
    d[q + 1] = L.wf1[fy + n];
    b[q] = L.wf2[p];
    f[q] = L.wf2[p + (long long)n * n];
  }
  // the weights of every row (EARLY)
  __device__ __forceinline__ void load(const LevelDev<T>& L, const Rows<R>& w, int i, int j0, int k) {
    if (!VAR || !EARLY) return;
    const int n = L.n;
    const T* w0 = L.wf0 + (long long)k * n * (n + 1);
    const T* w1 = L.wf1 + (long long)k * (n + 1) * n;
    const T* w2 = L.wf2 + (long long)(k + 1) * n * n;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const unsigned o = (unsigned)(min(j0 + q, n - 1) * (n + 1) + i);
      b[q] = f[q];
      l[q] = plane_at(w0, o);
      r[q] = plane_at(w0, o + 1);
      f[q] = plane_at(w2, (unsigned)w.col[q]);
    }
#pragma unroll
    for (int q = 0; q <= R; ++q) d[q] = plane_at(w1, (unsigned)(min(j0 + q, n) * n + i));
  }
  __device__ __forceinline__ T diag(const LevelDev<T>& L, int q, T s) const {
    if (!VAR) return L.wc * T(6) + s;
    return l[q] + r[q] + d[q] + d[q + 1] + (b[q] + f[q]) + s;
  }
};

// apply_pt for DIM = 3 from values already loaded: the face weights of row q,
// the centre, its in-plane neighbours l, r, d, u and the points below (b) and
// above (f), each 0 outside the grid.  Same arithmetic and order as apply_pt.
template <typename T, bool VAR, int R, bool EARLY>
__device__ __forceinline__ T apply_col3(const LevelDev<T>& L, const ColFaces<T, VAR, R, EARLY>& w, int q, T xc, T xl, T xr,
                                        T xd, T xu, T xb, T xf, T s) {
  if (!VAR) {
    T sum = (xc - xl) + (xc - xr) + (xc - xd) + (xc - xu);
    sum += (xc - xb) + (xc - xf);
    return L.wc * sum + s * xc;
  }
  T acc = w.l[q] * (xc - xl) + w.r[q] * (xc - xr) + w.d[q] * (xc - xd) + w.d[q + 1] * (xc - xu);
  acc += w.b[q] * (xc - xb) + w.f[q] * (xc - xf);
  return acc + s * xc;
}

// In-plane neighbour offsets of a column (0 where the neighbour is outside the
// grid: the load then reads the centre and the value is replaced by 0).
struct PlaneNb {
  int l, r, d, u;
};

__device__ __forceinline__ PlaneNb plane_nb(int i, int j, int n) {
  PlaneNb o;
  o.l = i > 0 ? -1 : 0;
  o.r = i < n - 1 ? 1 : 0;
  o.d = j > 0 ? -n : 0;
  o.u = j < n - 1 ? n : 0;
  return o;
}

// --------------------------------------------------------------------------
// smoother: x_out = x_in + omega D^-1 (b - (A+s) x_in)   (x_in = 0 if ZERO)
// DOT: partial = b . x_out  (r.z when this is the last sweep of z = M r)
// --------------------------------------------------------------------------
template <typename T, int DIM, bool VAR, bool ZERO, bool DOT>
__global__ __launch_bounds__(kBlock) void k_jacobi(LevelDev<T> L, const T* __restrict__ b,
                                                   const T* __restrict__ xin, T* __restrict__ xout,
                                                   const T* __restrict__ shift, const int* __restrict__ active,
                                                   T omega, double* __restrict__ partial,
                                                   unsigned long long* __restrict__ ctr, Fin fin) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  int i, j, k;
  tile_ijk<DIM>(tl, L.n, i, j, k);
  const bool ok = i < L.n && j < L.n;
  const long long off = (long long)sys * L.N;
  const long long p = ((long long)k * L.n + j) * L.n + i;
  const T s = shift[sys];
  // b and x_out, plus x_in unless the guess is zero; faces once per launch
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) * ((ZERO ? 2 : 3) + (VAR && sys == 0 ? DIM : 0)));
  double dot = 0.0;
  if (ok) {
    const T bv = b[off + p];
    T xn;
    if (ZERO) {
      xn = omega * bv / diag_pt<T, DIM, VAR>(L, i, j, k, s);
    } else {
      T dg;
      const T ax = apply_pt<T, DIM, VAR>(L, xin + off, i, j, k, p, s, &dg);
      xn = xin[off + p] + omega * (bv - ax) / dg;
    }
    xout[off + p] = xn;
    if (DOT) dot = (double)bv * (double)xn;
  }
  if (DOT) {
    write_partial_tile(tl, partial, sys, dot);
    finish(fin, partial, sys, gridDim.x * gridDim.y);
  }
}

// k_jacobi in 3D, marching along z (one workgroup per `planes` planes,
// kMarchRows rows per thread).
template <typename T, bool VAR, bool ZERO, bool DOT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && VAR && !DOT ? 4 : 1))) void
k_jacobi3(LevelDev<T> L, const T* __restrict__ b,
                                                    const T* __restrict__ xin, T* __restrict__ xout,
                                                    const T* __restrict__ shift, const int* __restrict__ active,
                                                    T omega, double* __restrict__ partial,
                                                    unsigned long long* __restrict__ ctr, Fin fin, int planes) {
  constexpr int R = kMarchRows;
  const Tile tl = VAR && sizeof(T) == 4 ? block_tile_shared() : block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) * ((ZERO ? 2 : 3) + (VAR && sys == 0 ? 3 : 0)));
  const int n = L.n;
  const Column c = march_column(tl, n, R, planes);
  double dot = 0.0;
  if (c.i < n && c.j < n) {
    const long long off = (long long)sys * L.N, nn = (long long)n * n;
    const Rows<R> w(c.i, c.j, n);
    const T s = shift[sys];
    const T* bs = b + off;
    T* xo = xout + off;
    ColFaces<T, VAR, R> fw;
    fw.start(L, w, c.k0);
    if (ZERO) {
      for (int k = c.k0; k < c.k1; ++k) {
        T bv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) bv[r] = bs[k * nn + w.col[r]];
        fw.load(L, w, c.i, c.j, k);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (!w.valid[r]) continue;
          fw.row(L, w, c.i, c.j, k, r);
          const T xn = omega * bv[r] / fw.diag(L, r, s);
          xo[k * nn + w.col[r]] = xn;
          if (DOT) dot += (double)bv[r] * (double)xn;
        }
      }
    } else {
      const T* xs = xin + off;
      T below[R], centre[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const long long p0 = c.k0 * nn + w.col[r];
        const T xb0 = xs[c.k0 > 0 ? p0 - nn : p0];
        below[r] = c.k0 > 0 ? xb0 : T(0);
        centre[r] = xs[p0];
      }
      for (int k = c.k0; k < c.k1; ++k) {
        const long long pk = k * nn;
        // every load of the plane first, then the arithmetic (loading the next
        // plane one step ahead measured slower)
        T xa[R], xl[R], xr[R], bv[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const long long p = pk + w.col[r];
          xa[r] = xs[k + 1 < n ? p + nn : p];
          xl[r] = xs[p + w.il];
          xr[r] = xs[p + w.ir];
          bv[r] = bs[p];
        }
        const T hd = xs[pk + w.col_d], hu = xs[pk + w.col_u];
        fw.load(L, w, c.i, c.j, k);
        T above[R];
#pragma unroll
        for (int r = 0; r < R; ++r) above[r] = k + 1 < n ? xa[r] : T(0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (!w.valid[r]) continue;
          fw.row(L, w, c.i, c.j, k, r);
          const T ax = apply_col3(L, fw, r, centre[r], w.il ? xl[r] : T(0), w.ir ? xr[r] : T(0),
                                             w.down(r, centre, hd), w.up(r, centre, hu), below[r], above[r], s);
          const T xn = centre[r] + omega * (bv[r] - ax) / fw.diag(L, r, s);
          xo[pk + w.col[r]] = xn;
          if (DOT) dot += (double)bv[r] * (double)xn;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          below[r] = centre[r];
          centre[r] = above[r];
        }
      }
    }
  }
  if (DOT) {
    write_partial_tile(tl, partial, sys, dot);
    finish(fin, partial, sys, gridDim.x * gridDim.y);
  }
}

// The first pre-smoothing sweep of the fine level (from x = 0) with the PCG
// residual update folded in: b = b_old - alpha q is written to bout with its
// squared norm into partial, and x_out = omega D^-1 b.  The sweep reads no
// neighbour of b, so the update needs no second pass.
template <typename T, int DIM, bool VAR>
__global__ __launch_bounds__(kBlock) void k_jacobi0_rup(LevelDev<T> L, const T* __restrict__ bold,
                                                        const T* __restrict__ q, const double* __restrict__ alpha,
                                                        T* __restrict__ bout, T* __restrict__ xout,
                                                        const T* __restrict__ shift, const int* __restrict__ active,
                                                        T omega, double* __restrict__ partial,
                                                        unsigned long long* __restrict__ ctr, Fin fin) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  const int n = L.n;
  // 2D: one point; 3D: kMarchRows rows over kMarchZ planes
  constexpr int R = DIM == 3 ? kMarchRows : 1;
  int i, j, k0, k1;
  if (DIM == 3) {
    const Column c = march_column(tl, n, R);
    i = c.i;
    j = c.j;
    k0 = c.k0;
    k1 = c.k1;
  } else {
    tile_ijk<DIM>(tl, n, i, j, k0);
    k1 = k0 + 1;
  }
  const long long off = (long long)sys * L.N;
  const T s = shift[sys];
  const T a = (T)alpha[sys];
  // b_old and q read, b and x_out written; faces once per launch
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) * (4 + (VAR && sys == 0 ? DIM : 0)));
  double rr = 0.0;
  if (i < n) {
    for (int k = k0; k < k1; ++k) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (j + r >= n) continue;
        const long long p = ((long long)k * n + j + r) * n + i;
        const T bv = bold[off + p] - a * q[off + p];
        bout[off + p] = bv;
        xout[off + p] = omega * bv / diag_pt<T, DIM, VAR>(L, i, j + r, k, s);
        rr += (double)bv * (double)bv;
      }
    }
  }
  write_partial_tile(tl, partial, sys, rr);
  finish(fin, partial, sys, gridDim.x * gridDim.y);
}

// 3D first fine sweep with the PCG residual update, forming q = (A + s) p
// itself from p while marching along z (as k_jacobi3 forms (A + s) x):
// b = b_old - alpha q to bout with |b|^2 into partial, x_out = omega D^-1 b.
// The stencil product then stores no q (one vector pass less per iteration).
template <typename T, bool VAR>
__global__ __launch_bounds__(kBlock) void k_jacobi0_rup3p(LevelDev<T> L, const T* __restrict__ bold,
                                                          const T* __restrict__ pv, const double* __restrict__ alpha,
                                                          T* __restrict__ bout, T* __restrict__ xout,
                                                          const T* __restrict__ shift, const int* __restrict__ active,
                                                          T omega, double* __restrict__ partial,
                                                          unsigned long long* __restrict__ ctr, Fin fin) {
  constexpr int R = kMarchRows;
  const Tile tl = VAR && sizeof(T) == 4 ? block_tile_shared() : block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  // b_old and p read, b and x_out written; faces once per launch
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) * (4 + (VAR && sys == 0 ? 3 : 0)));
  const int n = L.n;
  const Column c = march_column(tl, n, R);
  double rr = 0.0;
  if (c.i < n && c.j < n) {
    const long long off = (long long)sys * L.N, nn = (long long)n * n;
    const Rows<R> w(c.i, c.j, n);
    const T s = shift[sys];
    const T a = (T)alpha[sys];
    const T* ps = pv + off;
    const T* bs = bold + off;
    T below[R], centre[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const long long p0 = c.k0 * nn + w.col[r];
      const T pb0 = ps[c.k0 > 0 ? p0 - nn : p0];
      below[r] = c.k0 > 0 ? pb0 : T(0);
      centre[r] = ps[p0];
    }
    ColFaces<T, VAR, R> fw;
    fw.start(L, w, c.k0);
    for (int k = c.k0; k < c.k1; ++k) {
      const long long pk = k * nn;
      T pa[R], pl[R], pr[R], bv[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const long long p = pk + w.col[r];
        pa[r] = ps[k + 1 < n ? p + nn : p];
        pl[r] = ps[p + w.il];
        pr[r] = ps[p + w.ir];
        bv[r] = bs[p];
      }
      const T hd = ps[pk + w.col_d], hu = ps[pk + w.col_u];
      fw.load(L, w, c.i, c.j, k);
      T above[R];
#pragma unroll
      for (int r = 0; r < R; ++r) above[r] = k + 1 < n ? pa[r] : T(0);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!w.valid[r]) continue;
        const long long p = pk + w.col[r];
        fw.row(L, w, c.i, c.j, k, r);
        const T ap = apply_col3(L, fw, r, centre[r], w.il ? pl[r] : T(0), w.ir ? pr[r] : T(0),
                                           w.down(r, centre, hd), w.up(r, centre, hu), below[r], above[r], s);
        const T bn = bv[r] - a * ap;
        bout[off + p] = bn;
        xout[off + p] = omega * bn / fw.diag(L, r, s);
        rr += (double)bn * (double)bn;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        below[r] = centre[r];
        centre[r] = above[r];
      }
    }
  }
  write_partial_tile(tl, partial, sys, rr);
  finish(fin, partial, sys, gridDim.x * gridDim.y);
}

// --------------------------------------------------------------------------
// b_c = R (b - (A+s) x): full weighting of the fine residual (weights
// (1/4, 1/2, 1/4) per axis), fine node 2I+1 under coarse node I (0-based).
// --------------------------------------------------------------------------
template <typename T, int DIM, bool VAR>
__global__ __launch_bounds__(kBlock) void k_restrict(LevelDev<T> Lf, LevelDev<T> Lc, const T* __restrict__ b,
                                                     const T* __restrict__ x, T* __restrict__ bc,
                                                     const T* __restrict__ shift, const int* __restrict__ active,
                                                     unsigned long long* __restrict__ ctr) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  // per coarse point: b and x on its 2^dim fine points, b_c written
  count_bytes_tile(tl, ctr, (unsigned long long)Lc.N * sizeof(T) * (2 * (1 << DIM) + 1 + (VAR && sys == 0 ? DIM * (1 << DIM) : 0)));
  int I, J, K;
  tile_ijk<DIM>(tl, Lc.n, I, J, K);
  if (I >= Lc.n || J >= Lc.n) return;
  const int nf = Lf.n;
  const T s = shift[sys];
  const T* bs = b + (long long)sys * Lf.N;
  const T* xs = x + (long long)sys * Lf.N;
  const T wt[3] = {T(0.25), T(0.5), T(0.25)};
  T acc = T(0);
  const int kmin = DIM == 3 ? -1 : 0, kmax = DIM == 3 ? 1 : 0;
  for (int dk = kmin; dk <= kmax; ++dk) {
    const int fk = DIM == 3 ? 2 * K + 1 + dk : 0;
    const T wk = DIM == 3 ? wt[dk + 1] : T(1);
    for (int dj = -1; dj <= 1; ++dj) {
      const int fj = 2 * J + 1 + dj;
      for (int di = -1; di <= 1; ++di) {
        const int fi = 2 * I + 1 + di;
        const long long p = ((long long)fk * nf + fj) * nf + fi;
        const T r = bs[p] - apply_pt<T, DIM, VAR>(Lf, xs, fi, fj, fk, p, s, nullptr);
        acc += wk * wt[dj + 1] * wt[di + 1] * r;
      }
    }
  }
  bc[(long long)sys * Lc.N + ((long long)K * Lc.n + J) * Lc.n + I] = acc;
}

// --------------------------------------------------------------------------
// x_f += P x_c  (multilinear interpolation, P = 2^dim R^T)
// --------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ int axis_parents(int f, int nc, int* ci, T* w) {
  if (f & 1) {
    ci[0] = (f - 1) >> 1;
    w[0] = T(1);
    return 1;
  }
  int cnt = 0;
  const int c0 = (f >> 1) - 1, c1 = f >> 1;
  if (c0 >= 0) { ci[cnt] = c0; w[cnt] = T(0.5); ++cnt; }
  if (c1 < nc) { ci[cnt] = c1; w[cnt] = T(0.5); ++cnt; }
  return cnt;
}

template <typename T, int DIM>
__device__ __forceinline__ T interp_pt(const T* __restrict__ xc, int nc, int fi, int fj, int fk) {
  int ci[2], cj[2], ck[2];
  T wi[2], wj[2], wk[2];
  const int ni = axis_parents<T>(fi, nc, ci, wi);
  const int nj = axis_parents<T>(fj, nc, cj, wj);
  int nk = 1;
  ck[0] = 0;
  wk[0] = T(1);
  if (DIM == 3) nk = axis_parents<T>(fk, nc, ck, wk);
  T v = T(0);
  for (int c = 0; c < nk; ++c)
    for (int b = 0; b < nj; ++b)
      for (int a = 0; a < ni; ++a)
        v += wk[c] * wj[b] * wi[a] * xc[((long long)ck[c] * nc + cj[b]) * nc + ci[a]];
  return v;
}

template <typename T, int DIM>
__global__ __launch_bounds__(kBlock) void k_prolong(LevelDev<T> Lc, LevelDev<T> Lf, const T* __restrict__ xc,
                                                    T* __restrict__ xf, const int* __restrict__ active,
                                                    unsigned long long* __restrict__ ctr) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  // x_f read and written; x_c read once (1/2^dim per fine point)
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * 2 + (unsigned long long)Lc.N * sizeof(T));
  int i, j, k;
  tile_ijk<DIM>(tl, Lf.n, i, j, k);
  if (i >= Lf.n || j >= Lf.n) return;
  const long long p = ((long long)k * Lf.n + j) * Lf.n + i;
  xf[(long long)sys * Lf.N + p] += interp_pt<T, DIM>(xc + (long long)sys * Lc.N, Lc.n, i, j, k);
}

// --------------------------------------------------------------------------
// 3D transfer operators marching along z (grids of 2^L - 1 points: n_f = 2 n_c + 1)
// --------------------------------------------------------------------------
// The two coarse parents of fine index f on one axis and their weights: odd f
// lies on coarse point (f - 1) / 2 (weight 1, second weight 0); even f halfway
// between f/2 - 1 and f/2 (weight 1/2 each, 0 for a parent outside the grid,
// whose index is clamped).
template <typename T>
__device__ __forceinline__ void axis_pair(int f, int nc, int& a, int& b, T& wa, T& wb) {
  if (f & 1) {
    a = b = f >> 1;
    wa = T(1);
    wb = T(0);
  } else {
    a = (f >> 1) - 1;
    b = f >> 1;
    wa = a >= 0 ? T(0.5) : T(0);
    wb = b < nc ? T(0.5) : T(0);
    a = max(a, 0);
    b = min(b, nc - 1);
  }
}

// x_f += P x_c: one thread per fine column (i, j) over `planes` (even) fine planes.  The
// in-plane interpolant of each coarse plane is formed once and kept for the
// two or three fine planes that use it.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_prolong3(LevelDev<T> Lc, LevelDev<T> Lf, const T* __restrict__ xc,
                                                     T* __restrict__ xf, const int* __restrict__ active,
                                                     unsigned long long* __restrict__ ctr, int planes) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * 2 + (unsigned long long)Lc.N * sizeof(T));
  const int nf = Lf.n, nc = Lc.n;
  const Column c = march_column(tl, nf, 1, planes);
  if (c.i >= nf || c.j >= nf) return;
  int ia, ib, ja, jb;
  T wia, wib, wja, wjb;
  axis_pair<T>(c.i, nc, ia, ib, wia, wib);
  axis_pair<T>(c.j, nc, ja, jb, wja, wjb);
  const T* xcs = xc + (long long)sys * Lc.N;
  const long long ncc = (long long)nc * nc;
  const long long oaa = (long long)ja * nc + ia, oab = (long long)ja * nc + ib;
  const long long oba = (long long)jb * nc + ia, obb = (long long)jb * nc + ib;
  // the in-plane interpolant on coarse plane K (0 off the grid)
  auto plane = [&](int K) -> T {
    const long long base = (long long)min(max(K, 0), nc - 1) * ncc;
    const T v00 = xcs[base + oaa], v01 = xcs[base + oab], v10 = xcs[base + oba], v11 = xcs[base + obb];
    const T v = wja * (wia * v00 + wib * v01) + wjb * (wia * v10 + wib * v11);
    return (K >= 0 && K < nc) ? v : T(0);
  };
  // fine plane k: odd k lies on coarse plane (k - 1) / 2, even k halfway between
  // k/2 - 1 and k/2; (vlo, vhi) hold coarse planes Kc and Kc + 1
  int Kc = (c.k0 >> 1) - 1;
  T vlo = plane(Kc), vhi = plane(Kc + 1);
  T* xfs = xf + (long long)sys * Lf.N;
  const long long nnf = (long long)nf * nf, col = (long long)c.j * nf + c.i;
  for (int k = c.k0; k < c.k1; ++k) {
    const int klo = (k >> 1) - 1 + (k & 1);
    if (Kc < klo) {
      vlo = vhi;
      ++Kc;
      vhi = plane(Kc + 1);
    }
    const T v = (k & 1) ? vlo : T(0.5) * (vlo + vhi);
    const long long p = k * nnf + col;
    xfs[p] += v;
  }
}

// b_c = R (b - (A+s) x) in 3D.  A workgroup owns kRcx x kRcy coarse columns over
// `planes` coarse planes, i.e. the (2 kRcx + 1) x (2 kRcy + 1) fine columns under
// them.  Plane by plane, each fine point's residual is formed once and put in
// LDS; each coarse column then takes the weighted 3 x 3 sum of its plane, and
// the weighted sums of fine planes 2K, 2K+1, 2K+2 give coarse plane K (plane
// 2K+2 is shared with coarse plane K+1).  Every thread keeps x of its fine
// points at the plane below and at the current one in registers; the current
// plane also goes to an LDS tile with a one-point ring (loaded by the first
// threads), from which the in-plane neighbours are read, so a point costs two
// loads per plane (x above, b) instead of six, and the kernel holds far fewer
// registers (FP32: 98 VGPRs instead of 146, 4 waves per SIMD instead of 3).
constexpr int kRcx = 32, kRcy = 8;
constexpr int kRfx = 2 * kRcx + 1, kRfy = 2 * kRcy + 1, kRfn = kRfx * kRfy;
constexpr int kRhx = kRfx + 2, kRhy = kRfy + 2, kRhn = kRhx * kRhy;   // with the ring
constexpr int kRring = 2 * kRhx + 2 * (kRhy - 2);

static_assert(kRcx * kRcy == 256, "one coarse column per thread");
static_assert(kRring <= 256, "one ring point per thread at most");

template <typename T, bool VAR>
__global__ __launch_bounds__(256) void k_restrict3(LevelDev<T> Lf, LevelDev<T> Lc, const T* __restrict__ b,
                                                   const T* __restrict__ x, T* __restrict__ bc,
                                                   const T* __restrict__ shift, const int* __restrict__ active,
                                                   unsigned long long* __restrict__ ctr, int planes) {
  constexpr int PER = (kRfn + 255) / 256;
  constexpr bool EARLY = sizeof(T) == 4;   // the face weights with the plane's other loads (see ColFaces)
  __shared__ T rb[kRfn];
  __shared__ T xt[kRhn];
  const Tile tl = VAR && sizeof(T) == 4 ? block_tile_shared() : block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lc.N * sizeof(T) * (2 * 8 + 1 + (VAR && sys == 0 ? 3 * 8 : 0)));
  const int nf = Lf.n, nc = Lc.n;
  const int yt = (nc + kRcy - 1) / kRcy;
  const int kc = tl.y / yt;
  const int I0 = tl.x * kRcx, J0 = (tl.y - kc * yt) * kRcy;
  const int K0 = kc * planes, K1 = min(K0 + planes, nc);
  const int tid = threadIdx.x;
  const T s = shift[sys];
  const T* bs = b + (long long)sys * Lf.N;
  const T* xs = x + (long long)sys * Lf.N;
  const long long nnf = (long long)nf * nf;
  int fk = 2 * K0;
  T xm[PER], xc0[PER];   // x at the fine plane below and at the current one, per owned fine point
  T wf[PER];             // the weight of the face below the current plane
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + 256 * u;
    const int fy = q / kRfx, fx = q - fy * kRfx;
    const int fi = 2 * I0 + fx, fj = 2 * J0 + fy;
    xm[u] = T(0);
    xc0[u] = T(0);
    wf[u] = T(0);
    if (q < kRfn && fi < nf && fj < nf) {
      const long long p = fk * nnf + (long long)fj * nf + fi;
      if (VAR && EARLY) wf[u] = Lf.wf2[p];
      const T xb = xs[fk > 0 ? p - nnf : p];
      xm[u] = fk > 0 ? xb : T(0);
      xc0[u] = xs[p];
    }
  }
  // this thread's ring point (tid < kRring): its place in the tile and its
  // in-plane offset (-1 when outside the grid: it holds 0)
  int ring_h = -1;
  long long ring_off = -1;
  if (tid < kRring) {
    int hx, hy;
    if (tid < kRhx) {
      hx = tid;
      hy = 0;
    } else if (tid < 2 * kRhx) {
      hx = tid - kRhx;
      hy = kRhy - 1;
    } else {
      const int t2 = tid - 2 * kRhx;
      hx = (t2 & 1) ? kRhx - 1 : 0;
      hy = 1 + (t2 >> 1);
    }
    ring_h = hy * kRhx + hx;
    const int fi = 2 * I0 - 1 + hx, fj = 2 * J0 - 1 + hy;
    if (fi >= 0 && fi < nf && fj >= 0 && fj < nf) ring_off = (long long)fj * nf + fi;
  }
  const int ci = tid % kRcx, cj = tid / kRcx;
  // the residual on fine plane fk (into LDS), then this coarse column's
  // weighted in-plane sum of it; advances fk and the registers
  auto rplane = [&]() -> T {
    // x of plane fk into the tile (0 off the grid), x above and b loaded
    // (and the faces: see ColFaces)
    T xa[PER], bv[PER];
    ColFaces<T, VAR, 1> fw[PER];
    // faces of the point at offset o1 of the plane (o0: in a plane of wf0); the
    // one below in z is the one above of the plane before (planes of wf0 and
    // wf1 have as many faces)
    auto load_faces = [&](ColFaces<T, VAR, 1>& w, unsigned o1, unsigned o0) {
      const long long f0 = (long long)fk * nf * (nf + 1);
      w.l[0] = plane_at(Lf.wf0 + f0, o0);
      w.r[0] = plane_at(Lf.wf0 + f0, o0 + 1);
      w.d[0] = plane_at(Lf.wf1 + f0, o1);
      w.d[1] = plane_at(Lf.wf1 + f0, o1 + (unsigned)nf);
      w.f[0] = plane_at(Lf.wf2 + (fk + 1) * nnf, o1);
      if (!EARLY) w.b[0] = plane_at(Lf.wf2 + fk * nnf, o1);
    };
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = tid + 256 * u;
      const int fy = q / kRfx, fx = q - fy * kRfx;
      const int fi = 2 * I0 + fx, fj = 2 * J0 + fy;
      const bool in = q < kRfn && fi < nf && fj < nf;
      const unsigned o = in ? (unsigned)(fj * nf + fi) : 0u;
      xa[u] = plane_at(xs + (fk + 1 < nf ? fk + 1 : fk) * nnf, o);
      bv[u] = plane_at(bs + fk * nnf, o);
      if (VAR && EARLY) {
        load_faces(fw[u], o, in ? o + (unsigned)fj : 0u);
        fw[u].b[0] = wf[u];
        wf[u] = fw[u].f[0];
      }
      if (q < kRfn) xt[(fy + 1) * kRhx + fx + 1] = xc0[u];
    }
    if (ring_h >= 0) xt[ring_h] = ring_off >= 0 ? xs[fk * nnf + ring_off] : T(0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = tid + 256 * u;
      const int fy = q / kRfx, fx = q - fy * kRfx;
      const int fi = 2 * I0 + fx, fj = 2 * J0 + fy;
      if (q < kRfn) {
        T r = T(0);
        if (fi < nf && fj < nf) {
          const int h = (fy + 1) * kRhx + fx + 1;
          const T above = fk + 1 < nf ? xa[u] : T(0);
          if (VAR && !EARLY) load_faces(fw[u], (unsigned)(fj * nf + fi), (unsigned)(fj * (nf + 1) + fi));
          r = bv[u] - apply_col3(Lf, fw[u], 0, xc0[u], xt[h - 1], xt[h + 1], xt[h - kRhx], xt[h + kRhx],
                                            xm[u], above, s);
          xm[u] = xc0[u];
          xc0[u] = above;
        }
        rb[q] = r;
      }
    }
    __syncthreads();
    const T wt[3] = {T(0.25), T(0.5), T(0.25)};
    T acc = T(0);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      const int di = q % 3, dj = q / 3;
      acc += wt[dj] * wt[di] * rb[(2 * cj + dj) * kRfx + 2 * ci + di];
    }
    // (the next plane writes rb only after its first barrier, which every
    // thread reaches after this sum)
    ++fk;
    return acc;
  };
  const bool mine = I0 + ci < nc && J0 + cj < nc;
  T* bcs = bc + (long long)sys * Lc.N + ((long long)(J0 + cj) * nc + (I0 + ci));
  const long long ncc = (long long)nc * nc;
  T rlo = rplane();   // fine plane 2 K0
  for (int K = K0; K < K1; ++K) {
    const T rmid = rplane();   // 2K + 1
    const T rhi = rplane();    // 2K + 2
    if (mine) bcs[K * ncc] = T(0.25) * rlo + T(0.5) * rmid + T(0.25) * rhi;
    rlo = rhi;
  }
}

// --------------------------------------------------------------------------
// coarse solve: one V-cycle on the levels in H, one workgroup per system, the
// iterates in LDS.  Symmetric (nu Jacobi sweeps before and after), so the
// composite is an SPD preconditioner component.
//
// Bound by latency: about 40 dependent steps of one LDS round trip each.  So a
// thread owns its points of a level and keeps their right-hand side, face
// weights and inverse diagonal in registers for both halves of the cycle
// (loaded once, before the level's first step); an iterate has two zero-padded
// buffers, read from one and written to the other, which takes one barrier a
// step and no boundary tests; and a coarse point's right-hand side goes
// straight into its owner's registers.  Against the version that walked the
// points of every step in a loop, read the face weights in each sweep and
// copied the iterate back, with variable coefficients: 63^2 FP32, 2048 systems
// 101 -> 87 us a launch, the mean over a solve; 63^2, 8 systems 30 -> 13; 15^3,
// 8 systems 30 -> 15; FP64, 64 systems, 47^2 here (17 us) where 23^2 (21 us)
// and the two level kernels of 47^2 (9 us each) had run.
// --------------------------------------------------------------------------
// weight i of a half-cycle (selected without indexing the array, which would
// put the by-value argument in scratch memory)
template <typename T>
__device__ __forceinline__ T sweep_w(const Sweeps<T>& sw, int i) {
  return i == 0 ? sw.w[0] : (i == 1 ? sw.w[1] : sw.w[2]);
}

// (i, j, k) of point p of an n^DIM grid held in LDS: the quotients by n
// through a float reciprocal instead of an integer division.  Exact: p +
// 0.5 lies at least 0.5/n from every multiple of n, and for the LDS levels
// (p < 2^15) the float rounding error of (p + 0.5) * (1/n) stays below 1e-5.
template <int DIM>
__device__ __forceinline__ void ijk_of(int p, int n, float rn, int& i, int& j, int& k) {
  const int q = (int)(((float)p + 0.5f) * rn);
  i = p - q * n;
  if (DIM == 3) {
    k = (int)(((float)q + 0.5f) * rn);
    j = q - k * n;
  } else {
    j = q;
    k = 0;
  }
}

// x + r d, the product rounded first: fused, the error of a rounded damping or
// diagonal goes into every sweep in the same direction, where x + r d is a tie
// of the rounding (the FP32 preconditioner of 155^2 with constant coefficients,
// whose bottom level takes 312 sweeps, was off by 1.7e-7; so it is by 7.6e-8)
template <typename T>
__device__ __forceinline__ T add_step(T x, T r, T d) {
#pragma clang fp contract(off)
  const T t = r * d;
  return x + t;
}

// The P points of this thread on one LDS level: padded position (a position
// inside the grid for a lane without a point, which computes but does not
// write), face weights and inverse diagonal (an IEEE division, once a level).
// The operator is in its difference form: its rounding goes with the
// differences of neighbours, where (weights x neighbours) - diagonal x rounds
// with x.  Gathered, with the hardware reciprocal, the FP32 preconditioner of
// 155^2 with variable coefficients was off by 5.7e-7; in this form, and with
// the division rounded as IEEE does, by 7.5e-8 (2^-24 is 6.0e-8).
template <typename T, int DIM, bool VAR, int P, int NT>
struct LdsPoints {
  int S1, S2;
  int q[P];
  bool on[P];
  T wc, s, w[VAR ? 2 * DIM : 1][P], di[VAR ? P : 1];
  __device__ __forceinline__ LdsPoints(const LevelDev<T>& L, T shift) {
    const int n = L.n, N = (int)L.N;
    const float rn = 1.0f / (float)n;
    S1 = n + 2;
    S2 = S1 * S1;
    wc = L.wc;
    s = shift;
    if (!VAR) di[0] = T(1) / (wc * T(2 * DIM) + s);
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const int p = threadIdx.x + NT * u;
      on[u] = p < N;
      int i, j, k;
      ijk_of<DIM>(on[u] ? p : 0, n, rn, i, j, k);
      q[u] = ((DIM == 3 ? k + 1 : 0) * S1 + j + 1) * S1 + i + 1;
      if (VAR) {
        const int fx = (k * n + j) * (n + 1) + i, fy = (k * (n + 1) + j) * n + i;
        w[0][u] = L.wf0[fx];
        w[VAR ? 1 : 0][u] = L.wf0[fx + 1];
        w[VAR ? 2 : 0][u] = L.wf1[fy];
        w[VAR ? 3 : 0][u] = L.wf1[fy + n];
        if (DIM == 3) {
          const int fz = (k * n + j) * n + i;
          w[VAR && DIM == 3 ? 4 : 0][u] = L.wf2[fz];
          w[VAR && DIM == 3 ? 5 : 0][u] = L.wf2[fz + n * n];
        }
        T d = w[0][u];
#pragma unroll
        for (int f = 1; f < 2 * DIM; ++f) d += w[VAR ? f : 0][u];
        di[VAR ? u : 0] = T(1) / (d + s);
      }
    }
  }
  __device__ __forceinline__ T inv(int u) const { return di[VAR ? u : 0]; }
  // (A + s) at the point, the arithmetic of apply_pt
  __device__ __forceinline__ T apply(const T* A, int u) const {
    const T* c = A + q[u];
    const T x = c[0];
    if (!VAR) {
      T sum = (x - c[-1]) + (x - c[1]) + (x - c[-S1]) + (x - c[S1]);
      if (DIM == 3) sum += (x - c[-S2]) + (x - c[S2]);
      return wc * sum + s * x;
    }
    T sum = w[0][u] * (x - c[-1]) + w[VAR ? 1 : 0][u] * (x - c[1]) + w[VAR ? 2 : 0][u] * (x - c[-S1]) +
            w[VAR ? 3 : 0][u] * (x - c[S1]);
    if (DIM == 3)
      sum += w[VAR && DIM == 3 ? 4 : 0][u] * (x - c[-S2]) + w[VAR && DIM == 3 ? 5 : 0][u] * (x - c[S2]);
    return sum + s * x;
  }
  // one sweep X -> Y, then they change places
  __device__ __forceinline__ void sweep(T*& X, T*& Y, const T* b, T om) const {
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const T xn = add_step(X[q[u]], om * (b[u] - apply(X, u)), inv(u));
      if (on[u]) Y[q[u]] = xn;
    }
    __syncthreads();
    T* const t = X;
    X = Y;
    Y = t;
  }
};

// One level and everything below it, with the right-hand side b of this
// thread's points; returns the buffer that holds the level's iterate (every
// write of it behind a barrier).  The points are set up again after the coarser
// levels: held across them, the face weights of all levels together spill.
template <typename T, int DIM, bool VAR, int P, int NT, int LV>
__device__ __forceinline__ T* lds_cycle(const LdsHierarchy<T>& H, T* sm, T s, const T* b) {
  const LevelDev<T>& L = H.lev[LV];
  const int n = L.n, S1 = n + 2, S2 = S1 * S1;
  T* X = sm + H.off[LV];
  T* Y = X + (DIM == 3 ? S2 * S1 : S2);
  {
    const LdsPoints<T, DIM, VAR, P, NT> pt(L, s);
    // the first sweep, from zero
    const bool bottom = LV + 1 >= H.nlev;
    const T om0 = bottom ? (L.N == 1 ? T(1) : H.omega) : sweep_w(H.pre, 0);
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (pt.on[u]) X[pt.q[u]] = om0 * b[u] * pt.inv(u);
    __syncthreads();
    if (bottom) {
      if (L.N > 1)
        for (int m = 1; m < H.bottom_sweeps; ++m) pt.sweep(X, Y, b, H.omega);
      return X;
    }
    for (int m = 1; m < H.nu; ++m) pt.sweep(X, Y, b, sweep_w(H.pre, m));
    // the residual into Y
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (pt.on[u]) Y[pt.q[u]] = b[u] - pt.apply(X, u);
    __syncthreads();
  }
  if constexpr (LV + 1 < kMaxLdsLevels) {
    // full weighting of the residual into the coarse right-hand side
    const LevelDev<T>& Lc = H.lev[LV + 1];
    const int nc = Lc.n;
    T bc[1];
    {
      int I, J, K;
      ijk_of<DIM>((int)threadIdx.x < (int)Lc.N ? threadIdx.x : 0, nc, 1.0f / (float)nc, I, J, K);
      const T wt[3] = {T(0.25), T(0.5), T(0.25)};
      const T* c = Y + ((DIM == 3 ? 2 * K + 2 : 0) * S1 + 2 * J + 2) * S1 + 2 * I + 2;
      T acc = T(0);
#pragma unroll
      for (int dk = (DIM == 3 ? -1 : 0); dk <= (DIM == 3 ? 1 : 0); ++dk)
#pragma unroll
        for (int dj = -1; dj <= 1; ++dj)
#pragma unroll
          for (int dx = -1; dx <= 1; ++dx)
            acc += (DIM == 3 ? wt[dk + 1] : T(1)) * wt[dj + 1] * wt[dx + 1] * c[dk * S2 + dj * S1 + dx];
      bc[0] = acc;
    }
    const T* C = lds_cycle<T, DIM, VAR, 1, NT, LV + 1>(H, sm, s, bc);
    const LdsPoints<T, DIM, VAR, P, NT> pt(L, s);
    // x += P x_c: an odd index lies on a coarse point, an even one halfway
    // between two (the padding is the boundary); only this thread's points of X
    // change before the barrier
    const int T1 = nc + 2, T2 = T1 * T1;
    const float rn = 1.0f / (float)n;
#pragma unroll
    for (int u = 0; u < P; ++u) {
      int i, j, k;
      ijk_of<DIM>(pt.on[u] ? threadIdx.x + NT * u : 0, n, rn, i, j, k);
      const int oi = (i & 1) ? 0 : 1, oj = (j & 1) ? 0 : T1, ok = (DIM == 2 || (k & 1)) ? 0 : T2;
      const T* c = C + ((DIM == 3 ? (k + 1) / 2 : 0) * T1 + (j + 1) / 2) * T1 + (i + 1) / 2;
      // an index on a coarse point takes it twice, halved: exact
      T v = T(0.25) * ((c[0] + c[oi]) + (c[oj] + c[oj + oi]));
      if (DIM == 3) v = T(0.5) * (v + T(0.25) * ((c[ok] + c[ok + oi]) + (c[ok + oj] + c[ok + oj + oi])));
      if (pt.on[u]) X[pt.q[u]] += v;
    }
    __syncthreads();
    for (int m = H.nu - 1; m >= 0; --m) pt.sweep(X, Y, b, sweep_w(H.pre, m));
  }
  return X;
}

template <typename T, int DIM, bool VAR, int PER, int NT>
__global__ __launch_bounds__(NT) void k_coarse(LdsHierarchy<T> H, const T* __restrict__ b,
                                                           T* __restrict__ x, const T* __restrict__ shift,
                                                           const int* __restrict__ active,
                                                           unsigned long long* __restrict__ ctr, int elems) {
  extern __shared__ unsigned char smem_raw[];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int sys = blockIdx.x;
  if (!active[sys]) return;
  count_bytes<COUNT_ONE>(ctr, 2ULL * H.lev[0].N * sizeof(T));
  const int n = H.lev[0].n, N = (int)H.lev[0].N;
  const long long off = (long long)sys * N;
  T bv[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) bv[u] = b[off + min((int)threadIdx.x + NT * u, N - 1)];
  for (int i = threadIdx.x; i < elems; i += NT) sm[i] = T(0);
  const T s = shift[sys];
  __syncthreads();
  const T* X = lds_cycle<T, DIM, VAR, PER, NT, 0>(H, sm, s, bv);
  const float rn = 1.0f / (float)n;
  const int S1 = n + 2;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int p = threadIdx.x + NT * u;
    if (p < N) {
      int i, j, k;
      ijk_of<DIM>(p, n, rn, i, j, k);
      x[off + p] = X[((DIM == 3 ? k + 1 : 0) * S1 + j + 1) * S1 + i + 1];
    }
  }
}

// --------------------------------------------------------------------------
// Fused multigrid level kernels with LDS-staged halo tiles (2D).
//
// k_down: from b on level l, nu Jacobi sweeps starting at x = 0, the residual
// r = b - (A+s) x and its full weighting onto level l+1 -- one pass over b,
// writing x (owned points) and b_c.  A block owns a CX x CY tile of coarse
// points, i.e. fine points [2 I0, 2 I0 + 2 CX) per axis (the last tile also
// the final fine point), and stages b on that range widened by nu on each
// side plus one on the right; sweep m is valid on the range shrunk by m-1,
// the residual on the range shrunk by nu = exactly the points the weighting
// needs.  Points outside the grid hold 0 (Dirichlet) and are never updated.
//
// k_up: x = x_in + P x_c on an OX x OY tile widened by nu, nu Jacobi sweeps
// (valid region shrinking by one per sweep), x written on the tile, and the
// block partial of b.x when this is the finest level (r.z for the PCG).
// --------------------------------------------------------------------------
template <typename T, bool VAR>
__device__ __forceinline__ T lds_apply2(const T* __restrict__ X, int q, int RX, const LevelDev<T>& L, int gi, int gj,
                                        T s, T* dg) {
  const T xc = X[q];
  const T xl = X[q - 1], xr = X[q + 1], xd = X[q - RX], xu = X[q + RX];
  if (!VAR) {
    const T w = L.wc;
    if (dg) *dg = w * T(4) + s;
    return w * ((xc - xl) + (xc - xr) + (xc - xd) + (xc - xu)) + s * xc;
  }
  const int n = L.n;
  const long long fx = (long long)gj * (n + 1) + gi;
  const long long fy = (long long)gj * n + gi;
  const T wl = L.wf0[fx], wr = L.wf0[fx + 1], wd = L.wf1[fy], wu = L.wf1[fy + n];
  if (dg) *dg = wl + wr + wd + wu + s;
  return wl * (xc - xl) + wr * (xc - xr) + wd * (xc - xd) + wu * (xc - xu) + s * xc;
}

// Face weights of the LDS region points a thread owns in the fused 2D kernels
// (points tid + 256 u, u < PER), held in registers.  Constant coefficients:
// empty.  Points off the grid hold the weights of the nearest grid point
// (clamped; never used in a sweep).
template <typename T, bool VAR, int PER>
struct RegionFaces {
  T wl[VAR ? PER : 1], wr[VAR ? PER : 1], wd[VAR ? PER : 1], wu[VAR ? PER : 1];
  __device__ __forceinline__ void load(const LevelDev<T>& L, int tid, int RX, int RN, int gx0, int gy0) {
    if (!VAR) return;
    const int n = L.n;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = min(tid + 256 * u, RN - 1);
      const int ry = q / RX, rx = q - ry * RX;
      const int ci = min(max(gx0 + rx, 0), n - 1), cj = min(max(gy0 + ry, 0), n - 1);
      const int fx = cj * (n + 1) + ci;   // 2D faces: fewer than 2^31
      const int fy = cj * n + ci;
      wl[u] = L.wf0[fx];
      wr[u] = L.wf0[fx + 1];
      wd[u] = L.wf1[fy];
      wu[u] = L.wf1[fy + n];
    }
  }
  // D = sum of the faces + s (same order as diag_pt)
  __device__ __forceinline__ T diag(int u, T s) const { return wl[u] + wr[u] + wd[u] + wu[u] + s; }
  // (A + s) x at region point q from LDS values X (row length RX); same
  // arithmetic and order as lds_apply2; *dg = D when dg != nullptr
  __device__ __forceinline__ T apply(int u, const T* X, int q, int RX, T s, T* dg) const {
    const T xc = X[q];
    const T xl = X[q - 1], xr = X[q + 1], xd = X[q - RX], xu = X[q + RX];
    if (dg) *dg = wl[u] + wr[u] + wd[u] + wu[u] + s;
    return wl[u] * (xc - xl) + wr[u] * (xc - xr) + wd[u] * (xc - xd) + wu[u] * (xc - xu) + s * xc;
  }
};

// The fine-level vectors the 2D stencil product and fused level kernels write
// (p_new, q, x; the pre-smoothed iterate and the updated residual; z) are
// stored with the nontemporal hint: each is read again only by a later
// kernel, after more than the last-level cache has streamed through, so
// keeping them out of the caches leaves room for the halo re-reads (measured:
// 2 % faster per solve, the down kernel 5 %).

// Tile shapes of the 2D kernels, one row per launch-shape variant (variant 0
// is the default; a plan may time the others at creation and keep the
// fastest): coarse points per block of the down kernel, fine points per block
// of the up kernel, rows per thread and threads along x (of 256) of the
// stencil product.  The stencil product's default is 128 columns wide: each
// row of a tile then spans 8 cache lines of 128 bytes (FP64) plus one line of
// halo on each side, against 4 plus 2 at 64 columns, which took 3.5 % off its
// time at 1023^2 (256 columns, two rows per thread, was slower: less reuse
// along y).  The down kernel's default region is 133 fine columns wide for
// the same reason (7 % faster than 69 columns); the up kernel stays at 64
// fine columns, where it is faster than at 128.
// Variants 3 and 4 of the stencil product and of the down and up kernels are
// k_spmv_r2 / k_down2r / k_up2r (whole rows, levels of up to 1023 points per
// axis; a larger level runs variant 0 in their place, and the tuner skips
// them there): segments of 128 fine rows (variant 3) or 32 (variant 4, more
// workgroups for launches of few systems; 1023^2 with 30 systems: stencil
// product 121 -> 109 us in FP32 and 229 -> 214 us in FP64, the FP32 up
// kernel 108 -> 92 us, where 128-row segments were slower than the tiles).
constexpr int kDownTile[kTileVariants][2] = {{64, 6}, {32, 8}, {64, 8}, {64, 6}, {64, 6}};
constexpr int kUpTile[kTileVariants][2] = {{64, 16}, {64, 8}, {64, 24}, {64, 16}, {64, 16}};
constexpr int kSpmvTile[kTileVariants][2] = {{4, 128}, {2, 64}, {8, 128}, {4, 128}, {4, 128}};
constexpr int kRowsSeg = 128, kShortRowsSeg = 32;   // fine rows per workgroup
// The marching kernels keep the global loads of the next kRowLead rows in
// flight in a ring of registers: slot s serves steps s, s + kRowLead, ...,
// is used at the start of its step and is refilled after the step's
// barrier with the row kRowLead steps ahead (the barrier keeps the compiler
// from issuing the new load before the old value is used, so the slot stays
// one register and no register copy has to wait on a load).  The loop over
// steps is unrolled by kRowLead so that every slot index is a constant.  A
// load used in the step that issued it (or copied at its end) makes the wave
// wait there for every load in flight: one memory round trip per row.
constexpr int kRowLead = 3;
// the lead of the 3D marching kernels, in planes (a plane's loads are
// several points per thread)
constexpr int kPlaneLead = 2;
// A copy of a value the register allocator cannot merge with its source:
// the ring slot the source came from is free after it, so the refill load
// can go into the same register and no copy at the loop's end waits on it.
// A vector (one system's, or the face weights every system shares) as a
// buffer resource: loads and stores at this lane's byte offset voff (a vector
// register, fixed for the whole march) plus a byte offset soff that is the
// same for the whole workgroup (a scalar register, the row).  Addressing a
// row then costs no per-lane arithmetic, where a 64-bit pointer costs a
// 64-bit add per access.  Rows are clamped; a lane past the grid takes an
// offset out of the resource's range (kOffGrid), as is the second half of the
// last pair of a vector: such loads return 0, element by element, and nothing
// is stored.
constexpr int kBufWord3 = 0x00020000;   // resource word 3: 32-bit data format
constexpr unsigned kOffGrid = 0x80000000u;
template <typename T>
struct RowBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ RowBuf(const T* base, long long count)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, (int)(count * (long long)sizeof(T)), kBufWord3)) {}
  __device__ __forceinline__ T ld(unsigned voff, unsigned soff) const {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  }
  // the elements at voff and behind it (element-aligned is enough)
  __device__ __forceinline__ void ld2(T (&v)[2], unsigned voff, unsigned soff) const {
    if constexpr (sizeof(T) == 4) {
      const auto w = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
      v[0] = __uint_as_float(w[0]);
      v[1] = __uint_as_float(w[1]);
    } else {
      const auto w = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
      v[0] = __hiloint2double((int)w[1], (int)w[0]);
      v[1] = __hiloint2double((int)w[3], (int)w[2]);
    }
  }
  __device__ __forceinline__ void ld3(T (&v)[3], unsigned voff, unsigned soff) const {
    if constexpr (sizeof(T) == 4) {
      const auto w = __builtin_amdgcn_raw_buffer_load_b96(r, voff, soff, 0);
      v[0] = __uint_as_float(w[0]);
      v[1] = __uint_as_float(w[1]);
      v[2] = __uint_as_float(w[2]);
    } else {
      T a[2];
      ld2(a, voff, soff);
      v[0] = a[0];
      v[1] = a[1];
      v[2] = ld(voff + 2 * (unsigned)sizeof(T), soff);
    }
  }
  // NT: the nontemporal hint.  The row kernels run 1 - 2 % faster without it (two
  // rows of odd length share a line); the stencil product of a plan without a
  // fused hierarchy carries it, whose passes after it read other vectors first
  // (256^2 FP64, 512 systems: the vector update 199 -> 188 us, the product 150
  // -> 159).
  template <bool NT = false>
  __device__ __forceinline__ void st2(const T (&v)[2], unsigned voff, unsigned soff) const {
    if constexpr (sizeof(T) == 4) {
      const unsigned __attribute__((ext_vector_type(2))) w = {__float_as_uint(v[0]), __float_as_uint(v[1])};
      __builtin_amdgcn_raw_buffer_store_b64(w, r, voff, soff, NT ? 2 : 0);
    } else {
      const unsigned __attribute__((ext_vector_type(4))) w = {
          (unsigned)__double2loint(v[0]), (unsigned)__double2hiint(v[0]), (unsigned)__double2loint(v[1]),
          (unsigned)__double2hiint(v[1])};
      __builtin_amdgcn_raw_buffer_store_b128(w, r, voff, soff, NT ? 2 : 0);
    }
  }
  template <bool NT = false>
  __device__ __forceinline__ void st(T v, unsigned voff, unsigned soff) const {
    if constexpr (sizeof(T) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, NT ? 2 : 0);
    else
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(unsigned __attribute__((ext_vector_type(2))), v), r,
                                            voff, soff, NT ? 2 : 0);
  }
};

// Runs step(t, slot) for t = t0 .. t1 with slot = (t - t0) mod kRowLead as a
// compile-time constant: whole groups of kRowLead steps in a loop without
// exits (an exit inside the group makes the compiler peel the loop, and the
// waits of the loop then serve the peeled path too), then the remainder.
template <int LEAD, typename Step, int... S>
__device__ __forceinline__ void ring_march_impl(int t0, int t1, Step& step, std::integer_sequence<int, S...>) {
  int tb = t0;
  for (; tb + LEAD - 1 <= t1; tb += LEAD) (step(tb + S, std::integral_constant<int, S>{}), ...);
  const int rem = t1 - tb + 1;
  ((S < rem ? (step(tb + S, std::integral_constant<int, S>{}), 0) : 0), ...);
}
template <int LEAD = kRowLead, typename Step>
__device__ __forceinline__ void ring_march(int t0, int t1, Step step) {
  ring_march_impl<LEAD>(t0, t1, step, std::make_integer_sequence<int, LEAD>{});
}
// the lead of the 2D row kernels, in rows of two columns per thread (even, so
// that a slot has a fixed half of the double-buffered LDS rows)
template <typename T>
constexpr int row_lead() { return sizeof(T) == 8 ? 2 : 4; }
// Before a marching loop starts its ring: every load of the set-up has
// arrived.  The waits inside the loop must suit both the first step and the
// steady state; with set-up loads still in flight they are computed for the
// shorter history before the first step and wait for far more than the
// steady state needs, on every step.
__device__ __forceinline__ void ring_prologue_wait() { __builtin_amdgcn_s_waitcnt(0); }
template <typename T>
__device__ __forceinline__ T ring_take(T v) {
  T o;
  if constexpr (sizeof(T) == 4) asm("v_mov_b32 %0, %1" : "=v"(o) : "v"(v));
  else asm("v_mov_b64 %0, %1" : "=v"(o) : "v"(v));
  return o;
}
constexpr int kRowsMaxN = 1023;
constexpr int kRowsMinN = 255;   // smallest level the row kernels are the default on
// A row kernel's workgroup: its system and row segment, from a launch grid of
// (1, segments, systems): the segments of a system run next to each other.
// Systems first, (systems, segments), so that workgroups running at the same
// time share a segment's face weights in the L2, made the FP64 residual 1 %
// faster but the FP32 row kernels 1 - 2 % slower (511^2, 2048 systems).
struct RowTile {
  int sys, seg, nseg;
};
__device__ __forceinline__ RowTile row_tile() {
  RowTile r;
  r.sys = blockIdx.z;
  r.seg = blockIdx.y;
  r.nseg = gridDim.y;
  return r;
}
static inline dim3 rows_grid(int nseg, int nsys) { return dim3(1, nseg, nsys); }
// profiling: the workgroup of segment 0 of each system counts its bytes
__device__ __forceinline__ void count_bytes_row(const RowTile& rt, unsigned long long* ctr, unsigned long long b) {
  if (ctr == nullptr || threadIdx.x != 0 || rt.seg != 0) return;
  atomicAdd(ctr, b);
}
// whether the stencil product / down / up kernel of a level of n points per
// axis runs k_spmv_r2 / k_down2r / k_up2r in variant tv
static inline bool down_rows(int dim, int n, int tv) {
  const int v = tile_variant(tv);
  return dim == 2 && (v == kRowsVariant || v == kShortRowsVariant) && n <= kRowsMaxN;
}
static inline bool up_rows(int dim, int n, int tv) { return down_rows(dim, n, tv); }
static inline bool spmv_rows(int dim, int n, int tv) { return down_rows(dim, n, tv); }
// threads per workgroup, in waves: one per pair of columns (those three), one
// per column and at least one past the grid (the FP64 residual)
static inline int pair_threads(int n) { return (((n + 1) / 2 + 63) / 64) * 64; }
static inline int rows_threads(int n) { return ((n + 1 + 63) / 64) * 64; }
// fine rows per workgroup of a row variant (the down kernel: half as many coarse rows)
static inline int rows_seg(int tv) { return tile_variant(tv) == kShortRowsVariant ? kShortRowsSeg : kRowsSeg; }

// Reciprocal of a Jacobi diagonal, formed once per point and kernel: the sweeps
// multiply by it.  FP32: the hardware reciprocal (within 1 ulp); FP64: IEEE
// division.  A damped Jacobi sweep with D^-1 off by an ulp is the same
// symmetric smoother up to rounding, and the value is the same for a point in
// every launch shape.
__device__ __forceinline__ float jacobi_recip(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double jacobi_recip(double d) { return 1.0 / d; }

// The fused 2D level kernels are bound by instruction issue (FP32 moves half
// the bytes of FP64 per point with the same instructions), so their sweeps are
// branch-free: every thread updates all of its region points, points off the
// grid carry a zero inverse diagonal and stay exactly 0 (b = 0 there), and the
// LDS array is padded so that the neighbours of every lane's point, the
// unused lanes of the last row of threads included, are inside it (the pads
// hold zeros, everything else finite values).  A sweep's values are exact on
// the range it is valid on (shrinking by one point per sweep) and finite
// garbage outside it, which no valid point reads.  Per-point branches had
// kept one exec mask per point and phase alive, which spilled the scalar
// registers into vector lanes (about 600 lane moves per wave).

// RUP: the right-hand side is first advanced by the PCG step, b = b_old -
// alpha (A + s) p (read from b, written to bout on the owned points, |b|^2 into
// partial), so the vector update of the PCG iteration costs no pass of its
// own.  The product (A + s) p is formed here from p (pv), staged on the region
// widened by one point, with the stencil product's arithmetic: that kernel
// then only dots it with p and stores no q, one vector pass less per
// iteration.  bout must not be b: neighbouring blocks still read b_old in
// their halos.
// (occupancy: for FP32 constant coefficients the compiler is asked for 5
// waves per SIMD; left alone it takes a few registers more and one wave
// less.  Variable coefficients (4 face weights per region point in
// registers) and FP64 spill registers under such a request -- the 64 x 8
// variable-coefficient tile at 4 waves ran at half the speed it has at 3 --
// and are left to the compiler.)
template <typename T, bool VAR, int NU, bool RUP, int CX, int CY>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && !VAR ? 5 : 1))) void k_down2(
    LevelDev<T> Lf, LevelDev<T> Lc, const T* __restrict__ b,
                                               T* __restrict__ xout, T* __restrict__ bc,
                                               const T* __restrict__ shift, const int* __restrict__ active,
                                               Sweeps<T> om, unsigned long long* __restrict__ ctr,
                                               const T* __restrict__ pv, const double* __restrict__ alpha,
                                               T* __restrict__ bout, double* __restrict__ partial, Fin fin) {
  constexpr int RX = 2 * CX + 2 * NU + 1, RY = 2 * CY + 2 * NU + 1, RN = RX * RY;
  // RUP: p on the region widened by one point per side (row length PX),
  // staged in the same LDS array before it takes the iterate
  constexpr int PX = RX + 2, PY = RY + 2, PN = PX * PY;
  constexpr int PER = (RN + 255) / 256, PPER = RUP ? (PN + 255) / 256 : 1;
  // LDS: a zero pad of PAD values before the data, the data at PAD + q, and
  // room after it for the farthest neighbour any lane reads (lanes q >= RN of
  // the last row of threads included); the p layout (row length PX) reaches
  // further than the iterate layout
  constexpr int PAD = (RUP ? PX : RX) + 1;
  constexpr int QMAX = PER * 256 - 1;
  constexpr int PQMAX = RUP ? ((QMAX / RX) + 1) * PX + RX : 0;
  constexpr int HI = (QMAX + RX) > (PQMAX + PX) ? (QMAX + RX) : (PQMAX + PX);
  constexpr int DATA = PER * 256 > (RUP ? PPER * 256 : 0) ? PER * 256 : PPER * 256;
  constexpr int LN = PAD + (HI + 1 > DATA ? HI + 1 : DATA);
  // One LDS array: p (RUP), then the iterate, then the residual.  Thread tid
  // owns region points tid + 256 u (u < PER) throughout and keeps their b,
  // x and 1/D in registers; a sweep reads its neighbours from LDS, and its
  // results are written back after a barrier (a second barrier before the
  // next reads).
  __shared__ T sx[LN];
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * (RUP ? 4 : 2) +
                                   (unsigned long long)Lc.N * sizeof(T) +
                                   (VAR && sys == 0 ? (unsigned long long)Lf.N * sizeof(T) * 2 : 0ULL));
  const T am = RUP ? (T)alpha[sys] : T(0);
  const int nf = Lf.n, nc = Lc.n;
  const int I0 = tl.x * CX, J0 = tl.y * CY;
  const int gx0 = 2 * I0 - NU, gy0 = 2 * J0 - NU;
  const T sh = shift[sys];
  const T dcon = Lf.wc * T(4) + sh;   // the diagonal for constant coefficients
  const T rcon = jacobi_recip(dcon);
  const long long off = (long long)sys * Lf.N;
  const T* __restrict__ bs = b + off;
  const int tid = threadIdx.x;
  // the pads: zeros (the data range is written below before it is read)
  for (int i = tid; i < PAD; i += 256) sx[i] = T(0);
  for (int i = PAD + DATA + tid; i < LN; i += 256) sx[i] = T(0);
  // per point: whether it is on the grid (bit u of `in`); its grid index,
  // clamped into the grid for the loads, is recomputed where needed (held in
  // registers it cost occupancy)
  unsigned in = 0u;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + 256 * u;
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const bool on = q < RN && gi >= 0 && gi < nf && gj >= 0 && gj < nf;
    in |= (on ? 1u : 0u) << u;
  }
  auto gidx = [&](int u) {
    const int q = tid + 256 * u;
    const int ry = q / RX, rx = q - ry * RX;
    return min(max(gy0 + ry, 0), nf - 1) * nf + min(max(gx0 + rx, 0), nf - 1);
  };
  // variable coefficients: the four face weights of each of this thread's
  // region points, loaded once for every sweep and the residual
  RegionFaces<T, VAR, PER> fw;
  fw.load(Lf, tid, RX, RN, gx0, gy0);
  // stage b and the first sweep from x = 0: x1 = omega b / D.  All loads of a
  // thread are issued before any is used, so a wave keeps them all in flight.
  T bl[PER];
  if (RUP) {
    // p first, into LDS (0 off the grid); b is loaded after the barrier, so
    // the two sets of loads do not hold registers at the same time
    const T* __restrict__ ps = pv + off;
    T pl[PPER];
#pragma unroll
    for (int u = 0; u < PPER; ++u) {
      const int q = tid + 256 * u;
      const int py = q / PX, px = q - py * PX;
      const int gi = gx0 - 1 + px, gj = gy0 - 1 + py;
      pl[u] = ps[min(max(gj, 0), nf - 1) * nf + min(max(gi, 0), nf - 1)];
    }
#pragma unroll
    for (int u = 0; u < PPER; ++u) {
      const int q = tid + 256 * u;
      const int py = q / PX, px = q - py * PX;
      const int gi = gx0 - 1 + px, gj = gy0 - 1 + py;
      const bool on = q < PN && gi >= 0 && gi < nf && gj >= 0 && gj < nf;
      sx[PAD + q] = on ? pl[u] : T(0);
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) bl[u] = bs[gidx(u)];
  // 1/D per point (0 off the grid): held for variable coefficients, a select
  // of the one constant value otherwise
  T bv[PER], xv[PER], rdv[VAR ? PER : 1];
  auto rd = [&](int u) { return VAR ? rdv[VAR ? u : 0] : (((in >> u) & 1u) ? rcon : T(0)); };
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + 256 * u;
    const bool on = (in >> u) & 1u;
    T bn = bl[u];
    if (RUP) {
      const int ry = q / RX, rx = q - ry * RX;
      const int pq = PAD + (ry + 1) * PX + (rx + 1);
      const T ap = VAR ? fw.apply(u, sx, pq, PX, sh, nullptr) : lds_apply2<T, false>(sx, pq, PX, Lf, 0, 0, sh, nullptr);
      bn = bl[u] - am * ap;
    }
    bv[u] = on ? bn : T(0);
    if (VAR) rdv[VAR ? u : 0] = on ? jacobi_recip(fw.diag(u, sh)) : T(0);
    xv[u] = sweep_w(om, 0) * bv[u] * rd(u);
  }
  if (RUP) __syncthreads();   // every read of p done before sx takes the iterate
#pragma unroll
  for (int u = 0; u < PER; ++u) sx[PAD + tid + 256 * u] = xv[u];
  __syncthreads();
#pragma unroll
  for (int m = 1; m < NU; ++m) {   // sweep m+1, exact on the range shrunk by m
    const T wm = sweep_w(om, m);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = PAD + tid + 256 * u;
      const T ax = VAR ? fw.apply(u, sx, q, RX, sh, nullptr) : lds_apply2<T, false>(sx, q, RX, Lf, 0, 0, sh, nullptr);
      xv[u] = xv[u] + wm * (bv[u] - ax) * rd(u);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) sx[PAD + tid + 256 * u] = xv[u];
    __syncthreads();
  }
  // owned fine points: [2 I0, 2 I0 + 2 CX) per axis, extended to the grid end on the last tile
  {
    const int hx = (I0 + CX >= nc) ? nf : 2 * (I0 + CX);
    const int hy = (J0 + CY >= nc) ? nf : 2 * (J0 + CY);
    T* __restrict__ xs = xout + off;
    T* __restrict__ bo = RUP ? bout + off : nullptr;
    double rr = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = tid + 256 * u;
      const int ry = q / RX, rx = q - ry * RX;
      const int gi = gx0 + rx, gj = gy0 + ry;
      const bool own = ((in >> u) & 1u) && gi >= 2 * I0 && gi < hx && gj >= 2 * J0 && gj < hy;
      if (own) {
        const int g = gj * nf + gi;
        __builtin_nontemporal_store(xv[u], &xs[g]);
        if (RUP) __builtin_nontemporal_store(bv[u], &bo[g]);
      }
      if (RUP) rr += own ? (double)bv[u] * (double)bv[u] : 0.0;
    }
    if (RUP) {
      write_partial_tile(tl, partial, sys, rr);
      finish(fin, partial, sys, gridDim.x * gridDim.y);
    }
  }
  // residual b - (A + s) x, exact on the range shrunk by NU (fine points
  // 2 I0 .. 2 I0 + 2 CX, all on the grid: the weighting below reads no other),
  // formed from the final iterate in sx and then written over it
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = PAD + tid + 256 * u;
    xv[u] = bv[u] - (VAR ? fw.apply(u, sx, q, RX, sh, nullptr) : lds_apply2<T, false>(sx, q, RX, Lf, 0, 0, sh, nullptr));
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) sx[PAD + tid + 256 * u] = xv[u];
  __syncthreads();
  // full weighting: coarse (I, J) <- fine 2I+1 +- 1
  T* __restrict__ bcs = bc + (long long)sys * Lc.N;
  for (int q2 = tid; q2 < CX * CY; q2 += 256) {
    const int I = I0 + (q2 % CX), J = J0 + (q2 / CX);
    if (I < nc && J < nc) {
      const int cx = 2 * I + 1 - gx0, cy = 2 * J + 1 - gy0;
      const T* R = sx + PAD + cy * RX + cx;
      const T v = T(0.25) * R[0] + T(0.125) * (R[-1] + R[1] + R[-RX] + R[RX]) +
                  T(0.0625) * (R[-RX - 1] + R[-RX + 1] + R[RX - 1] + R[RX + 1]);
      bcs[J * nc + I] = v;
    }
  }
}

template <typename T, bool VAR, int NU, bool DOT, int OX, int OY>
__global__ __launch_bounds__(256) void k_up2(LevelDev<T> Lc, LevelDev<T> Lf, const T* __restrict__ xc,
                                             const T* __restrict__ xin, const T* __restrict__ b, T* __restrict__ xout,
                                             const T* __restrict__ shift, const int* __restrict__ active, Sweeps<T> om,
                                             double* __restrict__ partial, unsigned long long* __restrict__ ctr,
                                             Fin fin) {
  constexpr int RX = OX + 2 * NU, RY = OY + 2 * NU, RN = RX * RY;
  // FP64 constant coefficients: each sweep updates only the points it is
  // exact on (the range shrinking by one per sweep) behind a per-point test.
  // Branch-free, every point in every sweep, this kernel held 114 VGPRs (4
  // waves per SIMD) against 66 (7) and ran 25 % slower at 1023^2; in FP32 and
  // with variable coefficients the branch-free form is the faster one.
  constexpr bool GUARD = sizeof(T) == 8 && !VAR;
  // coarse values under the region, zero-padded: coarse index c at cx0 + (c - c0)
  constexpr int CRX = RX / 2 + 3, CRY = RY / 2 + 3, CRN = CRX * CRY;
  constexpr int PER = (RN + 255) / 256, CPER = (CRN + 255) / 256;
  // the iterate at PAD + q, zero pads around it (branch-free sweeps, as in k_down2)
  constexpr int PAD = RX + 1;
  constexpr int LN = PAD + PER * 256 + RX + 1;
  __shared__ T sx[LN];
  __shared__ T sc[CRN];
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * 3 + (unsigned long long)Lc.N * sizeof(T) +
                                   (VAR && sys == 0 ? (unsigned long long)Lf.N * sizeof(T) * 2 : 0ULL));
  const int nf = Lf.n, nc = Lc.n;
  const int ox0 = tl.x * OX, oy0 = tl.y * OY;
  const int gx0 = ox0 - NU, gy0 = oy0 - NU;
  // smallest coarse index any region point interpolates from (floor division)
  const int cx0 = ((gx0 >= 0) ? gx0 / 2 : -((-gx0 + 1) / 2)) - 1;
  const int cy0 = ((gy0 >= 0) ? gy0 / 2 : -((-gy0 + 1) / 2)) - 1;
  const T sh = shift[sys];
  const T rcon = jacobi_recip(Lf.wc * T(4) + sh);
  const long long off = (long long)sys * Lf.N;
  const T* __restrict__ xcs = xc + (long long)sys * Lc.N;
  const T* __restrict__ bs = b + off;
  const T* __restrict__ xis = xin + off;
  const int tid = threadIdx.x;
  for (int i = tid; i < PAD; i += 256) sx[i] = T(0);
  for (int i = PAD + PER * 256 + tid; i < LN; i += 256) sx[i] = T(0);
  unsigned in = 0u;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + 256 * u;
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const bool on = q < RN && gi >= 0 && gi < nf && gj >= 0 && gj < nf;
    in |= (on ? 1u : 0u) << u;
  }
  auto gidx = [&](int u) {
    const int q = tid + 256 * u;
    const int ry = q / RX, rx = q - ry * RX;
    return min(max(gy0 + ry, 0), nf - 1) * nf + min(max(gx0 + rx, 0), nf - 1);
  };
  RegionFaces<T, VAR, PER> fw;
  fw.load(Lf, tid, RX, RN, gx0, gy0);
  // every global load of the staging phase is issued up front (clamped
  // addresses, selected afterwards): the coarse tile, then b and x_in
  T cl[CPER], bl[PER], xl[PER];
#pragma unroll
  for (int u = 0; u < CPER; ++u) {
    const int q = tid + 256 * u;
    const int cy = q / CRX, cx = q - cy * CRX;
    cl[u] = xcs[min(max(cy0 + cy, 0), nc - 1) * nc + min(max(cx0 + cx, 0), nc - 1)];
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int g = gidx(u);
    bl[u] = bs[g];
    xl[u] = xis[g];
  }
#pragma unroll
  for (int u = 0; u < CPER; ++u) {
    const int q = tid + 256 * u;
    if (q < CRN) {
      const int cy = q / CRX, cx = q - cy * CRX;
      const int I = cx0 + cx, J = cy0 + cy;
      sc[q] = (I >= 0 && I < nc && J >= 0 && J < nc) ? cl[u] : T(0);
    }
  }
  __syncthreads();
  T bv[PER], xv[PER], rdv[VAR ? PER : 1];
  auto rd = [&](int u) { return VAR ? rdv[VAR ? u : 0] : (((in >> u) & 1u) ? rcon : T(0)); };
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    // lanes past the region interpolate at its last point (in range of sc)
    const int q = min(tid + 256 * u, RN - 1);
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const bool on = (in >> u) & 1u;
    // multilinear interpolation from the zero-padded coarse tile
    const int ia = (gi & 1) ? (gi - 1) / 2 : gi / 2 - 1;
    const int ja = (gj & 1) ? (gj - 1) / 2 : gj / 2 - 1;
    const T* C = sc + (ja - cy0) * CRX + (ia - cx0);
    T v;
    if (gi & 1) {
      v = (gj & 1) ? C[0] : T(0.5) * (C[0] + C[CRX]);
    } else {
      v = (gj & 1) ? T(0.5) * (C[0] + C[1]) : T(0.25) * (C[0] + C[1] + C[CRX] + C[CRX + 1]);
    }
    bv[u] = on ? bl[u] : T(0);
    xv[u] = on ? xl[u] + v : T(0);
    if (VAR) rdv[VAR ? u : 0] = on ? jacobi_recip(fw.diag(u, sh)) : T(0);
    sx[PAD + tid + 256 * u] = xv[u];
  }
  __syncthreads();
#pragma unroll
  for (int m = 1; m <= NU; ++m) {   // post-smoothing: the pre-smoothing weights reversed
    const T wm = sweep_w(om, NU - m);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = PAD + tid + 256 * u;
      if (GUARD) {   // only the points the sweep is exact on
        const int qq = tid + 256 * u;
        const int ry = qq / RX, rx = qq - ry * RX;
        if (((in >> u) & 1u) && rx >= m && rx < RX - m && ry >= m && ry < RY - m)
          xv[u] = xv[u] + wm * (bv[u] - lds_apply2<T, false>(sx, q, RX, Lf, 0, 0, sh, nullptr)) * rcon;
        continue;
      }
      const T ax = VAR ? fw.apply(u, sx, q, RX, sh, nullptr) : lds_apply2<T, false>(sx, q, RX, Lf, 0, 0, sh, nullptr);
      xv[u] = xv[u] + wm * (bv[u] - ax) * rd(u);
    }
    if (m < NU) {   // the last sweep's values are written out from registers
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) sx[PAD + tid + 256 * u] = xv[u];
      __syncthreads();
    }
  }
  double dot = 0.0;
  T* __restrict__ xs = xout + off;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + 256 * u;
    const int ry = q / RX, rx = q - ry * RX;
    const bool own = ((in >> u) & 1u) && rx >= NU && rx < NU + OX && ry >= NU && ry < NU + OY;
    if (own) __builtin_nontemporal_store(xv[u], &xs[(gy0 + ry) * nf + gx0 + rx]);
    if (DOT) dot += own ? (double)bv[u] * (double)xv[u] : 0.0;
  }
  if (DOT) {
    write_partial_tile(tl, partial, sys, dot);
    finish(fin, partial, sys, gridDim.x * gridDim.y);
  }
}

// --------------------------------------------------------------------------
// The 2D row kernels march along y over whole grid rows with two columns per
// thread: thread i has columns 2i and 2i + 1 in registers, and what it needs
// from its neighbours (the odd column of thread i - 1, the even one of thread
// i + 1) goes through LDS, double-buffered by the parity of the step, so that a
// row takes one barrier.  Thread i's LDS record is RowRec<T, ...> values wide,
// an odd number, so that a wave's accesses fall in different banks; the records
// before the first and behind the last thread stay 0 (columns off the grid).
// With one column per thread, two barriers and every face weight loaded twice
// (a face belongs to two columns and two rows) these kernels were bound by
// instruction issue: the up kernel of 511^2 took 58 vector, 63 scalar and 10
// memory instructions per row and wave.
// --------------------------------------------------------------------------
constexpr int kRowThreads = 512;   // pairs of columns: kRowsMaxN at most
extern __shared__ double row_lds[];   // (NT + 2) records

// LDS records of a row kernel with `words` values a thread and step
constexpr int row_rec(int words) { return 2 * words + 1; }
// (more than 64 KiB, which FP64 with three sweeps takes at 1023 columns, has to be asked for)
template <typename T, typename Kernel>
static inline size_t row_lds_bytes(Kernel* kern, int words, int threads) {
  const size_t bytes = (size_t)(threads + 2) * row_rec(words) * sizeof(T);
  if (bytes > 64 * 1024)
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  return bytes;
}
constexpr int down_words(int nu, bool rup) { return 2 * nu + 1 + (rup ? 2 : 0); }
constexpr int up_words(int nu) { return 2 * (2 * nu - 1); }
constexpr int spmv_words() { return 2; }

// What the row kernels share: a thread's pair of columns and the loads of the
// operator's rows.  l: the faces left of the pair, between and right of it;
// u: the faces above (below a row: u of the row before).
template <typename T, bool VAR>
struct RowPair {
  int n, i;
  bool on[2];         // the columns are on the grid
  unsigned cb;        // byte offset of the pair in a row (kOffGrid: none)
  unsigned rowb;      // bytes per row
  T m1;               // 1 where the odd column is on the grid, else 0
  RowBuf<T> w0, w1;
  struct Faces { T l[3], u[2]; };
  __device__ __forceinline__ RowPair(const LevelDev<T>& L, const T* any)
      : n(L.n), i(threadIdx.x), on{2 * (int)threadIdx.x < L.n, 2 * (int)threadIdx.x + 1 < L.n},
        cb(on[0] ? 2 * threadIdx.x * (unsigned)sizeof(T) : kOffGrid), rowb((unsigned)L.n * (unsigned)sizeof(T)),
        m1(on[1] ? T(1) : T(0)), w0(VAR ? L.wf0 : any, VAR ? (long long)(L.n + 1) * L.n : 1),
        w1(VAR ? L.wf1 : any, VAR ? (long long)(L.n + 1) * L.n : 1) {}
  __device__ __forceinline__ unsigned row(int r) const { return (unsigned)min(max(r, 0), n - 1) * rowb; }
  __device__ __forceinline__ bool in(int r) const { return r >= 0 && r < n; }
  // faces of row r (clamped; the faces above row -1 are those below row 0)
  __device__ __forceinline__ void faces(Faces& f, int r) const {
    if (VAR) {
      w0.ld3(f.l, cb, (unsigned)min(max(r, 0), n - 1) * (rowb + (unsigned)sizeof(T)));
      above(f.u, r);
    }
  }
  __device__ __forceinline__ void above(T (&u)[2], int r) const {
    if (VAR) w1.ld2(u, cb, (unsigned)min(max(r + 1, 0), n) * rowb);
  }
  // stores the columns that are on the grid
  template <bool NT = false>
  __device__ __forceinline__ void store(const RowBuf<T>& b, const T (&v)[2], int r) const {
    if (on[1]) b.template st2<NT>(v, cb, (unsigned)r * rowb);
    else if (on[0]) b.template st<NT>(v[0], cb, (unsigned)r * rowb);
  }
};

// (A + s) x at the pair from its row x, the values left and right of it, below
// and above (f: the row's faces, d: those below; the flux form of apply_pt)
template <typename T, bool VAR>
__device__ __forceinline__ void pair_apply(T (&y)[2], const typename RowPair<T, VAR>::Faces& f, const T (&d)[2],
                                           const T (&x)[2], T left, T right, const T (&dn)[2], const T (&up)[2], T wc,
                                           T sh) {
  const T e[2][2] = {{left, x[1]}, {x[0], right}};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (!VAR)
      y[c] = wc * ((x[c] - e[c][0]) + (x[c] - e[c][1]) + (x[c] - dn[c]) + (x[c] - up[c])) + sh * x[c];
    else
      y[c] = f.l[c] * (x[c] - e[c][0]) + f.l[c + 1] * (x[c] - e[c][1]) + d[c] * (x[c] - dn[c]) +
             f.u[c] * (x[c] - up[c]) + sh * x[c];
  }
}

// One damped Jacobi update x + w (b - (A + s) x) / diag at the pair, written as
// x + w ((b + the neighbours' face-weighted sum) / diag - x): diag holds every
// face weight and the shift, so the two agree in exact arithmetic, and this
// form takes 6 instead of 12 vector operations per point (the residual keeps
// the difference form).  r: 1 / diag, 0 off the grid, where x stays exactly 0.
template <typename T, bool VAR>
__device__ __forceinline__ void pair_relax(T (&y)[2], const typename RowPair<T, VAR>::Faces& f, const T (&d)[2],
                                           const T (&x)[2], T left, T right, const T (&dn)[2], const T (&up)[2], T wc,
                                           const T (&b)[2], T w, const T (&r)[2]) {
  const T e[2][2] = {{left, x[1]}, {x[0], right}};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const T nb = VAR ? b[c] + f.l[c] * e[c][0] + f.l[c + 1] * e[c][1] + d[c] * dn[c] + f.u[c] * up[c]
                     : b[c] + wc * ((e[c][0] + e[c][1]) + (dn[c] + up[c]));
    y[c] = x[c] + w * (r[c] * nb - x[c]);
  }
}

template <typename T, bool VAR>
__device__ __forceinline__ void pair_recip(T (&r)[2], const RowPair<T, VAR>& pr, bool in,
                                           const typename RowPair<T, VAR>::Faces& f, const T (&d)[2], T sh, T rcon) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const T v = VAR ? jacobi_recip(f.l[c] + f.l[c + 1] + d[c] + f.u[c] + sh) : rcon;
    r[c] = in && pr.on[c] ? v : T(0);
  }
}

// --------------------------------------------------------------------------
// k_down2r: the down kernel of k_down2 (same inputs and outputs) on whole grid
// rows.  A workgroup owns the fine rows of ky coarse rows (a launch parameter);
// it walks up its rows with the stages lagging one row behind each other, as
// the 3D kernels walk up their planes: at step t row t of b (RUP: b_old -
// alpha (A + s) p, p of rows t - 1 .. t + 1) enters, the first sweep is formed
// on it pointwise, sweep m + 1 on row t - m, the residual on row t - NU, and
// the full weighting of coarse row K once the residual of fine row 2K + 2 is
// there.  The rows below and above stay in registers.  A workgroup starts NU
// rows below its first owned row (warm-up), so every row it writes is exact.
// There is no halo across columns and none along y beyond the warm-up rows,
// where the tiles of k_down2 fetch 1.4 - 1.8 times their points (halo rows and
// columns, partial cache lines) and sweep that many.  Columns and rows outside
// the grid have a zero inverse diagonal, so they stay exactly 0.  With xout
// == nullptr the pre-smoothed iterate is not stored (the level's up kernel is
// k_up2r, which forms it again).
// --------------------------------------------------------------------------
template <typename T, bool VAR, int NU, bool RUP>
__global__ __launch_bounds__(kRowThreads) void k_down2r(LevelDev<T> Lf, LevelDev<T> Lc, const T* __restrict__ b,
                                                 T* __restrict__ xout, T* __restrict__ bc,
                                                 const T* __restrict__ shift, const int* __restrict__ active,
                                                 Sweeps<T> om, unsigned long long* __restrict__ ctr,
                                                 const T* __restrict__ pv, const double* __restrict__ alpha,
                                                 T* __restrict__ bout, double* __restrict__ partial, Fin fin,
                                                 int ky) {
  // a thread's LDS values per step: sweep m's pair at 2m, the even residual at
  // RES, p's pair at PV
  constexpr int WORDS = down_words(NU, RUP), REC = row_rec(WORDS), RES = 2 * NU, PV = RES + 1;
  constexpr int LEAD = row_lead<T>();
  const RowTile rt = row_tile();
  const int sys = rt.sys;
  if (!active[sys]) return;
  const bool keepx = xout != nullptr;
  count_bytes_row(rt, ctr, (unsigned long long)Lf.N * sizeof(T) * ((RUP ? 3 : 1) + (keepx ? 1 : 0)) +
                                   (unsigned long long)Lc.N * sizeof(T) +
                                   (VAR && sys == 0 ? (unsigned long long)Lf.N * sizeof(T) * 2 : 0ULL));
  const int nf = Lf.n, nc = Lc.n;
  const int K0 = rt.seg * ky, K1 = min(K0 + ky, nc);
  const int f1 = K1 == nc ? nf : 2 * K1;   // owned fine rows [2 K0, f1) (the last segment: the top one too)
  const int i = threadIdx.x, NT = blockDim.x;
  const T sh = shift[sys];
  const T rcon = jacobi_recip(Lf.wc * T(4) + sh);
  const T am = RUP ? (T)alpha[sys] : T(0);
  const long long off = (long long)sys * Lf.N;
  const RowPair<T, VAR> pr(Lf, b + off);
  const RowBuf<T> bsb(b + off, Lf.N), psb((RUP ? pv : b) + off, Lf.N), xsb((keepx ? xout : bc) + (keepx ? off : 0), keepx ? Lf.N : 0),
      bob((RUP ? bout : bc) + (RUP ? off : 0), RUP ? Lf.N : 0);
  typedef typename RowPair<T, VAR>::Faces Faces;
  T* lds = reinterpret_cast<T*>(row_lds);
  for (int j = i; j < (NT + 2) * REC; j += NT) lds[j] = T(0);
  T* rec = lds + (i + 1) * REC;
  const int t0 = 2 * K0 - NU, t1 = 2 * K1 + NU;
  // registers: bh[d] = b of row t - d; xh[m][0], xh[m][1] = sweep m+1's output
  // at its newest row of the previous step and the one below; fw[d], rd[d] =
  // faces and inverse diagonal of row t - d (fw[d + 1].u: the faces below it)
  T bh[NU + 1][2], xh[NU][2][2], rd[NU + 1][2];
  Faces fw[NU + 2];
#pragma unroll
  for (int d = 0; d <= NU + 1; ++d) {
    fw[d] = Faces{};
    if (d <= NU) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bh[d][c] = T(0);
        rd[d][c] = T(0);
        if (d < NU) xh[d][0][c] = xh[d][1][c] = T(0);
      }
    }
  }
  // the faces of the rows before the first step (valid where a sweep uses them)
#pragma unroll
  for (int d = 0; d <= NU; ++d) pr.faces(fw[d], t0 - 1 - d);
  __syncthreads();
  // p of rows t - 1, t, t + 1 (RUP; 0 outside the grid) during step t, p(t)
  // also in LDS; before the first step they hold rows t0 - 1 and t0
  T pm[2] = {T(0), T(0)}, pc[2] = {T(0), T(0)}, pa[2] = {T(0), T(0)};
  if (RUP) {
    psb.ld2(pc, pr.cb, pr.row(t0 - 1));
    psb.ld2(pa, pr.cb, pr.row(t0));
    const T mc = pr.in(t0 - 1) ? T(1) : T(0), ma = pr.in(t0) ? T(1) : T(0);
    pc[0] *= mc;
    pc[1] *= mc * pr.m1;
    pa[0] *= ma;
    pa[1] *= ma * pr.m1;
    rec[WORDS + PV] = pa[0];   // the half that step t0 reads
    rec[WORDS + PV + 1] = pa[1];
  }
  // the coarse column of this thread (threads I < nc) and its weighted
  // in-row sums of the residual on fine rows 2K and 2K + 1
  const bool restricts = i < nc;
  T s_lo = T(0), s_mid = T(0);
  const RowBuf<T> bcb(bc + (long long)sys * Lc.N, Lc.N);
  const unsigned cbc = restricts ? (unsigned)i * (unsigned)sizeof(T) : kOffGrid;   // this lane's coarse column
  double rr = 0.0;
  ring_prologue_wait();
  __syncthreads();
  // the ring of row loads (see kRowLead): slot s of step t holds b and the
  // faces of row t and p of row t + 1, as loaded (clamped rows, unmasked)
  T rb[LEAD][2], rp[LEAD][2];
  Faces rf[LEAD];
  auto fill = [&](int t, int s) {
    bsb.ld2(rb[s], pr.cb, pr.row(t));
    pr.faces(rf[s], t);
    if (RUP) psb.ld2(rp[s], pr.cb, pr.row(t + 1));
  };
#pragma unroll
  for (int s = 0; s < LEAD; ++s) fill(t0 + s, s);
  ring_march<LEAD>(t0, t1, [&](int t, auto slot) {
    constexpr int s = decltype(slot)::value;
    constexpr int WR = (s & 1) * WORDS, RD = WORDS - WR;   // the record's halves of this step and the one before
#pragma unroll
    for (int d = NU + 1; d > 0; --d) fw[d] = fw[d - 1];
#pragma unroll
    for (int d = NU; d > 0; --d)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bh[d][c] = bh[d - 1][c];
        rd[d][c] = rd[d - 1][c];
      }
    if (VAR) {
#pragma unroll
      for (int c = 0; c < 3; ++c) fw[0].l[c] = ring_take(rf[s].l[c]);
#pragma unroll
      for (int c = 0; c < 2; ++c) fw[0].u[c] = ring_take(rf[s].u[c]);
    }
    pair_recip<T, VAR>(rd[0], pr, pr.in(t), fw[0], fw[1].u, sh, rcon);
    if (RUP) {
      const T m = pr.in(t + 1) ? T(1) : T(0);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        pm[c] = pc[c];
        pc[c] = pa[c];
      }
      pa[0] = rp[s][0] * m;
      pa[1] = rp[s][1] * (m * pr.m1);
    }
    bh[0][0] = rb[s][0];
    bh[0][1] = rb[s][1];
    if (RUP) {
      T q[2];
      pair_apply<T, VAR>(q, fw[0], fw[1].u, pc, rec[RD + PV + 1 - REC], rec[RD + PV + REC], pm, pa, Lf.wc, sh);
#pragma unroll
      for (int c = 0; c < 2; ++c) bh[0][c] -= am * q[c];
      if (t >= 2 * K0 && t < f1) {
        pr.store(bob, bh[0], t);
        const double r0 = (double)bh[0][0], r1 = (double)(bh[0][1] * pr.m1);   // (lanes past the grid: 0)
        rr += r0 * r0;
        rr += r1 * r1;
      }
    }
    // sweep 1 on row t from x = 0; sweep m + 1 on row t - m from sweep m's
    // output (centre row in xh and LDS, below in xh, above just formed)
    T xn[NU][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) xn[0][c] = sweep_w(om, 0) * bh[0][c] * rd[0][c];
#pragma unroll
    for (int m = 1; m < NU; ++m)
      pair_relax<T, VAR>(xn[m], fw[m], fw[m + 1].u, xh[m - 1][0], rec[RD + 2 * m - 1 - REC], rec[RD + 2 * m - 2 + REC],
                         xh[m - 1][1], xn[m - 1], Lf.wc, bh[m], sweep_w(om, m), rd[m]);
    // the residual on row t - NU
    T res[2];
    pair_apply<T, VAR>(res, fw[NU], fw[NU + 1].u, xh[NU - 1][0], rec[RD + 2 * NU - 1 - REC],
                       rec[RD + 2 * NU - 2 + REC], xh[NU - 1][1], xn[NU - 1], Lf.wc, sh);
#pragma unroll
    for (int c = 0; c < 2; ++c) res[c] = bh[NU][c] - res[c];
    // the pre-smoothed iterate: sweep NU's newest row t - NU + 1
    const int gx = t - NU + 1;
    if (keepx && gx >= 2 * K0 && gx < f1) pr.store(xsb, xn[NU - 1], gx);
#pragma unroll
    for (int m = 0; m < NU; ++m)
#pragma unroll
      for (int c = 0; c < 2; ++c) rec[WR + 2 * m + c] = xn[m][c];
    rec[WR + RES] = res[0];
    if (RUP) {   // p(t + 1), the centre row of the next step
      rec[WR + PV] = pa[0];
      rec[WR + PV + 1] = pa[1];
    }
    __syncthreads();
    fill(t + LEAD, s);   // refill the slot with the rows LEAD steps ahead
    // full weighting: this coarse column's in-row sum of fine row f = t - NU
    // (fine columns 2I .. 2I + 2), and coarse row K = f/2 - 1 once f = 2K + 2
    // (weights 1/4, 1/2, 1/4 along y)
    const int f = t - NU;
    if (f >= 2 * K0) {
      const T acc = T(0.25) * res[0] + T(0.5) * res[1] + T(0.25) * rec[WR + RES + REC];
      const bool odd = f & 1;
      if (restricts && !odd && f != 2 * K0) {
        const int K = f / 2 - 1;
        bcb.st(T(0.25) * s_lo + T(0.5) * s_mid + T(0.25) * acc, cbc, (unsigned)K * (unsigned)nc * (unsigned)sizeof(T));
      }
      // selects, not stores in two branches: the compiler would merge those
      // into one store through a pointer and keep both sums in scratch memory
      s_mid = odd ? acc : s_mid;
      s_lo = odd ? s_lo : acc;
    }
#pragma unroll
    for (int m = 0; m < NU; ++m)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        xh[m][1][c] = xh[m][0][c];
        xh[m][0][c] = xn[m][c];
      }
  });
  if (RUP) {
    write_partial(partial, sys, rr, rt.seg, rt.nseg);
    finish(fin, partial, sys, rt.nseg);
  }
}

// k_up2r: the up kernel of k_up2 (same output; its sweeps in the form of
// pair_relax, equal in exact arithmetic) on whole grid rows, as k_down2r,
// without reading the pre-smoothed iterate: it forms it again from b, as the
// down kernel did (NU sweeps from zero, the same weights and order), so the
// down kernel of the level need not store it (8 bytes per point in FP32 less
// for the pair, 30 -> 22).  2 NU stages lag one row behind each other: at step
// t row t of b enters, pre-sweep k + 1 runs on row t - k (k < NU; the first one
// pointwise), the last of them adds P x_c, and post-sweep m on row
// t - NU + 1 - m (the pre-smoothing weights reversed); post-sweep NU's row
// t - 2 NU + 1 is written on the owned rows [rows s, rows (s + 1)) of
// segment s (rows: a launch parameter), with b.x when this is the finest
// level.  The even column of thread i lies between coarse columns i - 1 and i,
// the odd one on coarse column i; fine row r takes coarse row r / 2 (rounded
// down), an even one the mean with the coarse row before it, which is the row
// that the step before took.
template <typename T, bool VAR, int NU, bool DOT>
__global__ __launch_bounds__(kRowThreads) void k_up2r(LevelDev<T> Lc, LevelDev<T> Lf, const T* __restrict__ xc,
                                               const T* __restrict__ xin, const T* __restrict__ b,
                                               T* __restrict__ xout, const T* __restrict__ shift,
                                               const int* __restrict__ active, Sweeps<T> om,
                                               double* __restrict__ partial, unsigned long long* __restrict__ ctr,
                                               Fin fin, int rows) {
  (void)xin;
  constexpr int NS = 2 * NU;   // stages: NU pre-sweeps (the last one adds P x_c), NU post-sweeps
  constexpr int WORDS = up_words(NU), REC = row_rec(WORDS);   // LDS: the pairs of stages 0 .. NS - 2
  constexpr int LEAD = row_lead<T>();
  const RowTile rt = row_tile();
  const int sys = rt.sys;
  if (!active[sys]) return;
  count_bytes_row(rt, ctr, (unsigned long long)Lf.N * sizeof(T) * 2 + (unsigned long long)Lc.N * sizeof(T) +
                                   (VAR && sys == 0 ? (unsigned long long)Lf.N * sizeof(T) * 2 : 0ULL));
  const int nf = Lf.n, nc = Lc.n;
  const int y0 = rt.seg * rows, y1 = min(y0 + rows, nf);   // owned fine rows
  const int i = threadIdx.x, NT = blockDim.x;
  const T sh = shift[sys];
  const T rcon = jacobi_recip(Lf.wc * T(4) + sh);
  const long long off = (long long)sys * Lf.N;
  const RowPair<T, VAR> pr(Lf, b + off);
  const RowBuf<T> xcb(xc + (long long)sys * Lc.N, Lc.N), bsb(b + off, Lf.N), xsb(xout + off, Lf.N);
  typedef typename RowPair<T, VAR>::Faces Faces;
  T* lds = reinterpret_cast<T*>(row_lds);
  for (int j = i; j < (NT + 2) * REC; j += NT) lds[j] = T(0);
  T* rec = lds + (i + 1) * REC;
  // coarse columns i - 1 and i (0 outside the coarse grid)
  const unsigned ca0 = i >= 1 && i - 1 < nc ? (unsigned)(i - 1) * (unsigned)sizeof(T) : kOffGrid,
                 ca1 = i < nc ? (unsigned)i * (unsigned)sizeof(T) : kOffGrid;
  auto load_c = [&](int r, T (&v)[2]) {   // of fine row r
    const unsigned ko = (unsigned)min(max(r >> 1, 0), nc - 1) * (unsigned)nc * (unsigned)sizeof(T);
    v[0] = xcb.ld(ca0, ko);
    v[1] = xcb.ld(ca1, ko);
  };
  // their in-row interpolation at the pair's columns (0 off the coarse rows)
  auto interp = [&](int r, const T (&v)[2], T (&h)[2]) {
    const T k = (r >> 1) >= 0 && (r >> 1) < nc ? T(0.5) : T(0);
    h[0] = k * (v[0] + v[1]);
    h[1] = (k + k) * v[1];
  };
  const int t0 = y0 - (NS - 1), t1 = y1 + NS - 2;
  // registers: bh[d], fw[d], rd[d] = b, faces and inverse diagonal of row
  // t - d (fw[d + 1].u: the faces below it); xh[k][0], xh[k][1] = stage k's
  // output at its newest row of the previous step and the one below
  T bh[NS][2], xh[NS - 1][2][2], rd[NS][2], hp[2], hc[2];
  Faces fw[NS + 1];
#pragma unroll
  for (int d = 0; d <= NS; ++d) fw[d] = Faces{};
#pragma unroll
  for (int d = 0; d < NS; ++d) {
    pr.faces(fw[d], t0 - 1 - d);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bh[d][c] = T(0);
      rd[d][c] = T(0);
      if (d < NS - 1) xh[d][0][c] = xh[d][1][c] = T(0);
    }
  }
  {
    T v[2];
    load_c(t0 - NU, v);   // the row before the first one that P x_c is added on
    interp(t0 - NU, v, hc);
  }
  double dot = 0.0;
  ring_prologue_wait();
  __syncthreads();
  // the ring of row loads (see kRowLead): slot s of step t holds b and the
  // faces of row t and the coarse values of the row t - NU + 1 where P x_c is
  // added, as loaded
  T rb[LEAD][2], rc[LEAD][2];
  Faces rf[LEAD];
  auto fill = [&](int t, int s) {
    bsb.ld2(rb[s], pr.cb, pr.row(t));
    pr.faces(rf[s], t);
    load_c(t - (NU - 1), rc[s]);
  };
#pragma unroll
  for (int s = 0; s < LEAD; ++s) fill(t0 + s, s);
  ring_march<LEAD>(t0, t1, [&](int t, auto slot) {
    constexpr int s = decltype(slot)::value;
    constexpr int WR = (s & 1) * WORDS, RD = WORDS - WR;   // the record's halves of this step and the one before
#pragma unroll
    for (int d = NS; d > 0; --d) fw[d] = fw[d - 1];
#pragma unroll
    for (int d = NS - 1; d > 0; --d)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bh[d][c] = bh[d - 1][c];
        rd[d][c] = rd[d - 1][c];
      }
    if (VAR) {
#pragma unroll
      for (int c = 0; c < 3; ++c) fw[0].l[c] = ring_take(rf[s].l[c]);
#pragma unroll
      for (int c = 0; c < 2; ++c) fw[0].u[c] = ring_take(rf[s].u[c]);
    }
    pair_recip<T, VAR>(rd[0], pr, pr.in(t), fw[0], fw[1].u, sh, rcon);
    bh[0][0] = rb[s][0];
    bh[0][1] = rb[s][1];
    // P x_c on row r = t - NU + 1
    const int r = t - (NU - 1);
    hp[0] = hc[0];
    hp[1] = hc[1];
    interp(r, rc[s], hc);
    const T kp = (r & 1) ? T(0) : T(0.5), kc = T(1) - kp;
    // stage k on row t - k from stage k - 1's output (centre row in xh and
    // LDS, below in xh, above just formed); the pre-sweeps are those of the
    // down kernel (zero start, the first one pointwise)
    T xn[NS][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) xn[0][c] = sweep_w(om, 0) * bh[0][c] * rd[0][c];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      if (k > 0)
        pair_relax<T, VAR>(xn[k], fw[k], fw[k + 1].u, xh[k - 1][0], rec[RD + 2 * k - 1 - REC],
                           rec[RD + 2 * k - 2 + REC], xh[k - 1][1], xn[k - 1], Lf.wc, bh[k],
                           k < NU ? sweep_w(om, k) : sweep_w(om, NS - 1 - k), rd[k]);
      if (k == NU - 1) {   // x_pre + P x_c
        const bool in = pr.in(r);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const T v = xn[k][c] + (kp * hp[c] + kc * hc[c]);
          xn[k][c] = in && pr.on[c] ? v : T(0);
        }
      }
    }
    const int g = t - (NS - 1);
    if (g >= y0 && g < y1) {
      pr.store(xsb, xn[NS - 1], g);
      if (DOT) {
        dot += (double)bh[NS - 1][0] * (double)xn[NS - 1][0];   // (x is 0 off the grid)
        dot += (double)bh[NS - 1][1] * (double)xn[NS - 1][1];
      }
    }
#pragma unroll
    for (int k = 0; k < NS - 1; ++k)
#pragma unroll
      for (int c = 0; c < 2; ++c) rec[WR + 2 * k + c] = xn[k][c];
    __syncthreads();
    fill(t + LEAD, s);   // refill the slot with row t + LEAD
#pragma unroll
    for (int k = 0; k < NS - 1; ++k)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        xh[k][1][c] = xh[k][0][c];
        xh[k][0][c] = xn[k][c];
      }
  });
  if (DOT) {
    write_partial(partial, sys, dot, rt.seg, rt.nseg);
    finish(fin, partial, sys, rt.nseg);
  }
}

// --------------------------------------------------------------------------
// Fused 3D level kernels (constant coefficients), marching along z.  The 2D
// fused kernels stage a tile with a halo and run every sweep on it in LDS; in
// 3D a halo in z would cost about as much as the tile, so a workgroup owns an
// xy tile (with its halo) and walks up the planes with the stages lagging one
// plane behind each other.  At step t plane t enters; the first sweep (from
// x = 0 in the down kernel, the interpolated correction in the up kernel) is
// formed on it pointwise, and sweep m on plane t - m + 1 (down) or t - m (up).
// The newest plane of every stage goes into LDS for its in-plane neighbours;
// the planes above and below stay in registers.  A workgroup starts NU planes
// below its own (warm-up), so every plane it writes is exact; two barriers per
// plane.  Points off the grid (also planes below 0 and above n - 1) carry a
// zero right-hand side and a zero inverse diagonal, so they stay exactly 0,
// and the sweeps are branch-free as in the 2D kernels.
//
// k_down3: b (or, RUP, b_old - alpha (A + s) p formed on the fly, as in
// k_down2), NU sweeps from zero, the residual b - (A + s) x and its full
// weighting (the weights and order of k_restrict3); writes the pre-smoothed
// iterate on the owned fine planes and kD3Kz coarse planes of the coarse
// right-hand side.  One coarse column per thread.
// k_up3: x = x_in + P x_c (trilinear, as k_prolong3 along z), NU sweeps (the
// pre-smoothing weights reversed); writes the result on kU3Fz owned fine
// planes (and b.x when it is the finest level).
// --------------------------------------------------------------------------
constexpr int kD3Cx = 32, kD3Cy = 8, kD3Kz = 16;   // coarse columns and planes per workgroup (down)
constexpr int kU3Ox = 64, kU3Oy = 16, kU3Fz = 32;  // fine columns and planes per workgroup (up)
// 512 threads per workgroup: half the region points per thread of a
// 256-thread workgroup, so every sweep's planes fit in about 100 registers
// (FP32; 4 waves per SIMD instead of 2)
constexpr int kF3Threads = 512;
static_assert(kD3Cx * kD3Cy <= kF3Threads, "one coarse column per thread");

// (A + s) x at region point PAD + q from the in-plane values in LDS (row
// length RX) and the values below (xb) and above (xf): constant
// coefficients, the arithmetic and order of apply_col3
template <typename T>
__device__ __forceinline__ T lds_apply3(const T* X, int q, int RX, T xb, T xf, T w, T s) {
  const T xc = X[q];
  T sum = (xc - X[q - 1]) + (xc - X[q + 1]) + (xc - X[q - RX]) + (xc - X[q + RX]);
  sum += (xc - xb) + (xc - xf);
  return w * sum + s * xc;
}

// one damped Jacobi update at region point PAD + q (constant coefficients;
// xc = X[q], held in a register by the caller): x + w_m ((b + w times the
// six neighbours) r - x) with r the inverse diagonal (0 off the grid), equal
// to x + w_m (b - (A + s) x) r in exact arithmetic; 8 vector operations per
// point against 17
template <typename T>
__device__ __forceinline__ T lds_relax3(const T* X, int q, int RX, T xc, T xb, T xf, T w, T bb, T wm, T r) {
  T sum = (X[q - 1] + X[q + 1]) + (X[q - RX] + X[q + RX]);
  sum += xb + xf;
  return xc + wm * ((bb + w * sum) * r - xc);
}

template <typename T, int NU, bool RUP>
__global__ __launch_bounds__(kF3Threads) void k_down3(LevelDev<T> Lf, LevelDev<T> Lc, const T* __restrict__ b,
                                               T* __restrict__ xout, T* __restrict__ bc,
                                               const T* __restrict__ shift, const int* __restrict__ active,
                                               Sweeps<T> om, unsigned long long* __restrict__ ctr,
                                               const T* __restrict__ pv, const double* __restrict__ alpha,
                                               T* __restrict__ bout, double* __restrict__ partial, Fin fin) {
  constexpr int CX = kD3Cx, CY = kD3Cy;
  // the region: the owned fine columns with a halo of NU + 1; p (RUP) on
  // the region widened by one point, in a layout of its own
  constexpr int RX = 2 * CX + 2 * NU + 1, RY = 2 * CY + 2 * NU + 1, RN = RX * RY;
  constexpr int PX = RX + 2, PY = RY + 2, PN = PX * PY;
  constexpr int PER = (RN + kF3Threads - 1) / kF3Threads, PPER = RUP ? (PN + kF3Threads - 1) / kF3Threads : 1;
  constexpr int PAD = RX + 1, LX = PAD + PER * kF3Threads + RX + 1;
  constexpr int PADP = PX + 1, LP = RUP ? PADP + PPER * kF3Threads + PX + 1 : 1;
  __shared__ T sx[NU][LX];         // newest plane of each sweep's output
  __shared__ T sr[LX];             // residual plane
  __shared__ T sp[RUP ? 3 : 1][LP];   // p of planes z in slot z mod 3 (RUP): below, centre, above
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * (RUP ? 4 : 2) +
                                   (unsigned long long)Lc.N * sizeof(T));
  const int nf = Lf.n, nc = Lc.n;
  const int yt = (nc + CY - 1) / CY;
  const int kseg = tl.y / yt;
  const int I0 = tl.x * CX, J0 = (tl.y - kseg * yt) * CY;
  const int K0 = kseg * kD3Kz, K1 = min(K0 + kD3Kz, nc);
  const int fz1 = K1 == nc ? nf : 2 * K1;   // owned fine planes [2 K0, fz1) (the last segment: the top one too)
  const int gx0 = 2 * I0 - NU, gy0 = 2 * J0 - NU;
  const long long nn = (long long)nf * nf, off = (long long)sys * Lf.N;
  const T sh = shift[sys], w = Lf.wc;
  const T rcon = jacobi_recip(w * T(6) + sh);
  const T am = RUP ? (T)alpha[sys] : T(0);
  const int tid = threadIdx.x;
  // zero planes: the pads stay 0, the rest is written before a valid point reads it
  for (int i = tid; i < LX; i += kF3Threads) {
#pragma unroll
    for (int m = 0; m < NU; ++m) sx[m][i] = T(0);
    sr[i] = T(0);
  }
  if (RUP)
    for (int i = tid; i < LP; i += kF3Threads) sp[0][i] = sp[1][i] = sp[2][i] = T(0);
  __syncthreads();
  // region point u of this thread: on the grid in-plane (bit u of `in`),
  // owned (bit u of `own`), its in-plane offset clamped into the grid
  const int hx = (I0 + CX >= nc) ? nf : 2 * (I0 + CX);
  const int hy = (J0 + CY >= nc) ? nf : 2 * (J0 + CY);
  unsigned in = 0u, own = 0u;
  int col[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + kF3Threads * u;
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const bool on = q < RN && gi >= 0 && gi < nf && gj >= 0 && gj < nf;
    in |= (on ? 1u : 0u) << u;
    own |= ((on && gi >= 2 * I0 && gi < hx && gj >= 2 * J0 && gj < hy) ? 1u : 0u) << u;
    col[u] = min(max(gj, 0), nf - 1) * nf + min(max(gi, 0), nf - 1);
  }
  const T* __restrict__ bs = b + off;
  const T* __restrict__ ps = RUP ? pv + off : nullptr;
  // p-layout point u of this thread: on the grid (bit u of `pin`), its clamped in-plane offset
  unsigned pin = 0u;
  int pcol[PPER];
#pragma unroll
  for (int u = 0; u < PPER; ++u) {
    const int q = tid + kF3Threads * u;
    const int py = q / PX, px = q - py * PX;
    const int gi = gx0 - 1 + px, gj = gy0 - 1 + py;
    pin |= ((RUP && q < PN && gi >= 0 && gi < nf && gj >= 0 && gj < nf) ? 1u : 0u) << u;
    pcol[u] = min(max(gj, 0), nf - 1) * nf + min(max(gi, 0), nf - 1);
  }
  // a plane z of p at this thread's p-layout points (0 off the grid)
  auto load_p = [&](int z, T* dst) {
    const bool zin = z >= 0 && z < nf;
    const long long base = (long long)min(max(z, 0), nf - 1) * nn;
#pragma unroll
    for (int u = 0; u < PPER; ++u) {
      const T v = ps[base + pcol[u]];
      dst[u] = (zin && ((pin >> u) & 1u)) ? v : T(0);
    }
  };
  auto slot = [](int z) { return ((z % 3) + 3) % 3; };
  // planes t0 .. t1 enter: the first written residual (fine plane 2 K0)
  // depends on the first sweep down to plane 2 K0 - NU; the last is the
  // residual of fine plane 2 K1
  const int t0 = 2 * K0 - NU, t1 = 2 * K1 + NU;
  // registers: bh[d] = b of plane t - d; xh[m][0], xh[m][1] = sweep m+1's
  // output at its newest plane of the previous step and the one below
  T bh[NU + 1][PER], xh[NU][2][PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
#pragma unroll
    for (int d = 0; d <= NU; ++d) bh[d][u] = T(0);
#pragma unroll
    for (int m = 0; m < NU; ++m) xh[m][0][u] = xh[m][1][u] = T(0);
  }
  if (RUP) {
    for (int z = t0 - 1; z <= t0 + 1; ++z) {
      T pl[PPER];
      load_p(z, pl);
#pragma unroll
      for (int u = 0; u < PPER; ++u) sp[slot(z)][PADP + tid + kF3Threads * u] = pl[u];
    }
  }
  // the coarse column of this thread: its centre fine point in the region and
  // the weighted in-plane sums of the residual on fine planes 2K and 2K + 1
  const bool restricts = tid < CX * CY;   // whole waves
  const int ci = tid % CX, cj = restricts ? tid / CX : 0;
  const bool mine = restricts && I0 + ci < nc && J0 + cj < nc;
  const int rcq = PAD + (2 * cj + NU) * RX + (2 * ci + NU);   // fine (2I, 2J) of its 3 x 3 block
  T s_lo = T(0), s_mid = T(0);
  const long long ncc = (long long)nc * nc;
  T* __restrict__ bcs = bc + (long long)sys * Lc.N + ((long long)(J0 + cj) * nc + (I0 + ci));
  T* __restrict__ xs = xout + off;
  T* __restrict__ bo = RUP ? bout + off : nullptr;
  double rr = 0.0;
  ring_prologue_wait();
  __syncthreads();
  // the ring of plane loads (see kRowLead; kPlaneLead planes ahead): slot s
  // of step t holds b of plane t and p of plane t + 2 (RUP), as loaded
  // (clamped planes, unmasked)
  T rbv[kPlaneLead][PER], rpv[kPlaneLead][RUP ? PPER : 1];
  auto fill = [&](int t, int s) {
    const long long bb = (long long)min(max(t, 0), nf - 1) * nn;
#pragma unroll
    for (int u = 0; u < PER; ++u) rbv[s][u] = bs[bb + col[u]];
    if (RUP) {
      const long long pb = (long long)min(max(t + 2, 0), nf - 1) * nn;
#pragma unroll
      for (int u = 0; u < PPER; ++u) rpv[s][u] = ps[pb + pcol[u]];
    }
  };
#pragma unroll
  for (int s = 0; s < kPlaneLead; ++s) fill(t0 + s, s);
  ring_march<kPlaneLead>(t0, t1, [&](int t, auto sl) {
    constexpr int s = decltype(sl)::value;
    const long long base = (long long)min(max(t, 0), nf - 1) * nn;
    // in-grid mask of plane g for point u (0 off the grid, above and below it)
    auto on_at = [&](int g, int u) { return g >= 0 && g < nf && ((in >> u) & 1u); };
#pragma unroll
    for (int d = NU; d > 0; --d)
#pragma unroll
      for (int u = 0; u < PER; ++u) bh[d][u] = bh[d - 1][u];
    const bool wr_t = RUP && t >= 2 * K0 && t < fz1;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      T bn = rbv[s][u];
      if (RUP) {
        const int q = tid + kF3Threads * u;
        const int ry = q / RX, rx = q - ry * RX;
        const int pq = PADP + (ry + 1) * PX + (rx + 1);
        bn = bn - am * lds_apply3<T>(sp[slot(t)], pq, PX, sp[slot(t - 1)][pq], sp[slot(t + 1)][pq], w, sh);
      }
      bh[0][u] = on_at(t, u) ? bn : T(0);
      if (wr_t && ((own >> u) & 1u)) {
        __builtin_nontemporal_store(bh[0][u], &bo[base + col[u]]);
        rr += (double)bh[0][u] * (double)bh[0][u];
      }
    }
    // sweep 1 on plane t from x = 0; sweep m + 1 on plane t - m from sweep
    // m's output (centre plane in sx[m - 1], below in xh, above just formed)
    T xn[NU][PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) xn[0][u] = sweep_w(om, 0) * bh[0][u] * (on_at(t, u) ? rcon : T(0));
#pragma unroll
    for (int m = 1; m < NU; ++m) {
      const T wm = sweep_w(om, m);
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int q = PAD + tid + kF3Threads * u;
        xn[m][u] = lds_relax3<T>(sx[m - 1], q, RX, xh[m - 1][0][u], xh[m - 1][1][u], xn[m - 1][u], w, bh[m][u], wm,
                                 on_at(t - m, u) ? rcon : T(0));
      }
    }
    // the residual on plane t - NU
    T res[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = PAD + tid + kF3Threads * u;
      res[u] = bh[NU][u] - lds_apply3<T>(sx[NU - 1], q, RX, xh[NU - 1][1][u], xn[NU - 1][u], w, sh);
    }
    // the pre-smoothed iterate: sweep NU's newest plane t - NU + 1
    const int gx = t - NU + 1;
    if (gx >= 2 * K0 && gx < fz1) {
      const long long bx = (long long)gx * nn;
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if ((own >> u) & 1u) __builtin_nontemporal_store(xn[NU - 1][u], &xs[bx + col[u]]);
    }
    __syncthreads();   // every read of this step's LDS planes is done
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = PAD + tid + kF3Threads * u;
#pragma unroll
      for (int m = 0; m < NU; ++m) sx[m][q] = xn[m][u];
      sr[q] = res[u];
    }
    if (RUP) {   // p(t + 2) takes the slot of p(t - 1) (0 off the grid)
      const bool zin = t + 2 >= 0 && t + 2 < nf;
#pragma unroll
      for (int u = 0; u < PPER; ++u)
        sp[slot(t + 2)][PADP + tid + kF3Threads * u] = (zin && ((pin >> u) & 1u)) ? rpv[s][u] : T(0);
    }
    __syncthreads();
    fill(t + kPlaneLead, s);   // refill the slot with the planes kPlaneLead steps ahead
    // full weighting: this coarse column's in-plane sum of fine plane f = t - NU,
    // and coarse plane K = f/2 - 1 once f = 2K + 2 (weights 1/4, 1/2, 1/4 along z)
    const int f = t - NU;
    if (restricts && f >= 2 * K0) {
      const T wt[3] = {T(0.25), T(0.5), T(0.25)};
      T acc = T(0);
#pragma unroll
      for (int q = 0; q < 9; ++q) {
        const int di = q % 3, dj = q / 3;
        acc += wt[dj] * wt[di] * sr[rcq + dj * RX + di];
      }
      const bool odd = f & 1;
      if (!odd && f != 2 * K0) {
        const int K = f / 2 - 1;
        if (mine) bcs[K * ncc] = T(0.25) * s_lo + T(0.5) * s_mid + T(0.25) * acc;
      }
      // selects, not stores in two branches (see k_down2r)
      s_mid = odd ? acc : s_mid;
      s_lo = odd ? s_lo : acc;
    }
    // shift the registers one plane up
#pragma unroll
    for (int u = 0; u < PER; ++u) {
#pragma unroll
      for (int m = 0; m < NU; ++m) {
        xh[m][1][u] = xh[m][0][u];
        xh[m][0][u] = xn[m][u];
      }
    }
  });
  if (RUP) {
    write_partial_tile(tl, partial, sys, rr);
    finish(fin, partial, sys, gridDim.x * gridDim.y);
  }
}

template <typename T, int NU, bool DOT>
__global__ __launch_bounds__(kF3Threads) void k_up3(LevelDev<T> Lc, LevelDev<T> Lf, const T* __restrict__ xc,
                                             const T* __restrict__ xin, const T* __restrict__ b, T* __restrict__ xout,
                                             const T* __restrict__ shift, const int* __restrict__ active, Sweeps<T> om,
                                             double* __restrict__ partial, unsigned long long* __restrict__ ctr,
                                             Fin fin) {
  constexpr int OX = kU3Ox, OY = kU3Oy;
  constexpr int RX = OX + 2 * NU, RY = OY + 2 * NU, RN = RX * RY;
  constexpr int PER = (RN + kF3Threads - 1) / kF3Threads;
  constexpr int PAD = RX + 1, LX = PAD + PER * kF3Threads + RX + 1;
  // the coarse columns under the region, zero-padded: coarse index c at cx0 + (c - c0)
  constexpr int CRX = RX / 2 + 3, CRY = RY / 2 + 3, CRN = CRX * CRY;
  constexpr int CPER = (CRN + kF3Threads - 1) / kF3Threads;
  __shared__ T sx[NU][LX];   // newest plane of the correction and of sweeps 1 .. NU-1
  __shared__ T sc[CRN];      // one coarse plane under the region
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)Lf.N * sizeof(T) * 3 + (unsigned long long)Lc.N * sizeof(T));
  const int nf = Lf.n, nc = Lc.n;
  const int yt = (nf + OY - 1) / OY;
  const int zseg = tl.y / yt;
  const int ox0 = tl.x * OX, oy0 = (tl.y - zseg * yt) * OY;
  const int z0 = zseg * kU3Fz, z1 = min(z0 + kU3Fz, nf);
  const int gx0 = ox0 - NU, gy0 = oy0 - NU;
  const int cx0 = ((gx0 >= 0) ? gx0 / 2 : -((-gx0 + 1) / 2)) - 1;
  const int cy0 = ((gy0 >= 0) ? gy0 / 2 : -((-gy0 + 1) / 2)) - 1;
  const long long nn = (long long)nf * nf, off = (long long)sys * Lf.N, ncc = (long long)nc * nc;
  const T sh = shift[sys], w = Lf.wc;
  const T rcon = jacobi_recip(w * T(6) + sh);
  const int tid = threadIdx.x;
  // zero planes: the pads stay 0, the rest is written before a valid point reads it
  for (int i = tid; i < LX; i += kF3Threads) {
#pragma unroll
    for (int m = 0; m < NU; ++m) sx[m][i] = T(0);
  }
  unsigned in = 0u, own = 0u;
  int col[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int q = tid + kF3Threads * u;
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const bool on = q < RN && gi >= 0 && gi < nf && gj >= 0 && gj < nf;
    in |= (on ? 1u : 0u) << u;
    own |= ((on && rx >= NU && rx < NU + OX && ry >= NU && ry < NU + OY) ? 1u : 0u) << u;
    col[u] = min(max(gj, 0), nf - 1) * nf + min(max(gi, 0), nf - 1);
  }
  const T* __restrict__ xcs = xc + (long long)sys * Lc.N;
  const T* __restrict__ bs = b + off;
  const T* __restrict__ xis = xin + off;
  // coarse plane K under the region into sc (0 off the grid)
  auto stage = [&](int K) {
    const long long cb = (long long)min(max(K, 0), nc - 1) * ncc;
    T cl[CPER];
#pragma unroll
    for (int u = 0; u < CPER; ++u) {
      const int q = tid + kF3Threads * u;
      const int cy = q / CRX, cx = q - cy * CRX;
      cl[u] = xcs[cb + (long long)min(max(cy0 + cy, 0), nc - 1) * nc + min(max(cx0 + cx, 0), nc - 1)];
    }
#pragma unroll
    for (int u = 0; u < CPER; ++u) {
      const int q = tid + kF3Threads * u;
      if (q < CRN) {
        const int cy = q / CRX, cx = q - cy * CRX;
        const int I = cx0 + cx, J = cy0 + cy;
        sc[q] = (K >= 0 && K < nc && I >= 0 && I < nc && J >= 0 && J < nc) ? cl[u] : T(0);
      }
    }
  };
  // the in-plane interpolant of the staged coarse plane at region point u
  // (lanes past the region interpolate at its last point, in range of sc)
  auto interp = [&](int u) -> T {
    const int q = min(tid + kF3Threads * u, RN - 1);
    const int ry = q / RX, rx = q - ry * RX;
    const int gi = gx0 + rx, gj = gy0 + ry;
    const int ia = (gi & 1) ? (gi - 1) / 2 : gi / 2 - 1;
    const int ja = (gj & 1) ? (gj - 1) / 2 : gj / 2 - 1;
    const T* C = sc + (ja - cy0) * CRX + (ia - cx0);
    if (gi & 1) return (gj & 1) ? C[0] : T(0.5) * (C[0] + C[CRX]);
    return (gj & 1) ? T(0.5) * (C[0] + C[1]) : T(0.25) * (C[0] + C[1] + C[CRX] + C[CRX + 1]);
  };
  // lowest coarse plane of fine plane t (odd t lies on it, even t halfway to the next)
  auto klo = [](int t) { return (t >> 1) - 1 + (t & 1); };
  // planes t0 .. t1 enter: the owned plane z0 needs the correction down to z0 - NU
  const int t0 = z0 - NU, t1 = z1 + NU - 1;
  // vlo, vhi: the in-plane interpolants of coarse planes Kc and Kc + 1
  int Kc = klo(t0);
  T vlo[PER], vhi[PER];
  stage(Kc);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) vlo[u] = interp(u);
  __syncthreads();
  stage(Kc + 1);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) vhi[u] = interp(u);
  // registers: bh[d] = b of plane t - d; xh[m][0], xh[m][1] = stage m's
  // output (m = 0: the corrected x) at its newest plane of the previous step and
  // the one below
  T bh[NU + 1][PER], xh[NU][2][PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
#pragma unroll
    for (int d = 0; d <= NU; ++d) bh[d][u] = T(0);
#pragma unroll
    for (int m = 0; m < NU; ++m) xh[m][0][u] = xh[m][1][u] = T(0);
  }
  T* __restrict__ xs = xout + off;
  double dot = 0.0;
  ring_prologue_wait();
  __syncthreads();
  // the ring of plane loads (see kRowLead; kPlaneLead planes ahead): slot s
  // of step t holds x_in and b of plane t and the coarse plane klo(t + 1) + 1
  // under the region (staged at step t when klo(t + 1) > klo(t)), as loaded
  // (clamped, unmasked)
  T rxv[kPlaneLead][PER], rbv[kPlaneLead][PER], rcv[kPlaneLead][CPER];
  auto fill = [&](int t, int s) {
    const long long bb = (long long)min(max(t, 0), nf - 1) * nn;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      rxv[s][u] = xis[bb + col[u]];
      rbv[s][u] = bs[bb + col[u]];
    }
    const long long cb = (long long)min(max(klo(t + 1) + 1, 0), nc - 1) * ncc;
#pragma unroll
    for (int u = 0; u < CPER; ++u) {
      const int q = tid + kF3Threads * u;
      const int cy = q / CRX, cx = q - cy * CRX;
      rcv[s][u] = xcs[cb + (long long)min(max(cy0 + cy, 0), nc - 1) * nc + min(max(cx0 + cx, 0), nc - 1)];
    }
  };
#pragma unroll
  for (int s = 0; s < kPlaneLead; ++s) fill(t0 + s, s);
  ring_march<kPlaneLead>(t0, t1, [&](int t, auto sl) {
    constexpr int s = decltype(sl)::value;
    auto on_at = [&](int g, int u) { return g >= 0 && g < nf && ((in >> u) & 1u); };
    if (klo(t) > Kc) {   // sc holds coarse plane Kc + 2 (staged in the previous step)
      ++Kc;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        vlo[u] = vhi[u];
        vhi[u] = interp(u);
      }
    }
#pragma unroll
    for (int d = NU; d > 0; --d)
#pragma unroll
      for (int u = 0; u < PER; ++u) bh[d][u] = bh[d - 1][u];
    // stage 0 on plane t: x_in + P x_c; stage m on plane t - m
    T xn[NU + 1][PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const bool on = on_at(t, u);
      bh[0][u] = on ? rbv[s][u] : T(0);
      const T v = (t & 1) ? vlo[u] : T(0.5) * (vlo[u] + vhi[u]);
      xn[0][u] = on ? rxv[s][u] + v : T(0);
    }
#pragma unroll
    for (int m = 1; m <= NU; ++m) {
      const T wm = sweep_w(om, NU - m);
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int q = PAD + tid + kF3Threads * u;
        xn[m][u] = lds_relax3<T>(sx[m - 1], q, RX, xh[m - 1][0][u], xh[m - 1][1][u], xn[m - 1][u], w, bh[m][u], wm,
                                 on_at(t - m, u) ? rcon : T(0));
      }
    }
    const int g = t - NU;
    if (g >= z0 && g < z1) {
      const long long bx = (long long)g * nn;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const bool o = (own >> u) & 1u;
        if (o) __builtin_nontemporal_store(xn[NU][u], &xs[bx + col[u]]);
        if (DOT) dot += o ? (double)bh[NU][u] * (double)xn[NU][u] : 0.0;
      }
    }
    __syncthreads();   // every read of this step's LDS planes is done
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int q = PAD + tid + kF3Threads * u;
#pragma unroll
      for (int m = 0; m < NU; ++m) sx[m][q] = xn[m][u];
    }
    if (klo(t + 1) > Kc) {   // coarse plane Kc + 2 into sc (0 off the grid)
      const int K = Kc + 2;
#pragma unroll
      for (int u = 0; u < CPER; ++u) {
        const int q = tid + kF3Threads * u;
        if (q < CRN) {
          const int cy = q / CRX, cx = q - cy * CRX;
          const int I = cx0 + cx, J = cy0 + cy;
          sc[q] = (K >= 0 && K < nc && I >= 0 && I < nc && J >= 0 && J < nc) ? rcv[s][u] : T(0);
        }
      }
    }
    __syncthreads();
    fill(t + kPlaneLead, s);   // refill the slot with the planes kPlaneLead steps ahead
#pragma unroll
    for (int u = 0; u < PER; ++u)
#pragma unroll
      for (int m = 0; m < NU; ++m) {
        xh[m][1][u] = xh[m][0][u];
        xh[m][0][u] = xn[m][u];
      }
  });
  if (DOT) {
    write_partial_tile(tl, partial, sys, dot);
    finish(fin, partial, sys, gridDim.x * gridDim.y);
  }
}

// --------------------------------------------------------------------------
// PCG pieces
// --------------------------------------------------------------------------
// p_new = z + beta p_old and q = (A+s) p_new in one pass (p_new formed at the
// stencil points on the fly); p_old and p_new are different buffers.
// XUP: also x += alpha_prev p_old, the iterate update of the previous PCG
// iteration, deferred to this pass which reads p_old anyway.  alpha == 0 marks
// "nothing pending" (first iteration); p_old is then not used.
//
// 3D version, marching along z with kMarchRows rows per thread: p_new =
// z + beta p_old is formed once per point; the rows' values below and at the
// point stay in registers.
template <typename T, bool VAR, bool XUP, bool WQ>
__global__ __launch_bounds__(kBlock) void k_spmv_p3(LevelDev<T> L, const T* __restrict__ z, const T* __restrict__ pold,
                                                    T* __restrict__ pnew, T* __restrict__ q,
                                                    const double* __restrict__ beta, const T* __restrict__ shift,
                                                    const int* __restrict__ active, double* __restrict__ partial,
                                                    unsigned long long* __restrict__ ctr, Fin fin,
                                                    T* __restrict__ x, const double* __restrict__ alpha) {
  constexpr int R = kMarchRows;
  const Tile tl = VAR && sizeof(T) == 4 ? block_tile_shared() : block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  const T bt = (T)beta[sys];
  const T ap = XUP ? (T)alpha[sys] : T(0);
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) *
                                ((bt == T(0) ? 3 : 4) - (WQ ? 0 : 1) + (XUP && ap != T(0) ? 2 : 0) +
                                 (VAR && sys == 0 ? 3 : 0)));
  const int n = L.n;
  const Column c = march_column(tl, n, R);
  double dot = 0.0;
  if (c.i < n && c.j < n) {
    const long long off = (long long)sys * L.N, nn = (long long)n * n;
    const Rows<R> w(c.i, c.j, n);
    const T* zs = z + off;
    // beta = 0 (first iteration): p_old may hold anything, so read z in its place
    const T* pe = bt == T(0) ? zs : pold + off;
    const T s = shift[sys];
    T below[R], centre[R], pold_c[R];   // pold_c: p_old at the point (alpha != 0 => beta != 0)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const long long p0 = c.k0 * nn + w.col[r];
      const long long pb = c.k0 > 0 ? p0 - nn : p0;
      const T zb = zs[pb], eb = pe[pb], zc = zs[p0], ec = pe[p0];
      below[r] = c.k0 > 0 ? zb + bt * eb : T(0);
      centre[r] = zc + bt * ec;
      pold_c[r] = ec;
    }
    ColFaces<T, VAR, R> fw;
    fw.start(L, w, c.k0);
    for (int k = c.k0; k < c.k1; ++k) {
      const long long pk = k * nn;
      // every load of the plane first, then the arithmetic
      T za[R], ea[R], zl[R], el[R], zr[R], er[R], xv[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const long long p = pk + w.col[r];
        const long long pa = k + 1 < n ? p + nn : p;
        za[r] = zs[pa];
        ea[r] = pe[pa];
        zl[r] = zs[p + w.il];
        el[r] = pe[p + w.il];
        zr[r] = zs[p + w.ir];
        er[r] = pe[p + w.ir];
        xv[r] = XUP ? x[off + p] : T(0);
      }
      const T zd = zs[pk + w.col_d], ed = pe[pk + w.col_d], zu = zs[pk + w.col_u], eu = pe[pk + w.col_u];
      fw.load(L, w, c.i, c.j, k);
      const T hd = zd + bt * ed, hu = zu + bt * eu;
      T above[R];
#pragma unroll
      for (int r = 0; r < R; ++r) above[r] = k + 1 < n ? za[r] + bt * ea[r] : T(0);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!w.valid[r]) continue;
        const long long p = pk + w.col[r];
        const T lv = w.il ? zl[r] + bt * el[r] : T(0), rv = w.ir ? zr[r] + bt * er[r] : T(0);
        fw.row(L, w, c.i, c.j, k, r);
        const T qv = apply_col3(L, fw, r, centre[r], lv, rv, w.down(r, centre, hd), w.up(r, centre, hu),
                                           below[r], above[r], s);
        pnew[off + p] = centre[r];
        if (WQ) q[off + p] = qv;
        if (XUP && ap != T(0)) x[off + p] = xv[r] + ap * pold_c[r];
        dot += (double)centre[r] * (double)qv;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        below[r] = centre[r];
        centre[r] = above[r];
        pold_c[r] = ea[r];
      }
    }
  }
  write_partial_tile(tl, partial, sys, dot);
  finish(fin, partial, sys, gridDim.x * gridDim.y);
}

// 2D version: each thread owns R consecutive rows of one column (a workgroup
// of TX x (256 / TX) threads covers TX x (256 / TX) R points), so the column's p_new values are formed
// once and reused by the rows above and below; only the left/right neighbours
// are extra loads.
template <typename T, bool VAR, bool XUP, bool WQ, int R, int TX>
__global__ __launch_bounds__(kBlock) void k_spmv_p2(LevelDev<T> L, const T* __restrict__ z, const T* __restrict__ pold,
                                                    T* __restrict__ pnew, T* __restrict__ q,
                                                    const double* __restrict__ beta, const T* __restrict__ shift,
                                                    const int* __restrict__ active, double* __restrict__ partial,
                                                    unsigned long long* __restrict__ ctr, Fin fin,
                                                    T* __restrict__ x, const double* __restrict__ alpha) {
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active[sys]) return;
  const T bt = (T)beta[sys];
  const T ap = XUP ? (T)alpha[sys] : T(0);
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * sizeof(T) *
                                ((bt == T(0) ? 3 : 4) - (WQ ? 0 : 1) + (XUP && ap != T(0) ? 2 : 0) +
                                 (VAR && sys == 0 ? 2 : 0)));
  const int n = L.n;
  const int i = tl.x * TX + threadIdx.x;
  const int j0 = (tl.y * (kBlock / TX) + threadIdx.y) * R;
  const long long off = (long long)sys * L.N;
  double dot = 0.0;
  if (i < n && j0 < n) {
    const T* zs = z + off;
    // beta = 0 (first iteration): p_old may hold anything, so read z in its place
    const T* pe = bt == T(0) ? zs : pold + off;
    const T s = shift[sys];
    const int il = i > 0 ? i - 1 : i, ir = i < n - 1 ? i + 1 : i;
    // every load first (clamped rows/columns), then the arithmetic
    T zc[R + 2], pc[R + 2], zl[R], pl[R], zr[R], pr[R], xv[R];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
      const int jj = min(max(j0 - 1 + r, 0), n - 1);
      const long long g = (long long)jj * n + i;
      zc[r] = zs[g];
      pc[r] = pe[g];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const long long row = (long long)min(j0 + r, n - 1) * n;
      zl[r] = zs[row + il];
      pl[r] = pe[row + il];
      zr[r] = zs[row + ir];
      pr[r] = pe[row + ir];
      if (XUP) xv[r] = x[off + row + i];
    }
    T v[R + 2];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
      const int jj = j0 - 1 + r;
      v[r] = (jj >= 0 && jj < n) ? zc[r] + bt * pc[r] : T(0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = j0 + r;
      if (j < n) {
        const T c = v[r + 1], dn = v[r], up = v[r + 2];
        const T lv = i > 0 ? zl[r] + bt * pl[r] : T(0);
        const T rv = i < n - 1 ? zr[r] + bt * pr[r] : T(0);
        T qv;
        if (!VAR) {
          qv = L.wc * ((c - lv) + (c - rv) + (c - dn) + (c - up)) + s * c;
        } else {
          const long long fx = (long long)j * (n + 1) + i;
          const long long fy = (long long)j * n + i;
          qv = L.wf0[fx] * (c - lv) + L.wf0[fx + 1] * (c - rv) + L.wf1[fy] * (c - dn) + L.wf1[fy + n] * (c - up) +
               s * c;
        }
        const long long g = off + (long long)j * n + i;
        __builtin_nontemporal_store(c, &pnew[g]);
        if (WQ) __builtin_nontemporal_store(qv, &q[g]);
        // the deferred update uses p_old = pc (pe is p_old whenever alpha != 0)
        if (XUP && ap != T(0)) __builtin_nontemporal_store(xv[r] + ap * pc[r + 1], &x[g]);
        dot += (double)c * (double)qv;
      }
    }
  }
  write_partial_tile(tl, partial, sys, dot);
  finish(fin, partial, sys, gridDim.x * gridDim.y);
}

// Row-marching version of k_spmv_p2 (launch-shape variant 3), two columns per
// thread: a workgroup walks `rows` rows (a launch parameter); p_new of the rows
// below, at and above the current one stays in registers and the current row's
// p_new is in LDS for the left/right neighbours, so z and p_old are read once
// per point (plus one row above and below a segment).  Same values per point
// as k_spmv_p2.
template <typename T, bool VAR, bool XUP, bool WQ>
__global__ __launch_bounds__(kRowThreads) void k_spmv_r2(LevelDev<T> L, const T* __restrict__ z, const T* __restrict__ pold,
                                                  T* __restrict__ pnew, T* __restrict__ q,
                                                  const double* __restrict__ beta, const T* __restrict__ shift,
                                                  const int* __restrict__ active, double* __restrict__ partial,
                                                  unsigned long long* __restrict__ ctr, Fin fin,
                                                  T* __restrict__ x, const double* __restrict__ alpha, int rows) {
  constexpr int WORDS = spmv_words(), REC = row_rec(WORDS);   // LDS: p_new's pair
  // (without face weights FP64 has registers for four rows of lead too: 255^2,
  // 512 systems 185 -> 175 us)
  constexpr int LEAD = VAR ? row_lead<T>() : 4;
  const RowTile rt = row_tile();
  const int sys = rt.sys;
  if (!active[sys]) return;
  const T bt = (T)beta[sys];
  const T ap = XUP ? (T)alpha[sys] : T(0);
  count_bytes_row(rt, ctr, (unsigned long long)L.N * sizeof(T) *
                                ((bt == T(0) ? 3 : 4) - (WQ ? 0 : 1) + (XUP && ap != T(0) ? 2 : 0) +
                                 (VAR && sys == 0 ? 2 : 0)));
  const int n = L.n;
  const int i = threadIdx.x, NT = blockDim.x;
  const int j0 = rt.seg * rows, j1 = min(j0 + rows, n);
  const long long off = (long long)sys * L.N;
  const T* __restrict__ zs = z + off;
  // beta = 0 (first iteration): p_old may hold anything, so read z in its place
  const T* __restrict__ pe = bt == T(0) ? zs : pold + off;
  const RowPair<T, VAR> pr(L, zs);
  const RowBuf<T> zsb(zs, L.N), peb(pe, L.N), xb(XUP ? x + off : zs, L.N), pnb(pnew + off, L.N), qb(WQ ? q + off : pnew + off, L.N);
  typedef typename RowPair<T, VAR>::Faces Faces;
  const T s_ = shift[sys];
  T* lds = reinterpret_cast<T*>(row_lds);
  for (int j = i; j < (NT + 2) * REC; j += NT) lds[j] = T(0);
  T* rec = lds + (i + 1) * REC;
  __syncthreads();
  // p_new of a row off the grid is 0: a factor rather than a select (a select
  // lets the compiler move a load into a branch and wait there for every load
  // in flight)
  auto p_new = [&](const T (&zv)[2], const T (&ev)[2], int r, T (&v)[2]) {
    const T m = pr.in(r) ? T(1) : T(0);
    v[0] = (zv[0] + bt * ev[0]) * m;
    v[1] = (zv[1] + bt * ev[1]) * (m * pr.m1);
  };
  // p_new below and at row j0 (dn, c), p_old at row j0 (pc), the faces below it
  T dn[2], c[2], pc[2], fd[2] = {T(0), T(0)};
  {
    T zb[2], eb[2], zc[2];
    zsb.ld2(zb, pr.cb, pr.row(j0 - 1));
    peb.ld2(eb, pr.cb, pr.row(j0 - 1));
    zsb.ld2(zc, pr.cb, pr.row(j0));
    peb.ld2(pc, pr.cb, pr.row(j0));
    pr.above(fd, j0 - 1);
    p_new(zb, eb, j0 - 1, dn);
    p_new(zc, pc, j0, c);
  }
  rec[WORDS] = c[0];   // the half that the first step reads
  rec[WORDS + 1] = c[1];
  double dot = 0.0;
  ring_prologue_wait();
  __syncthreads();
  auto walk = [&](auto upd_c) {
    constexpr bool UPD = XUP && decltype(upd_c)::value;
    // the ring of row loads (see kRowLead): slot s of step j holds z and
    // p_old of row j + 1 and x and the faces of row j, as loaded (clamped
    // rows, unmasked)
    T rz[LEAD][2], re[LEAD][2], rx[LEAD][2];
    Faces rf[LEAD];
    auto fill = [&](int j, int s) {
      const unsigned ra = pr.row(j + 1);
      zsb.ld2(rz[s], pr.cb, ra);
      peb.ld2(re[s], pr.cb, ra);
      if (UPD) xb.ld2(rx[s], pr.cb, pr.row(j));
      pr.faces(rf[s], j);
    };
#pragma unroll
    for (int s = 0; s < LEAD; ++s) fill(j0 + s, s);
    ring_march<LEAD>(j0, j1 - 1, [&](int j, auto slot) {
      constexpr int s = decltype(slot)::value;
      constexpr int WR = (s & 1) * WORDS, RD = WORDS - WR;
      T up[2], qv[2];
      p_new(rz[s], re[s], j + 1, up);
      pair_apply<T, VAR>(qv, rf[s], fd, c, rec[RD + 1 - REC], rec[RD + REC], dn, up, L.wc, s_);
      pr.template store<WQ>(pnb, c, j);
      if (WQ) pr.template store<WQ>(qb, qv, j);
      // the deferred update uses p_old = pc (pe is p_old whenever alpha != 0)
      if (UPD) {
        const T xv[2] = {rx[s][0] + ap * pc[0], rx[s][1] + ap * pc[1]};
        pr.template store<WQ>(xb, xv, j);
      }
      // (off the grid c is 0)
      dot += (double)c[0] * (double)qv[0];
      dot += (double)c[1] * (double)qv[1];
      rec[WR] = up[0];
      rec[WR + 1] = up[1];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        pc[e] = ring_take(re[s][e]);   // p_old of row j + 1, the next step's pc
        if (VAR) fd[e] = ring_take(rf[s].u[e]);
        dn[e] = c[e];
        c[e] = up[e];
      }
      __syncthreads();
      fill(j + LEAD, s);
    });
  };
  if (XUP && ap != T(0)) walk(std::true_type{});
  else walk(std::false_type{});
  write_partial(partial, sys, dot, rt.seg, rt.nseg);
  finish(fin, partial, sys, rt.nseg);
}

// --------------------------------------------------------------------------
constexpr int kFlatItems = 4;

template <typename T>
__global__ __launch_bounds__(256) void k_update_xr(long long N, T* __restrict__ x, T* __restrict__ r,
                                                   const T* __restrict__ pv, const T* __restrict__ q,
                                                   const double* __restrict__ alpha, const int* __restrict__ active,
                                                   double* __restrict__ partial, unsigned long long* __restrict__ ctr,
                                                   Fin fin) {
  const int sys = blockIdx.y;
  if (!active[sys]) return;
  count_bytes<COUNT_FLAT>(ctr, (unsigned long long)N * sizeof(T) * 6);
  const T a = (T)alpha[sys];
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
  double rr = 0.0;
  // all loads first (clamped index), then the updates and stores
  T xv[kFlatItems], pl[kFlatItems], rl[kFlatItems], ql[kFlatItems];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = min(base + (long long)it * 256, N - 1);
    xv[it] = x[off + p];
    pl[it] = pv[off + p];
    rl[it] = r[off + p];
    ql[it] = q[off + p];
  }
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = base + (long long)it * 256;
    if (p < N) {
      x[off + p] = xv[it] + a * pl[it];
      const T rv = rl[it] - a * ql[it];
      r[off + p] = rv;
      rr += (double)rv * (double)rv;
    }
  }
  write_partial_flat(partial, sys, rr);
  finish(fin, partial, sys, gridDim.x);
}

// The deferred update of the last PCG iteration: x += alpha p_last, with
// p_last in pa when the system's iteration count is even and in pb otherwise
// (iteration c reads p_old from pa for even c and writes p_new to the other).
template <typename T>
__global__ __launch_bounds__(256) void k_finish_x(long long N, T* __restrict__ x, const T* __restrict__ pa,
                                                  const T* __restrict__ pb, const double* __restrict__ alpha,
                                                  const int* __restrict__ iters, unsigned long long* __restrict__ ctr) {
  const int sys = blockIdx.y;
  const int it = iters[sys];
  const T a = (T)alpha[sys];
  if (it <= 0 || a == T(0)) return;
  count_bytes<COUNT_FLAT>(ctr, (unsigned long long)N * sizeof(T) * 3);
  const T* pl = ((it - 1) & 1) ? pa : pb;
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
  T xv[kFlatItems], pv[kFlatItems];
#pragma unroll
  for (int k = 0; k < kFlatItems; ++k) {
    const long long p = min(base + (long long)k * 256, N - 1);
    xv[k] = x[off + p];
    pv[k] = pl[off + p];
  }
#pragma unroll
  for (int k = 0; k < kFlatItems; ++k) {
    const long long p = base + (long long)k * 256;
    if (p < N) x[off + p] = xv[k] + a * pv[k];
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_update_p(long long N, T* __restrict__ pv, const T* __restrict__ z,
                                                  const double* __restrict__ beta, const int* __restrict__ active,
                                                  unsigned long long* __restrict__ ctr) {
  const int sys = blockIdx.y;
  if (!active[sys]) return;
  const T bt = (T)beta[sys];
  count_bytes<COUNT_FLAT>(ctr, (unsigned long long)N * sizeof(T) * (bt == T(0) ? 2 : 3));
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = base + (long long)it * 256;
    if (p < N) pv[off + p] = bt == T(0) ? z[off + p] : z[off + p] + bt * pv[off + p];
  }
}

// r = (T) f[rhs of system], x = 0, partial = ||r||^2 (FP64 from the FP64 input).
template <typename T>
__global__ __launch_bounds__(256) void k_copy_rhs(long long N, const double* __restrict__ f, T* __restrict__ r,
                                                  T* __restrict__ x, int nrhs,
                                                  const int* __restrict__ active, double* __restrict__ partial) {
  const int sys = blockIdx.y;
  if (!active[sys]) return;
  const int rhs = sys % nrhs;
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
  double ff = 0.0;
  double fl[kFlatItems];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) fl[it] = f[(long long)rhs * N + min(base + (long long)it * 256, N - 1)];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = base + (long long)it * 256;
    if (p < N) {
      const double fv = fl[it];
      r[off + p] = (T)fv;
      x[off + p] = T(0);
      ff += fv * fv;
    }
  }
  write_partial_flat(partial, sys, ff);
}

// --------------------------------------------------------------------------
// FP64 refinement residual: r32 = f - (A + s) x64, e = 0, partial = ||r||^2
// --------------------------------------------------------------------------
// k_residual64 in 2D with the stencil product's layout: R rows per thread over
// TX columns, the column's values of the rows above and below from the
// thread's own registers, every load issued before the arithmetic (a
// one-point-per-thread launch reads each x value from the caches five times)
constexpr int kRes2Rows = 4, kRes2Cols = 128;
// RT: float for the refinement (r32, and e = 0), double for the residual of an
// FP64 plan's starting iterate (e not written)
template <bool VAR, typename RT = float>
__global__ __launch_bounds__(kBlock) void k_residual64_2(LevelDev<double> L, const double* __restrict__ f,
                                                         const double* __restrict__ x64, float* __restrict__ e,
                                                         RT* __restrict__ r32, const double* __restrict__ shift,
                                                         const int* __restrict__ active64, int nrhs,
                                                         double* __restrict__ partial,
                                                         unsigned long long* __restrict__ ctr) {
  constexpr int R = kRes2Rows, TX = kRes2Cols;
  const Tile tl = block_tile();
  const int sys = tl.z;
  if (!active64[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * (8 + 8 + 4 + 4 + (VAR && sys == 0 ? 16 : 0)));
  const int n = L.n;
  const int i = tl.x * TX + threadIdx.x;
  const int j0 = (tl.y * (kBlock / TX) + threadIdx.y) * R;
  double rr = 0.0;
  if (i < n && j0 < n) {
    const long long off = (long long)sys * L.N;
    const double* __restrict__ xs = x64 + off;
    const double* __restrict__ fs = f + (long long)(sys % nrhs) * L.N;
    const double s = shift[sys];
    const int il = i > 0 ? i - 1 : i, ir = i < n - 1 ? i + 1 : i;
    double xc[R + 2], xl[R], xr[R], fv[R];
    double wl[VAR ? R : 1], wr[VAR ? R : 1], wd[VAR ? R : 1], wu[VAR ? R : 1];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) xc[r] = xs[min(max(j0 - 1 + r, 0), n - 1) * n + i];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int row = min(j0 + r, n - 1) * n;
      xl[r] = xs[row + il];
      xr[r] = xs[row + ir];
      fv[r] = fs[row + i];
      if (VAR) {
        const int jr = min(j0 + r, n - 1);
        const int fx = jr * (n + 1) + i, fy = jr * n + i;
        wl[VAR ? r : 0] = L.wf0[fx];
        wr[VAR ? r : 0] = L.wf0[fx + 1];
        wd[VAR ? r : 0] = L.wf1[fy];
        wu[VAR ? r : 0] = L.wf1[fy + n];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = j0 + r;
      if (j < n) {
        const double c = xc[r + 1];
        const double dn = j > 0 ? xc[r] : 0.0, up = j < n - 1 ? xc[r + 2] : 0.0;
        const double lv = i > 0 ? xl[r] : 0.0, rv = i < n - 1 ? xr[r] : 0.0;
        double ax;
        if (!VAR) {
          ax = L.wc * ((c - lv) + (c - rv) + (c - dn) + (c - up)) + s * c;
        } else {
          ax = wl[VAR ? r : 0] * (c - lv) + wr[VAR ? r : 0] * (c - rv) + wd[VAR ? r : 0] * (c - dn) +
               wu[VAR ? r : 0] * (c - up) + s * c;
        }
        const double rv64 = fv[r] - ax;
        const long long g = off + (long long)j * n + i;
        r32[g] = (RT)rv64;
        if constexpr (sizeof(RT) == 4) e[g] = 0.0f;
        rr += rv64 * rv64;
      }
    }
  }
  write_partial_tile(tl, partial, sys, rr);
}

// Row-marching version of k_residual64_2 for wide launches: one thread per
// grid column, a workgroup walks kRes2rRows rows of one system with x64 of
// the rows below, at and above in registers and the current row in LDS, so
// x64 is read once per point (the 128 x 8 tiles read 1.25 - 1.5 times; 511^2,
// 2048 systems: 3290 -> 2890 us per launch).  Same values per point as
// k_residual64_2.
constexpr int kRes2rRows = 128;

// With UPD the kernel first applies the inner solve's correction, as
// k_x_from_e does (x64 += e, e taking the pending update e + alpha p when
// pa != nullptr), to every row it reads, and forms the residual of the
// updated iterate: one pass instead of two.  It writes the updated x64 and
// clears e on its own rows except the first and last one of its segment;
// those are the rows a neighbouring workgroup reads (with their old x64
// and e), and k_update_seg_rows updates and clears them after this kernel.
struct XUpdate {
  const float* pa;      // nullptr: e alone
  const float* pb;
  const double* alpha;
  const int* iters;
  int assign;           // x64 = e instead of x64 += e (x64 not read: the first update of a solve)
};
template <bool VAR, bool UPD, typename RT = float>
__global__ __launch_bounds__(1024) void k_residual64_2r(LevelDev<double> L, const double* __restrict__ f,
                                                        double* __restrict__ x64, float* __restrict__ e,
                                                        RT* __restrict__ r32, const double* __restrict__ shift,
                                                        const int* __restrict__ active64, int nrhs,
                                                        double* __restrict__ partial,
                                                        unsigned long long* __restrict__ ctr, XUpdate xu) {
  constexpr int LW = 1024 + 2;
  __shared__ double sx[LW];   // x64 of the current row, zero pads at columns -1 and blockDim.x
  const RowTile rt = row_tile();
  const int sys = rt.sys, seg = rt.seg;
  if (!active64[sys]) return;
  count_bytes_row(rt, ctr, (unsigned long long)L.N * (8 + 8 + 4 + 4 + (UPD ? 8 + 4 : 0) + (VAR && sys == 0 ? 16 : 0)));
  const int n = L.n;
  const int i = threadIdx.x, NT = blockDim.x;
  const int j0 = seg * kRes2rRows, j1 = min(j0 + kRes2rRows, n);
  const bool col_on = i < n;
  const int ic = min(i, n - 1), q = 1 + i;
  const long long off = (long long)sys * L.N;
  double* __restrict__ xs = x64 + off;
  const double* __restrict__ fs = f + (long long)(sys % nrhs) * L.N;
  const double sh = shift[sys];
  const unsigned cb = (unsigned)ic * 8u, rowb = (unsigned)n * 8u;
  const RowBuf<double> xsb(xs, L.N), fsb(fs, L.N);
  const RowBuf<double> w0b(VAR ? L.wf0 : xs, VAR ? (long long)(n + 1) * n : 1), w1b(VAR ? L.wf1 : xs, VAR ? (long long)(n + 1) * n : 1);
  const RowBuf<RT> rb32(r32 + off, L.N);
  const RowBuf<float> eb(e + off, L.N);
  // the pending update of the inner solve (UPD)
  const int its = UPD && xu.pa ? xu.iters[sys] : 0;
  const float a = UPD && xu.pa ? (float)xu.alpha[sys] : 0.0f;
  const bool pend = its > 0 && a != 0.0f;
  const float* pl = pend ? (((its - 1) & 1) ? xu.pa : xu.pb) + off : e + off;
  const RowBuf<float> plb(pl, L.N);
  if (i < 2) sx[i == 0 ? 0 : NT + 1] = 0.0;
  auto crow = [&](int r) { return min(max(r, 0), n - 1); };
  // 1 on the grid, 0 off it (a factor, not a select: see k_spmv_r2)
  auto on_f = [&](int r) { return (col_on && r >= 0 && r < n) ? 1.0 : 0.0; };
  // the iterate of a row from its loads (UPD: x64 + e, the arithmetic of k_x_from_e)
  auto xnew = [&](double xv, float ev, float pv) {
    if (!UPD) return xv;
    const float en = pend ? ev + a * pv : ev;
    return xv + (double)en;
  };
  const bool assign = UPD && xu.assign;
  auto ldrow = [&](int r) {
    const unsigned o = (unsigned)crow(r) * rowb, o4 = (unsigned)crow(r) * (unsigned)n * 4u;
    const double xv = assign ? 0.0 : xsb.ld(cb, o);
    const float ev = UPD ? eb.ld(cb / 2, o4) : 0.0f, pv = UPD && pend ? plb.ld(cb / 2, o4) : 0.0f;
    return xnew(xv, ev, pv) * on_f(r);
  };
  // x64 of rows j - 1, j, j + 1 during step j (dn, c, up); before the first
  // step c and up hold rows j0 - 1 and j0
  double dn = 0.0, c = ldrow(j0 - 1), up = ldrow(j0);
  sx[q] = up;
  double rr = 0.0;
  ring_prologue_wait();
  __syncthreads();
  // the ring of row loads (see kRowLead): slot s of step j holds x64 (UPD:
  // and e, p) of row j + 1 and f and the faces of row j, as loaded (clamped
  // rows, unmasked)
  double rx[kRowLead], rf[kRowLead], wl[kRowLead], wr[kRowLead], wd[kRowLead], wu[kRowLead];
  float re[kRowLead], rp[kRowLead];
  auto fill = [&](int j, int s) {
    const unsigned rw = (unsigned)crow(j) * rowb, ra = (unsigned)crow(j + 1) * rowb;
    rx[s] = assign ? 0.0 : xsb.ld(cb, ra);
    if (UPD) {
      re[s] = eb.ld(cb / 2, ra / 2);
      rp[s] = pend ? plb.ld(cb / 2, ra / 2) : 0.0f;
    }
    rf[s] = fsb.ld(cb, rw);
    if (VAR) {
      const unsigned fx = (unsigned)crow(j) * (unsigned)(n + 1) * 8u;
      wl[s] = w0b.ld(cb, fx);
      wr[s] = w0b.ld(cb + 8u, fx);
      wd[s] = w1b.ld(cb, rw);
      wu[s] = w1b.ld(cb, rw + rowb);
    }
  };
#pragma unroll
  for (int s = 0; s < kRowLead; ++s) fill(j0 + s, s);
  ring_march(j0, j1 - 1, [&](int j, auto slot) {
    constexpr int s = decltype(slot)::value;
    const int row = j * n;   // 2D grids: fewer than 2^31 points
    dn = c;
    c = up;
    up = xnew(rx[s], UPD ? re[s] : 0.0f, UPD ? rp[s] : 0.0f) * on_f(j + 1);
    const double lv = sx[q - 1], rv = sx[q + 1];
    double ax;
    if (!VAR) ax = L.wc * ((c - lv) + (c - rv) + (c - dn) + (c - up)) + sh * c;
    else ax = wl[s] * (c - lv) + wr[s] * (c - rv) + wd[s] * (c - dn) + wu[s] * (c - up) + sh * c;
    const double rv64 = rf[s] - ax;
    if (col_on) {
      const unsigned g = (unsigned)row * 4u, ib = (unsigned)i * 4u;
      rb32.st((RT)rv64, ib * (unsigned)(sizeof(RT) / 4), g * (unsigned)(sizeof(RT) / 4));
      // UPD: the segment's first and last rows are left to k_update_seg_rows
      if (sizeof(RT) == 4 && (!UPD || (j != j0 && j != j1 - 1))) {
        eb.st(0.0f, ib, g);
        if (UPD) xsb.st(c, 2u * ib, 2u * g);
      }
      rr += rv64 * rv64;
    }
    __syncthreads();   // every read of row j's x64 is done
    sx[q] = up;
    __syncthreads();
    fill(j + kRowLead, s);
  });
  write_partial(partial, sys, rr, seg, rt.nseg);
}

// After k_residual64_2r<.., true>: x64 += e (with the pending update, as
// there) and e = 0 on the first and last row of every row segment.  One
// workgroup per system and such row, one thread per column.
__global__ __launch_bounds__(1024) void k_update_seg_rows(long long N, int n, double* __restrict__ x64,
                                                          float* __restrict__ e, const int* __restrict__ active64,
                                                          XUpdate xu) {
  const int sys = blockIdx.z;
  if (!active64[sys]) return;
  const int k = blockIdx.y;   // row 2 s or 2 s + 1 of segment s: its first or last row
  const int j0 = (k / 2) * kRes2rRows, j1 = min(j0 + kRes2rRows, n);
  const int j = (k & 1) ? j1 - 1 : j0;
  const int i = threadIdx.x;
  if (i >= n || ((k & 1) && j == j0)) return;   // a one-row segment: its row once
  const int its = xu.pa ? xu.iters[sys] : 0;
  const float a = xu.pa ? (float)xu.alpha[sys] : 0.0f;
  const bool pend = its > 0 && a != 0.0f;
  const long long g = (long long)sys * N + (long long)j * n + i;
  float en = e[g];
  if (pend) {
    const float* pl = ((its - 1) & 1) ? xu.pa : xu.pb;
    en = en + a * pl[g];
  }
  x64[g] = (xu.assign ? 0.0 : x64[g]) + (double)en;
  e[g] = 0.0f;
}

// the FP64 residual of a 2D batch of nsys systems walks whole rows when the
// other kernels do (levels of 255 - 1023 points, enough row segments)
static inline bool residual_rows(int dim, int n, long long nsys) {
  return dim == 2 && n >= kRowsMinN && n <= kRowsMaxN && nsys * ((n + kRes2rRows - 1) / kRes2rRows) >= kFillBlocks;
}

// k_residual64 in 3D, marching along z with kMarchRows rows per thread
template <bool VAR, typename RT = float>
__global__ __launch_bounds__(kBlock) void k_residual64_3(LevelDev<double> L, const double* __restrict__ f,
                                                         const double* __restrict__ x64, float* __restrict__ e,
                                                         RT* __restrict__ r32, const double* __restrict__ shift,
                                                         const int* __restrict__ active64, int nrhs,
                                                         double* __restrict__ partial,
                                                         unsigned long long* __restrict__ ctr) {
  constexpr int R = kMarchRows;
  const Tile tl = VAR ? block_tile_shared() : block_tile();
  const int sys = tl.z;
  if (!active64[sys]) return;
  count_bytes_tile(tl, ctr, (unsigned long long)L.N * (8 + 8 + 4 + 4 + (VAR && sys == 0 ? 8 * 3 : 0)));
  const int n = L.n;
  const Column c = march_column(tl, n, R);
  double rr = 0.0;
  if (c.i < n && c.j < n) {
    const long long off = (long long)sys * L.N, nn = (long long)n * n;
    const Rows<R> w(c.i, c.j, n);
    const double* xs = x64 + off;
    const double* fs = f + (long long)(sys % nrhs) * L.N;
    const double s = shift[sys];
    double below[R], centre[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const long long p0 = c.k0 * nn + w.col[r];
      const double xb0 = xs[c.k0 > 0 ? p0 - nn : p0];
      below[r] = c.k0 > 0 ? xb0 : 0.0;
      centre[r] = xs[p0];
    }
    ColFaces<double, VAR, R, true> fw;
    fw.start(L, w, c.k0);
    for (int k = c.k0; k < c.k1; ++k) {
      const long long pk = k * nn;
      double xa[R], xl[R], xr[R], fv[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const long long p = pk + w.col[r];
        xa[r] = xs[k + 1 < n ? p + nn : p];
        xl[r] = xs[p + w.il];
        xr[r] = xs[p + w.ir];
        fv[r] = fs[p];
      }
      const double hd = xs[pk + w.col_d], hu = xs[pk + w.col_u];
      fw.load(L, w, c.i, c.j, k);
      double above[R];
#pragma unroll
      for (int r = 0; r < R; ++r) above[r] = k + 1 < n ? xa[r] : 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!w.valid[r]) continue;
        const long long p = pk + w.col[r];
        const double ax = apply_col3(L, fw, r, centre[r], w.il ? xl[r] : 0.0, w.ir ? xr[r] : 0.0,
                                                     w.down(r, centre, hd), w.up(r, centre, hu), below[r], above[r], s);
        const double rv = fv[r] - ax;
        r32[off + p] = (RT)rv;
        if constexpr (sizeof(RT) == 4) e[off + p] = 0.0f;
        rr += rv * rv;
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        below[r] = centre[r];
        centre[r] = above[r];
      }
    }
  }
  write_partial_tile(tl, partial, sys, rr);
}

// first refinement step: x64 = 0 so r = f; partial = ||f||^2
// zero_x false: x64 is cleared only where f is 0 (a right-hand side that is
// 0 everywhere leaves its system inactive, and its x64 must read 0); the
// first x64 update of the refinement then assigns x64 = e instead of adding
__global__ __launch_bounds__(256) void k_first_residual(long long N, const double* __restrict__ f,
                                                        double* __restrict__ x64, float* __restrict__ e,
                                                        float* __restrict__ r32, int nrhs,
                                                        const int* __restrict__ active64,
                                                        double* __restrict__ partial, bool zero_x) {
  const int sys = blockIdx.y;
  if (!active64[sys]) return;
  const int rhs = sys % nrhs;
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
  double ff = 0.0;
  double fl[kFlatItems];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) fl[it] = f[(long long)rhs * N + min(base + (long long)it * 256, N - 1)];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = base + (long long)it * 256;
    if (p < N) {
      const double fv = fl[it];
      r32[off + p] = (float)fv;
      if (zero_x || fv == 0.0) x64[off + p] = 0.0;
      e[off + p] = 0.0f;
      ff += fv * fv;
    }
  }
  write_partial_flat(partial, sys, ff);
}

// x64 += e (final refinement update after the last inner solve)
// With pa != nullptr the inner solve's last deferred iterate update is
// applied here too (as k_finish_x would, in FP32 and the same expression):
// e + alpha p_last is formed in registers and never stored, one pass less.
__global__ __launch_bounds__(256) void k_x_from_e(long long N, const float* __restrict__ e, double* __restrict__ x64,
                                                  const int* __restrict__ active64, const float* __restrict__ pa,
                                                  const float* __restrict__ pb, const double* __restrict__ alpha,
                                                  const int* __restrict__ iters) {
  const int sys = blockIdx.y;
  if (!active64[sys]) return;
  const long long off = (long long)sys * N;
  const long long base = (long long)blockIdx.x * 256 * kFlatItems + threadIdx.x;
  const int its = pa ? iters[sys] : 0;
  const float a = pa ? (float)alpha[sys] : 0.0f;
  const bool pend = its > 0 && a != 0.0f;
  const float* pl = ((its - 1) & 1) ? pa : pb;
  double xl[kFlatItems];
  float el[kFlatItems], pv[kFlatItems];
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = min(base + (long long)it * 256, N - 1);
    xl[it] = x64[off + p];
    el[it] = e[off + p];
    pv[it] = pend ? pl[off + p] : 0.0f;
  }
#pragma unroll
  for (int it = 0; it < kFlatItems; ++it) {
    const long long p = base + (long long)it * 256;
    const float en = pend ? el[it] + a * pv[it] : el[it];
    if (p < N) x64[off + p] = xl[it] + (double)en;
  }
}

// Output o (blockIdx.z), right-hand side r (blockIdx.y):
// u[o rows + r] = base_w base[r] + sum_j w_j x[j * stride + r] over the output's
// terms, summed in the fixed order base, j = begin..end-1 (eq. (16); the base
// term serves the sequential forms).  base may be u itself (each element is
// read before it is written).
// With pa != nullptr each system's last deferred iterate update is still
// pending and is applied here, as k_finish_x would (same expression), while x
// is read: x_j + alpha_j p_j, never stored (p = pa or pb by the parity of the
// system's iteration count).
// With partial != nullptr the block's sum of u^2 goes there (k_row_sum adds
// them: the output norms of the error bound, without reading u again).
// kCombineItems points per thread, every load of a term in flight before the
// sums (1023^2, 10 terms: one point per thread moved 4.2 TB/s).
constexpr int kCombineItems = 4;
__global__ __launch_bounds__(256) void k_combine(long long N, const double* x, const double* __restrict__ w,
                                                 CombineTerms t, int stride, double* u, const double* base,
                                                 double base_w, unsigned long long* __restrict__ ctr, int wsys,
                                                 const double* __restrict__ pa, const double* __restrict__ pb,
                                                 const double* __restrict__ alpha, const int* __restrict__ iters,
                                                 double* __restrict__ partial) {
  constexpr int K = kCombineItems;
  const int r = blockIdx.y, o = blockIdx.z;
  const int jb = t.begin[o], je = t.begin[o + 1];
  const int row = o * gridDim.y + r;
  const long long p0 = (long long)blockIdx.x * 256 * K + threadIdx.x;
  count_bytes<COUNT_FLAT>(ctr, (unsigned long long)N * 8ULL * ((je - jb) * (pa ? 2 : 1) + 1 + (base ? 1 : 0)));
  long long pt[K];
  double acc[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    pt[i] = min(p0 + 256 * i, N - 1);
    acc[i] = base ? base_w * base[(long long)r * N + pt[i]] : 0.0;
  }
#pragma unroll 2
  for (int j = jb; j < je; ++j) {
    const long long sys = (long long)j * stride + r;
    const double wv = wsys ? w[sys] : w[j];
    // per-system weights: a zero weight marks an unused slot, whose x is not read
    if (wsys && wv == 0.0) continue;
    double xv[K];
#pragma unroll
    for (int i = 0; i < K; ++i) xv[i] = x[sys * N + pt[i]];
    if (pa) {
      const int it = iters[sys];
      const double a = alpha[sys];
      if (it > 0 && a != 0.0) {
        const double* pl = (((it - 1) & 1) ? pa : pb) + sys * N;
#pragma unroll
        for (int i = 0; i < K; ++i) xv[i] = xv[i] + a * pl[pt[i]];
      }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) acc[i] += wv * xv[i];
  }
  double uu = 0.0;
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (p0 + 256 * i < N) {
      u[(long long)row * N + pt[i]] = acc[i];
      uu += acc[i] * acc[i];
    }
  if (partial) write_partial(partial, row, uu, blockIdx.x, gridDim.x);
}

// out[r] = the sum of the nblk partials of row r, in a fixed order (the result
// does not depend on which other rows share the launch)
__global__ __launch_bounds__(1024) void k_row_sum(const double* __restrict__ partial, int nblk,
                                                  double* __restrict__ out) {
  const int r = blockIdx.x;
  double v = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) v += partial[(size_t)r * nblk + b];
  const double tot = block_sum(v);
  if (threadIdx.x == 0) out[r] = tot;
}

template <int DIM, bool VAR>
__global__ __launch_bounds__(kBlock) void k_apply64(LevelDev<double> L, const double* __restrict__ x,
                                                    double* __restrict__ y, double s) {
  const Tile tl = block_tile();
  const int v = tl.z;
  int i, j, k;
  tile_ijk<DIM>(tl, L.n, i, j, k);
  if (i >= L.n || j >= L.n) return;
  const long long off = (long long)v * L.N;
  const long long p = ((long long)k * L.n + j) * L.n + i;
  y[off + p] = apply_pt<double, DIM, VAR>(L, x + off, i, j, k, p, s, nullptr);
}

// --------------------------------------------------------------------------
// per-system scalar updates: one block per system sums the block partials in
// a fixed order, thread 0 advances that system's state.
// --------------------------------------------------------------------------
__device__ void apply_op(int op, double tot, const SysState& S, int sys, double tol, int max_iter) {
  switch (op) {
    case OP_INIT: {  // tot = ||b||^2 of the PCG right-hand side
      S.bnorm2[sys] = tot;
      S.iters[sys] = 0;
      S.relres[sys] = 1.0;
      S.beta[sys] = 0.0;
      S.alpha[sys] = 0.0;   // no deferred iterate update pending
      if (!(tot > 0.0)) {
        S.active[sys] = 0;
        if (!isfinite(tot)) S.flags[sys] |= 1;
        S.relres[sys] = 0.0;
      }
      break;
    }
    case OP_BETA: {  // tot = r.z
      if (S.iters[sys] == 0) {
        S.rho[sys] = tot;
        S.beta[sys] = 0.0;
      } else {
        S.beta[sys] = tot / S.rho[sys];
        S.rho[sys] = tot;
      }
      if (!isfinite(tot)) {
        S.flags[sys] |= 1;
        S.active[sys] = 0;
      }
      break;
    }
    case OP_ALPHA: {  // tot = p.q
      if (!(tot > 0.0) || !isfinite(tot)) {
        // p.q <= 0 only when the residual has vanished to rounding: stop here
        if (!isfinite(tot)) S.flags[sys] |= 1;
        S.active[sys] = 0;
        S.alpha[sys] = 0.0;
      } else {
        S.alpha[sys] = S.rho[sys] / tot;
      }
      break;
    }
    case OP_RESID: {  // tot = ||r||^2
      const int it = S.iters[sys] + 1;
      S.iters[sys] = it;
      S.total_iters[sys] += 1;
      const double rel = sqrt(tot / S.bnorm2[sys]);
      S.relres[sys] = rel;
      if (!isfinite(rel)) {
        S.flags[sys] |= 1;
        S.active[sys] = 0;
      } else if (rel <= (S.tol_inner ? S.tol_inner[sys] : S.tol_pcg ? S.tol_pcg[sys] : tol) || it >= max_iter) {
        S.active[sys] = 0;
      }
      break;
    }
    case OP_START: {  // tot = ||f||^2; the first OP_OUTER follows, on the direct solution's residual
      S.alpha[sys] = 0.0;
      if (!isfinite(tot)) {
        S.flags[sys] |= 1;
        S.relres64[sys] = tot;
        S.active64[sys] = 0;
        S.active[sys] = 0;
        break;
      }
      S.fnorm2[sys] = tot;
      if (!(tot > 0.0)) {
        S.relres64[sys] = 0.0;
        S.outer[sys] = 1;
        S.active64[sys] = 0;
        S.active[sys] = 0;
      }
      break;
    }
    case OP_RESTART: {  // tot = ||f - (A+s) x||^2 of the direct solution
      const double rel = sqrt(tot / S.bnorm2[sys]);
      S.relres[sys] = rel;
      if (!isfinite(rel)) {
        S.flags[sys] |= 1;
        S.active[sys] = 0;
      } else if (rel <= (S.tol_pcg ? S.tol_pcg[sys] : tol)) {
        S.active[sys] = 0;
      }
      break;
    }
    case OP_OUTER: {  // tot = ||f - (A+s) x64||^2 ; first call: x64 = 0 so tot = ||f||^2
      const int o = S.outer[sys];
      S.alpha[sys] = 0.0;   // the inner solve's deferred update has been applied (or is void)
      if (!isfinite(tot)) {
        S.flags[sys] |= 1;
        S.relres64[sys] = tot;
        S.active64[sys] = 0;
        S.active[sys] = 0;
        break;
      }
      if (o == 0 && !S.started) S.fnorm2[sys] = tot;
      const double fn = S.fnorm2[sys];
      const double rel = fn > 0.0 ? sqrt(tot / fn) : 0.0;
      S.relres64[sys] = rel;
      S.outer[sys] = o + 1;
      const double to = S.tol_outer ? S.tol_outer[sys] : tol;
      if (rel <= to || o >= max_iter) {
        S.active64[sys] = 0;
        S.active[sys] = 0;
      } else {
        S.active[sys] = 1;   // re-arm the inner solve on this residual
        S.bnorm2[sys] = tot;
        S.iters[sys] = 0;
        S.relres[sys] = 1.0;
        S.beta[sys] = 0.0;
        if (S.tol_inner) {
          // a step that can finish the system asks only for what is left
          const double want = 0.5 * to / rel;
          S.tol_inner[sys] = want > S.inner_floor ? want : S.inner_floor;
        }
      }
      break;
    }
  }
}

// With pr.host set, the last block to end tells the host how many systems are
// active after the operation: one 64-bit count of the blocks (low half) and of
// the active systems (high half), left at 0 for the next launch.
__global__ __launch_bounds__(256) void k_scalars(int op, const double* __restrict__ partial, int nblk, SysState S,
                                                 double tol, int max_iter, Progress pr) {
  const int sys = blockIdx.x;
  const int* act = op != OP_OUTER ? S.active : S.active64;
  const bool on = act[sys] != 0;
  if (on) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) v += partial[(size_t)sys * nblk + b];
    const double tot = block_sum(v);
    if (threadIdx.x == 0) apply_op(op, tot, S, sys, tol, max_iter);
  }
  if (!pr.host || threadIdx.x != 0) return;
  const unsigned long long mine = 1ULL + (on && act[sys] ? 1ULL << 32 : 0ULL);
  const unsigned long long tot = atomicAdd(pr.count, mine) + mine;
  if ((unsigned)tot != gridDim.x) return;
  atomicExch(pr.count, 0ULL);
  const unsigned long long seq = pr.count[1] + 1;   // only one block gets here in a launch
  pr.count[1] = seq;
  __hip_atomic_store(pr.host, seq << 32 | tot >> 32, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The scalar state of system i at the start of a solve: counters and flags
// cleared, no iterate update pending, the used systems active: system j R + r
// for r < nrhs, or as the uploaded slot terms say, which are unpacked to the
// per-system arrays.  Returns whether the system is used.
__device__ __forceinline__ int begin_system(const SysState& S, int i, int nsys, int R, int nrhs,
                                            const SlotUpload& up) {
  S.flags[i] = 0;
  S.total_iters[i] = 0;
  S.outer[i] = 0;
  S.alpha[i] = 0.0;
  int on = (i % R) < nrhs;
  if (up.staged) {
    const double* h = up.staged;
    up.w[i] = h[i];
    up.s64[i] = h[nsys + i];
    up.tol[i] = h[2 * nsys + i];
    const float* h32 = reinterpret_cast<const float*>(h + 3 * (size_t)nsys);
    if (up.s32) up.s32[i] = h32[i];
    if (up.s64b) up.s64b[i] = h[nsys + i];
    on = reinterpret_cast<const int*>(h32 + nsys)[i];
  }
  S.active[i] = on;
  S.active64[i] = on;
  return on;
}

// One block per system: see launch_start.  BEGIN: the solve's first launch on
// the scalar state (begin_system of all nsys = gridDim.x systems).
template <bool BEGIN>
__global__ __launch_bounds__(256) void k_start(int op, const double* __restrict__ partial, int nblk, int R,
                                               SysState S, int* __restrict__ gate, double tol, int nrhs,
                                               SlotUpload up) {
  const int sys = blockIdx.x, nsys = gridDim.x;
  const bool mixed = op == OP_START;
  const double* per = mixed ? S.tol_outer : S.tol_pcg;
  double stop = per ? per[sys] : tol;
  int act;
  if (BEGIN) {
    act = (sys % R) < nrhs;
    if (up.staged) {
      act = reinterpret_cast<const int*>(reinterpret_cast<const float*>(up.staged + 3 * (size_t)nsys) + nsys)[sys];
      stop = up.staged[2 * (size_t)nsys + sys];
    }
    if (threadIdx.x == 0) begin_system(S, sys, nsys, R, nrhs, up);
  } else {
    act = (mixed ? S.active64 : S.active)[sys];
  }
  if (!act) {
    if (threadIdx.x == 0) gate[sys] = 0;
    return;
  }
  double v = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) v += partial[(size_t)(sys % R) * nblk + b];
  const double tot = block_sum(v);
  if (threadIdx.x != 0) return;
  apply_op(op, tot, S, sys, tol, 0);
  gate[sys] = tot > 0.0 && isfinite(tot) && stop <= kDirectTol ? 1 : 2;
}

// The end of a solve in one workgroup: op applied to every system (op < 0: none
// is left to), the output norms summed, and the state handed to the host:
// `words` doubles from `state` to pinned memory, then the sequence number that
// the host waits for.  A wave sums a system's partials; for a few hundred
// systems this is shorter than three launches and a copy, of 3 - 5 us each.
__global__ __launch_bounds__(1024) void k_conclude(int op, const double* __restrict__ partial, int nblk, int nsys,
                                                   SysState S, double tol, int max_iter,
                                                   const double* __restrict__ upartial, int unblk, int rows,
                                                   double* unorm, const double* state, int words, double* host,
                                                   unsigned* host_seq, unsigned seq) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  auto wave_sum = [&](const double* p, int n) {
    double v = 0.0;
    int b = lane;
    for (; b + 7 * 64 < n; b += 8 * 64) {   // eight loads in flight
      double w[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) w[k] = p[b + k * 64];
#pragma unroll
      for (int k = 0; k < 8; ++k) v += w[k];
    }
    for (; b < n; b += 64) v += p[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
  if (op >= 0)
    for (int s = wave; s < nsys; s += 16) {
      if (!(op == OP_OUTER ? S.active64 : S.active)[s]) continue;
      const double tot = wave_sum(partial + (size_t)s * nblk, nblk);
      if (lane == 0) apply_op(op, tot, S, s, tol, max_iter);
    }
  for (int r = 15 - wave; r < rows; r += 16) {
    const double tot = wave_sum(upartial + (size_t)r * unblk, unblk);
    if (lane == 0) unorm[r] = tot;
  }
  __syncthreads();
  for (int i = tid; i < words; i += 1024) host[i] = state[i];
  __threadfence_system();
  __syncthreads();
  if (tid == 0) __hip_atomic_store(host_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// n flags to pinned memory, then the sequence number
__global__ __launch_bounds__(1024) void k_report_flags(const int* __restrict__ flags, int n, int* host,
                                                       unsigned* host_seq, unsigned seq) {
  for (int i = threadIdx.x; i < n; i += 1024) host[i] = flags[i];
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(host_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------
// one point per thread (2D stencil kernels; 3D transfer operators)
static inline dim3 point_grid(int dim, int n, int nsys) {
  const int xt = (n + kTileX - 1) / kTileX;
  const int yt = (n + kTileY - 1) / kTileY;
  return dim3(xt, yt * (dim == 3 ? n : 1), nsys);
}

// 3D kernels marching along z: kMarchZ planes per workgroup, `rows` rows per thread
// Threads along x of a marching workgroup on a grid of n points per axis (the
// rest of the 256 along y).  Rows of n points are not aligned to 128-byte
// lines, so a wide row segment wastes a smaller share of its lines (255^3
// mixed: 64 -> 128 -> 256 columns took the solve from 39.9 to 37.4 to
// 36.5 ms); a narrow grid would leave most of a wide workgroup idle.
static inline int march_x(int n) { return n >= 192 ? 256 : (n >= 96 ? 128 : 64); }
static inline dim3 march_block(int n) { return dim3(march_x(n), kBlock / march_x(n)); }

// Planes per workgroup of a marching launch with `tiles` workgroups per layer
// of planes (over all its systems): kMarchZ, halved while that leaves fewer
// than 8 workgroups per CU.  A workgroup walks its planes one memory latency at
// a time, so on the coarse levels of a few systems 8 planes are 8 - 28 us
// whatever the grid (127^3, 9 systems, variable coefficients, on its 63^3 and
// 31^3 levels: sweeps 9.6 and 8.1 -> 7.2 and 4.8 us, sweeps from zero 20 and 17
// -> under 8, restrictions 23 and 24 -> 15 and 8); shorter walks read their
// first and last plane again.  Only for kernels that write no partials: those
// are grouped by kMarchZ, whatever else shares the launch.
// Below `few` planes only while there are fewer than 4 workgroups per CU: a
// restriction reads 2 mz + 1 fine planes for mz coarse ones (15^3 FP32, 512 systems: 2 planes 33
// us, 4 planes 28, 8 planes 26; 63^3, 18 systems: 1 plane 15.8, 2 planes 13.9).
static inline int march_planes(int n, long long tiles, int least, int few = 0) {
  int mz = kMarchZ;
  while (mz > least && tiles * ((n + mz - 1) / mz) < (mz > few ? 2048 : 1024)) mz /= 2;
  return mz;
}

static inline dim3 march_grid(int n, int nsys, int rows, int planes = kMarchZ) {
  const int mx = march_x(n), my = kBlock / mx;
  const int xt = (n + mx - 1) / mx;
  const int yt = (n + my * rows - 1) / (my * rows);
  const int zt = (n + planes - 1) / planes;
  return dim3(xt, yt * zt, nsys);
}

static inline long long march_tiles(int n, int nsys, int rows) {
  const int mx = march_x(n), my = kBlock / mx;
  return (long long)((n + mx - 1) / mx) * ((n + my * rows - 1) / (my * rows)) * nsys;
}

// the smoothing sweeps, the stencil product and the FP64 residual (the kernels
// that write per-block partials outside the fused 2D path)
static inline dim3 stencil_grid(int dim, int n, int nsys) {
  return dim == 3 ? march_grid(n, nsys, kMarchRows) : point_grid(dim, n, nsys);
}
static inline dim3 stencil_block(int dim, int n) { return dim == 3 ? march_block(n) : dim3(kTileX, kTileY); }

int stencil_blocks(int dim, int n) {
  const dim3 g = stencil_grid(dim, n, 1);
  return (int)(g.x * g.y);
}

// the 2D stencil product: TX x ((256 / TX) R) points per workgroup
static inline dim3 spmv2_grid(int n, int nsys, int tv) {
  const int tx = kSpmvTile[tile_variant(tv)][1];
  const int rows = (kBlock / tx) * kSpmvTile[tile_variant(tv)][0];
  return dim3((n + tx - 1) / tx, (n + rows - 1) / rows, nsys);
}

int spmv_blocks(int dim, int n, int tv) {
  if (dim != 2) return stencil_blocks(dim, n);
  if (spmv_rows(dim, n, tv)) return (n + rows_seg(tv) - 1) / rows_seg(tv);
  const dim3 g = spmv2_grid(n, 1, tv);
  return (int)(g.x * g.y);
}

int flat_blocks(long long N) {
  const long long per = 256LL * kFlatItems;
  return (int)((N + per - 1) / per);
}

static inline dim3 flat_grid(long long N, int nsys) {
  const long long per = 256LL * kFlatItems;
  return dim3((unsigned)((N + per - 1) / per), nsys, 1);
}

// Calls f(std::integral_constant<int, v>) for the runtime variant tv.
template <typename F>
static inline void with_tile(int tv, F&& f) {
  static_assert(kTileVariants == 5, "one case per variant");
  switch (tile_variant(tv)) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    default: f(std::integral_constant<int, 0>{}); break;
  }
}


bool tile_variant_distinct(int kind, int dim, int n, int tv) {
  (void)kind;
  const int v = tile_variant(tv);
  if (v != kRowsVariant && v != kShortRowsVariant) return true;
  return down_rows(dim, n, tv);
}

#define BURA_DISPATCH_DV(dim, var, KERNEL, ...)        \
  do {                                                 \
    if (dim == 2) {                                    \
      if (var) KERNEL(2, true, __VA_ARGS__);           \
      else KERNEL(2, false, __VA_ARGS__);              \
    } else {                                           \
      if (var) KERNEL(3, true, __VA_ARGS__);           \
      else KERNEL(3, false, __VA_ARGS__);              \
    }                                                  \
  } while (0)

template <typename T>
void Launch<T>::jacobi(int dim, bool var, const LevelDev<T>& L, const T* b, const T* xin, T* xout, const T* shift,
                       const int* active, T omega, bool zero_guess, double* partial, int nsys, hipStream_t st,
                       unsigned long long* ctr, Fin fin) {
  const bool dot = partial != nullptr;
  // (a sweep from zero reads no other plane, so it may take them one by one)
  const int mz = dim == 3 && !dot ? march_planes(L.n, march_tiles(L.n, nsys, kMarchRows), zero_guess ? 1 : 2) : kMarchZ;
  const dim3 g = dim == 3 ? march_grid(L.n, nsys, kMarchRows, mz) : stencil_grid(dim, L.n, nsys);
  const dim3 blk = stencil_block(dim, L.n);
#define K_JAC(D, V, Z, DT)                                                                                      \
  do {                                                                                                          \
    if (D == 3)                                                                                                 \
      hipLaunchKernelGGL((k_jacobi3<T, V, Z, DT>), g, blk, 0, st, L, b, xin, xout, shift, active, omega, partial, \
                         ctr, fin, mz);                                                                         \
    else                                                                                                        \
      hipLaunchKernelGGL((k_jacobi<T, 2, V, Z, DT>), g, blk, 0, st, L, b, xin, xout, shift, active, omega,       \
                         partial, ctr, fin);                                                                    \
  } while (0)
#define K_JAC4(D, V, dummy)                       \
  do {                                            \
    if (zero_guess) {                             \
      if (dot) K_JAC(D, V, true, true);           \
      else K_JAC(D, V, true, false);              \
    } else {                                      \
      if (dot) K_JAC(D, V, false, true);          \
      else K_JAC(D, V, false, false);             \
    }                                             \
  } while (0)
  BURA_DISPATCH_DV(dim, var, K_JAC4, 0);
#undef K_JAC4
#undef K_JAC
}

template <typename T>
void Launch<T>::jacobi_rup(int dim, bool var, const LevelDev<T>& L, const T* bold, const T* q, const double* alpha,
                           T* bout, T* xout, const T* shift, const int* active, T omega, double* partial, int nsys,
                           hipStream_t st, unsigned long long* ctr, Fin fin, const T* p) {
  const dim3 g = stencil_grid(dim, L.n, nsys), blk = stencil_block(dim, L.n);
  if (dim == 3 && !q) {   // q formed from p
    if (var)
      hipLaunchKernelGGL((k_jacobi0_rup3p<T, true>), g, blk, 0, st, L, bold, p, alpha, bout, xout, shift, active,
                         omega, partial, ctr, fin);
    else
      hipLaunchKernelGGL((k_jacobi0_rup3p<T, false>), g, blk, 0, st, L, bold, p, alpha, bout, xout, shift, active,
                         omega, partial, ctr, fin);
    return;
  }
#define K_JR(D, V, dummy)                                                                                         \
  hipLaunchKernelGGL((k_jacobi0_rup<T, D, V>), g, blk, 0, st, L, bold, q, alpha, bout, xout, shift, active, omega, \
                     partial, ctr, fin)
  BURA_DISPATCH_DV(dim, var, K_JR, 0);
#undef K_JR
}

template <typename T>
void Launch<T>::restrict_residual(int dim, bool var, const LevelDev<T>& Lf, const LevelDev<T>& Lc, const T* b,
                                  const T* x, T* bc, const T* shift, const int* active, int nsys, hipStream_t st,
                                  unsigned long long* ctr) {
  if (dim == 3) {
    const int nc = Lc.n;
    const int xt = (nc + kRcx - 1) / kRcx, yt = (nc + kRcy - 1) / kRcy;
    const int mz = march_planes(nc, (long long)xt * yt * nsys, 1, 4);
    const dim3 g3(xt, yt * ((nc + mz - 1) / mz), nsys);
    if (var) hipLaunchKernelGGL((k_restrict3<T, true>), g3, dim3(256), 0, st, Lf, Lc, b, x, bc, shift, active, ctr, mz);
    else hipLaunchKernelGGL((k_restrict3<T, false>), g3, dim3(256), 0, st, Lf, Lc, b, x, bc, shift, active, ctr, mz);
    return;
  }
  const dim3 g = point_grid(dim, Lc.n, nsys), blk(kTileX, kTileY);
#define K_RES(D, V, dummy) hipLaunchKernelGGL((k_restrict<T, D, V>), g, blk, 0, st, Lf, Lc, b, x, bc, shift, active, ctr)
  BURA_DISPATCH_DV(dim, var, K_RES, 0);
#undef K_RES
}

template <typename T>
void Launch<T>::prolong_add(int dim, const LevelDev<T>& Lc, const LevelDev<T>& Lf, const T* xc, T* xf,
                            const int* active, int nsys, hipStream_t st, unsigned long long* ctr) {
  if (dim == 2)
    hipLaunchKernelGGL((k_prolong<T, 2>), point_grid(2, Lf.n, nsys), dim3(kTileX, kTileY), 0, st, Lc, Lf, xc, xf,
                       active, ctr);
  else {
    const int mz = march_planes(Lf.n, march_tiles(Lf.n, nsys, 1), 2);
    hipLaunchKernelGGL((k_prolong3<T>), march_grid(Lf.n, nsys, 1, mz), march_block(Lf.n), 0, st, Lc, Lf, xc, xf,
                       active, ctr, mz);
  }
}

template <typename T>
void Launch<T>::coarse_solve(int dim, bool var, const LdsHierarchy<T>& H, const T* b, T* x, const T* shift,
                             const int* active, int nsys, size_t lds_bytes, hipStream_t st,
                             unsigned long long* ctr) {
  // As many threads as the first level has points, in steps of 256, 512 and
  // 1024.  Where there are enough systems to fill the chip either way, the
  // threads that the levels below leave idle count: 31^2 then takes two points
  // per thread of 512.  FP64, 2048 systems: 31^2 64 -> 40 us, 15^2 42 -> 32,
  // 7^3 38 -> 28.
  const int N0 = (int)H.lev[0].N, N1 = H.nlev > 1 ? (int)H.lev[1].N : 0;
  const int per = (N0 + kCoarseThreads - 1) / kCoarseThreads;
  const int elems = (int)(lds_bytes / sizeof(T));
#define K_CO(D, V, P, NT_)                                                                                       \
  do {                                                                                                           \
    auto* kern = k_coarse<T, D, V, P, NT_>;                                                                      \
    if (lds_bytes > 64 * 1024)                                                                                   \
      (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);  \
    hipLaunchKernelGGL(kern, dim3(nsys), dim3(NT_), lds_bytes, st, H, b, x, shift, active, ctr, elems);          \
  } while (0)
#define K_COP(D, V, dummy)                                                \
  do {                                                                    \
    if (N0 <= 256) K_CO(D, V, 1, 256);                                    \
    else if (N0 <= 512) K_CO(D, V, 1, 512);                               \
    else if (N0 <= 1024 && N1 <= 512 && nsys >= 1024) K_CO(D, V, 2, 512); \
    else if (per <= 1) K_CO(D, V, 1, kCoarseThreads);                     \
    else if (per == 2) K_CO(D, V, 2, kCoarseThreads);                     \
    else if (per <= 4) K_CO(D, V, 4, kCoarseThreads);                     \
    else K_CO(D, V, 6, kCoarseThreads);                                   \
  } while (0)
  BURA_DISPATCH_DV(dim, var, K_COP, 0);
#undef K_COP
#undef K_CO
}

template <typename T>
void Launch<T>::update_xr(const LevelDev<T>& L, int dim, T* x, T* r, const T* p, const T* q, const double* alpha,
                          const int* active, double* partial, int nsys, hipStream_t st, unsigned long long* ctr,
                          Fin fin) {
  (void)dim;
  hipLaunchKernelGGL((k_update_xr<T>), flat_grid(L.N, nsys), dim3(256), 0, st, L.N, x, r, p, q, alpha, active, partial,
                     ctr, fin);
}

template <typename T>
void Launch<T>::update_p(const LevelDev<T>& L, int dim, T* p, const T* z, const double* beta, const int* active,
                         int nsys, hipStream_t st, unsigned long long* ctr) {
  (void)dim;
  hipLaunchKernelGGL((k_update_p<T>), flat_grid(L.N, nsys), dim3(256), 0, st, L.N, p, z, beta, active, ctr);
}

template <typename T>
void Launch<T>::copy_rhs(const LevelDev<T>& L, int dim, const double* f, T* r, T* x, int nrhs, const int* active,
                         double* partial, int nsys, hipStream_t st) {
  (void)dim;
  // a batch is either all systems (sys = j * nrhs + r) or one pole (sys = r): rhs = sys % nrhs
  hipLaunchKernelGGL((k_copy_rhs<T>), flat_grid(L.N, nsys), dim3(256), 0, st, L.N, f, r, x, nrhs, active, partial);
}

template <typename T>
void Launch<T>::spmv_p(int dim, bool var, const LevelDev<T>& L, const T* z, const T* pold, T* pnew, T* q,
                       const double* beta, const T* shift, const int* active, double* partial, int nsys,
                       hipStream_t st, unsigned long long* ctr, Fin fin, T* x, const double* alpha, int tv) {
  const bool xup = x != nullptr;
  if (dim == 2 && spmv_rows(dim, L.n, tv)) {
    const int rows = rows_seg(tv);
    const dim3 g = rows_grid((L.n + rows - 1) / rows, nsys), blk(pair_threads(L.n));
#define K_SR(V, X_, Q_) \
  hipLaunchKernelGGL((k_spmv_r2<T, V, X_, Q_>), g, blk, row_lds_bytes<T>(k_spmv_r2<T, V, X_, Q_>, spmv_words(), blk.x), \
                     st, L, z, pold, pnew, q, beta, shift, active, partial, \
                     ctr, fin, x, alpha, rows)
    if (var) {
      if (!q) K_SR(true, true, false); else if (xup) K_SR(true, true, true); else K_SR(true, false, true);
    } else {
      if (!q) K_SR(false, true, false); else if (xup) K_SR(false, true, true); else K_SR(false, false, true);
    }
#undef K_SR
    return;
  }
  if (dim == 2) {
    const dim3 g2 = spmv2_grid(L.n, nsys, tv);
    with_tile(tv, [&](auto v) {
      constexpr int R = kSpmvTile[decltype(v)::value][0], TX = kSpmvTile[decltype(v)::value][1];
      const dim3 blk2(TX, kBlock / TX);
#define K_SP2(V, X_, Q_) \
  hipLaunchKernelGGL((k_spmv_p2<T, V, X_, Q_, R, TX>), g2, blk2, 0, st, L, z, pold, pnew, q, beta, shift, active, \
                     partial, ctr, fin, x, alpha)
      // q == nullptr: the product is only dotted with p (the fused down
      // kernel forms it again from p); that needs the deferred x update
      if (var) {
        if (!q) K_SP2(true, true, false); else if (xup) K_SP2(true, true, true); else K_SP2(true, false, true);
      } else {
        if (!q) K_SP2(false, true, false); else if (xup) K_SP2(false, true, true); else K_SP2(false, false, true);
      }
#undef K_SP2
    });
    return;
  }
  const dim3 g = march_grid(L.n, nsys, kMarchRows), blk = march_block(L.n);
#define K_SP3(V, X_, Q_)                                                                                          \
  hipLaunchKernelGGL((k_spmv_p3<T, V, X_, Q_>), g, blk, 0, st, L, z, pold, pnew, q, beta, shift, active, partial, \
                     ctr, fin, x, alpha)
  // q == nullptr: only p_new.q (the first fine sweep forms q from p_new)
  if (var) {
    if (!q) K_SP3(true, true, false); else if (xup) K_SP3(true, true, true); else K_SP3(true, false, true);
  } else {
    if (!q) K_SP3(false, true, false); else if (xup) K_SP3(false, true, true); else K_SP3(false, false, true);
  }
#undef K_SP3
}

template <typename T>
void Launch<T>::finish_x(long long N, T* x, const T* pa, const T* pb, const double* alpha, const int* iters,
                         int nsys, hipStream_t st, unsigned long long* ctr) {
  hipLaunchKernelGGL((k_finish_x<T>), flat_grid(N, nsys), dim3(256), 0, st, N, x, pa, pb, alpha, iters, ctr);
}

template <typename T>
bool Launch<T>::fused_down(int dim, bool var, int nu, const LevelDev<T>& Lf, const LevelDev<T>& Lc, const T* b,
                           T* xout, T* bc, const T* shift, const int* active, Sweeps<T> om, int nsys, hipStream_t st,
                           unsigned long long* ctr, const T* p, const double* alpha, T* bout, double* partial,
                           Fin fin, int tv, int tv_up) {
  const bool rup = bout != nullptr;
  if (dim == 3) {
    if (var || nu < 1 || nu > 2) return false;
    const dim3 g((Lc.n + kD3Cx - 1) / kD3Cx, ((Lc.n + kD3Cy - 1) / kD3Cy) * ((Lc.n + kD3Kz - 1) / kD3Kz), nsys);
#define K_D3(NU_, R_)                                                                                        \
  hipLaunchKernelGGL((k_down3<T, NU_, R_>), g, dim3(kF3Threads), 0, st, Lf, Lc, b, xout, bc, shift, active, om, ctr, \
                     p, alpha, bout, partial, fin)
    if (rup) {
      if (nu == 1) K_D3(1, true); else K_D3(2, true);
    } else {
      if (nu == 1) K_D3(1, false); else K_D3(2, false);
    }
#undef K_D3
    return true;
  }
  if (dim != 2 || nu < 1 || nu > 3) return false;
  if (down_rows(dim, Lf.n, tv)) {
    if (up_rows(dim, Lf.n, tv_up)) xout = nullptr;   // k_up2r forms the pre-smoothed iterate again
    const int ky = rows_seg(tv) / 2;
    const dim3 g = rows_grid((Lc.n + ky - 1) / ky, nsys), blk(pair_threads(Lf.n));
#define K_DR0(V, NU_, R_)                                                                                     \
  hipLaunchKernelGGL((k_down2r<T, V, NU_, R_>), g, blk,                                              \
                     row_lds_bytes<T>(k_down2r<T, V, NU_, R_>, down_words(NU_, R_), blk.x), st, Lf, Lc, b, xout, bc, shift, active, om, ctr, p, \
                     alpha, bout, partial, fin, ky)
#define K_DR(V, NU_) do { if (rup) K_DR0(V, NU_, true); else K_DR0(V, NU_, false); } while (0)
    if (var) {
      if (nu == 1) K_DR(true, 1); else if (nu == 2) K_DR(true, 2); else K_DR(true, 3);
    } else {
      if (nu == 1) K_DR(false, 1); else if (nu == 2) K_DR(false, 2); else K_DR(false, 3);
    }
#undef K_DR
#undef K_DR0
    return true;
  }
  with_tile(tv, [&](auto v) {
    constexpr int CX = kDownTile[decltype(v)::value][0], CY = kDownTile[decltype(v)::value][1];
    const dim3 g((Lc.n + CX - 1) / CX, (Lc.n + CY - 1) / CY, nsys), blk(256);
#define K_DN0(V, NU_, R_)                                                                                          \
  hipLaunchKernelGGL((k_down2<T, V, NU_, R_, CX, CY>), g, blk, 0, st, Lf, Lc, b, xout, bc, shift, active, om, ctr, \
                     p, alpha, bout, partial, fin)
#define K_DN(V, NU_) do { if (rup) K_DN0(V, NU_, true); else K_DN0(V, NU_, false); } while (0)
    if (var) {
      if (nu == 1) K_DN(true, 1); else if (nu == 2) K_DN(true, 2); else K_DN(true, 3);
    } else {
      if (nu == 1) K_DN(false, 1); else if (nu == 2) K_DN(false, 2); else K_DN(false, 3);
    }
#undef K_DN
#undef K_DN0
  });
  return true;
}

int down_blocks(int dim, int n, int tv) {
  const int nc = (n - 1) / 2;
  if (dim == 3)
    return ((nc + kD3Cx - 1) / kD3Cx) * ((nc + kD3Cy - 1) / kD3Cy) * ((nc + kD3Kz - 1) / kD3Kz);
  if (down_rows(dim, n, tv)) return (nc + rows_seg(tv) / 2 - 1) / (rows_seg(tv) / 2);
  const int cx = kDownTile[tile_variant(tv)][0], cy = kDownTile[tile_variant(tv)][1];
  return ((nc + cx - 1) / cx) * ((nc + cy - 1) / cy);
}

// The default shapes on a level of n points per axis when nsys systems share
// each launch.  The row-marching kernels (variant 3) fetch each point about
// once where the tiles fetch 1.3 - 1.8 times, but make one workgroup per
// system and segment of rows: on levels of at least kRowsMinN points per axis
// whose launches still make kFillBlocks of them they are the default (511^2,
// 2048 systems: stencil product 1286 -> 1105 us, down 1684 -> 1265, up 1351
// -> 811, the solve 107 -> 85 ms); with fewer systems (1023^2, 30 systems:
// 240 workgroups) or on small levels they are slower.  Otherwise the
// 64-column down tile (variant 0) fetches fewer halo lines but makes fewer
// workgroups than the 32 x 8 tile (variant 1): below about four per CU
// (one-system solves, coarse levels) variant 1 keeps more of the chip busy.

static inline bool rows_default(int dim, int n, long long nsys, int blocks) {
  return dim == 2 && n >= kRowsMinN && n <= kRowsMaxN && nsys * blocks >= kFillBlocks;
}

int default_down_tile(int dim, int n, long long nsys) {
  if (dim != 2) return 0;
  if (rows_default(dim, n, nsys, down_blocks(dim, n, kRowsVariant))) return kRowsVariant;
  return nsys * down_blocks(dim, n, 0) >= kFillBlocks ? 0 : 1;
}

int default_up_tile(int dim, int n, long long nsys) {
  return rows_default(dim, n, nsys, up_blocks(dim, n, kRowsVariant)) ? kRowsVariant : 0;
}

int default_spmv_tile(int dim, int n, long long nsys) {
  return rows_default(dim, n, nsys, spmv_blocks(dim, n, kRowsVariant)) ? kRowsVariant : 0;
}

template <typename T>
bool Launch<T>::fused_up(int dim, bool var, int nu, const LevelDev<T>& Lc, const LevelDev<T>& Lf, const T* xc,
                         const T* xin, const T* b, T* xout, const T* shift, const int* active, Sweeps<T> om,
                         double* partial, int nsys, hipStream_t st, unsigned long long* ctr, Fin fin, int tv) {
  const bool dot = partial != nullptr;
  if (dim == 3) {
    if (var || nu < 1 || nu > 2) return false;
    const dim3 g((Lf.n + kU3Ox - 1) / kU3Ox, ((Lf.n + kU3Oy - 1) / kU3Oy) * ((Lf.n + kU3Fz - 1) / kU3Fz), nsys);
#define K_U3(NU_, D_)                                                                                          \
  hipLaunchKernelGGL((k_up3<T, NU_, D_>), g, dim3(kF3Threads), 0, st, Lc, Lf, xc, xin, b, xout, shift, active, om, partial, \
                     ctr, fin)
    if (dot) {
      if (nu == 1) K_U3(1, true); else K_U3(2, true);
    } else {
      if (nu == 1) K_U3(1, false); else K_U3(2, false);
    }
#undef K_U3
    return true;
  }
  if (dim != 2 || nu < 1 || nu > 3) return false;
  if (up_rows(dim, Lf.n, tv)) {
    const int rows = rows_seg(tv);
    const dim3 g = rows_grid((Lf.n + rows - 1) / rows, nsys), blk(pair_threads(Lf.n));
#define K_UR0(V, NU_, D_)                                                                                        \
  hipLaunchKernelGGL((k_up2r<T, V, NU_, D_>), g, blk,                                                    \
                     row_lds_bytes<T>(k_up2r<T, V, NU_, D_>, up_words(NU_), blk.x), st, Lc, Lf, xc, xin, b, xout, shift, active, om, partial, \
                     ctr, fin, rows)
#define K_UR(V, NU_) do { if (dot) K_UR0(V, NU_, true); else K_UR0(V, NU_, false); } while (0)
    if (var) {
      if (nu == 1) K_UR(true, 1); else if (nu == 2) K_UR(true, 2); else K_UR(true, 3);
    } else {
      if (nu == 1) K_UR(false, 1); else if (nu == 2) K_UR(false, 2); else K_UR(false, 3);
    }
#undef K_UR
#undef K_UR0
    return true;
  }
  with_tile(tv, [&](auto v) {
    constexpr int OX = kUpTile[decltype(v)::value][0], OY = kUpTile[decltype(v)::value][1];
    const dim3 g((Lf.n + OX - 1) / OX, (Lf.n + OY - 1) / OY, nsys), blk(256);
#define K_UP(V, NU_, D_) \
  hipLaunchKernelGGL((k_up2<T, V, NU_, D_, OX, OY>), g, blk, 0, st, Lc, Lf, xc, xin, b, xout, shift, active, om,   \
                     partial, ctr, fin)
#define K_UPD(V, NU_) do { if (dot) K_UP(V, NU_, true); else K_UP(V, NU_, false); } while (0)
    if (var) {
      if (nu == 1) K_UPD(true, 1); else if (nu == 2) K_UPD(true, 2); else K_UPD(true, 3);
    } else {
      if (nu == 1) K_UPD(false, 1); else if (nu == 2) K_UPD(false, 2); else K_UPD(false, 3);
    }
#undef K_UPD
#undef K_UP
  });
  return true;
}

int up_blocks(int dim, int n, int tv) {
  if (dim == 3) return ((n + kU3Ox - 1) / kU3Ox) * ((n + kU3Oy - 1) / kU3Oy) * ((n + kU3Fz - 1) / kU3Fz);
  if (up_rows(dim, n, tv)) return (n + rows_seg(tv) - 1) / rows_seg(tv);
  const int ox = kUpTile[tile_variant(tv)][0], oy = kUpTile[tile_variant(tv)][1];
  return ((n + ox - 1) / ox) * ((n + oy - 1) / oy);
}

// the most blocks per system any reduction-writing launch shape can have
int max_partial_blocks(int dim, int n, long long N) {
  int m = std::max({stencil_blocks(dim, n), flat_blocks(N), residual_blocks(dim, n, 1)});
  for (int v = 0; v < kTileVariants; ++v)
    m = std::max({m, up_blocks(dim, n, v), down_blocks(dim, n, v), spmv_blocks(dim, n, v)});
  return m;
}

template struct Launch<float>;
template struct Launch<double>;

void launch_residual64(int dim, bool var, const LevelDev<double>& L, const double* f, const double* x64, float* e,
                       float* r32, const double* shift, const int* active64, double* partial, int nrhs, int nsys,
                       bool first, hipStream_t st, unsigned long long* ctr, bool zero_x) {
  if (first) {
    hipLaunchKernelGGL(k_first_residual, flat_grid(L.N, nsys), dim3(256), 0, st, L.N, f, const_cast<double*>(x64), e,
                       r32, nrhs, active64, partial, zero_x);
    return;
  }
  if (dim == 3) {
    const dim3 g = stencil_grid(dim, L.n, nsys), blk = stencil_block(dim, L.n);
    if (var)
      hipLaunchKernelGGL((k_residual64_3<true>), g, blk, 0, st, L, f, x64, e, r32, shift, active64, nrhs, partial, ctr);
    else
      hipLaunchKernelGGL((k_residual64_3<false>), g, blk, 0, st, L, f, x64, e, r32, shift, active64, nrhs, partial,
                         ctr);
  } else if (residual_rows(dim, L.n, nsys)) {
    const dim3 g = rows_grid((L.n + kRes2rRows - 1) / kRes2rRows, nsys), blk(rows_threads(L.n));
    double* x = const_cast<double*>(x64);   // not written without the update
    if (var)
      hipLaunchKernelGGL((k_residual64_2r<true, false>), g, blk, 0, st, L, f, x, e, r32, shift, active64, nrhs, partial,
                         ctr, XUpdate{});
    else
      hipLaunchKernelGGL((k_residual64_2r<false, false>), g, blk, 0, st, L, f, x, e, r32, shift, active64, nrhs,
                         partial, ctr, XUpdate{});
  } else {
    constexpr int rows_per_block = (kBlock / kRes2Cols) * kRes2Rows;
    const dim3 g2((L.n + kRes2Cols - 1) / kRes2Cols, (L.n + rows_per_block - 1) / rows_per_block, nsys);
    const dim3 b2(kRes2Cols, kBlock / kRes2Cols);
    if (var)
      hipLaunchKernelGGL((k_residual64_2<true>), g2, b2, 0, st, L, f, x64, e, r32, shift, active64, nrhs, partial, ctr);
    else
      hipLaunchKernelGGL((k_residual64_2<false>), g2, b2, 0, st, L, f, x64, e, r32, shift, active64, nrhs, partial,
                         ctr);
  }
}

void launch_residual_fp64(int dim, const LevelDev<double>& L, const double* f, const double* x, double* r,
                          const double* shift, const int* active, double* partial, int nrhs, int nsys, hipStream_t st,
                          unsigned long long* ctr) {
  float* no_e = nullptr;
  if (dim == 3) {
    hipLaunchKernelGGL((k_residual64_3<false, double>), stencil_grid(dim, L.n, nsys), stencil_block(dim, L.n), 0, st,
                       L, f, x, no_e, r, shift, active, nrhs, partial, ctr);
  } else if (residual_rows(dim, L.n, nsys)) {
    const dim3 g = rows_grid((L.n + kRes2rRows - 1) / kRes2rRows, nsys), blk(rows_threads(L.n));
    hipLaunchKernelGGL((k_residual64_2r<false, false, double>), g, blk, 0, st, L, f, const_cast<double*>(x), no_e, r,
                       shift, active, nrhs, partial, ctr, XUpdate{});
  } else {
    constexpr int rows_per_block = (kBlock / kRes2Cols) * kRes2Rows;
    const dim3 g2((L.n + kRes2Cols - 1) / kRes2Cols, (L.n + rows_per_block - 1) / rows_per_block, nsys);
    hipLaunchKernelGGL((k_residual64_2<false, double>), g2, dim3(kRes2Cols, kBlock / kRes2Cols), 0, st, L, f, x, no_e,
                       r, shift, active, nrhs, partial, ctr);
  }
}

void launch_start(int op, const double* partial, int nblk, int R, int nsys, const SysState& S, int* gate, double tol,
                  hipStream_t st, const SlotUpload* begin, int nrhs) {
  if (begin)
    hipLaunchKernelGGL(k_start<true>, dim3(nsys), dim3(256), 0, st, op, partial, nblk, R, S, gate, tol, nrhs, *begin);
  else
    hipLaunchKernelGGL(k_start<false>, dim3(nsys), dim3(256), 0, st, op, partial, nblk, R, S, gate, tol, nrhs,
                       SlotUpload{});
}

void launch_conclude(int op, const double* partial, int nblk, int nsys, const SysState& S, double tol, int max_iter,
                     const double* upartial, int unblk, int rows, double* unorm, const void* state, size_t bytes,
                     void* host, unsigned* host_seq, unsigned seq, hipStream_t st) {
  hipLaunchKernelGGL(k_conclude, dim3(1), dim3(1024), 0, st, op, partial, nblk, nsys, S, tol, max_iter, upartial,
                     unblk, rows, unorm, (const double*)state, (int)(bytes / 8), (double*)host, host_seq, seq);
}

void launch_report_flags(const int* flags, int n, int* host, unsigned* host_seq, unsigned seq, hipStream_t st) {
  hipLaunchKernelGGL(k_report_flags, dim3(1), dim3(1024), 0, st, flags, n, host, host_seq, seq);
}

bool residual_marches_rows(int dim, int n, long long nsys) { return residual_rows(dim, n, nsys); }

bool launch_update_residual64(int dim, bool var, const LevelDev<double>& L, const double* f, double* x64, float* e,
                              float* r32, const double* shift, const int* active64, double* partial, int nrhs,
                              int nsys, hipStream_t st, unsigned long long* ctr, const float* pa, const float* pb,
                              const double* alpha, const int* iters, bool assign) {
  if (!residual_rows(dim, L.n, nsys)) return false;
  const int nseg = (L.n + kRes2rRows - 1) / kRes2rRows;
  const dim3 g = rows_grid(nseg, nsys), blk(rows_threads(L.n));
  const XUpdate xu{pa, pb, alpha, iters, assign ? 1 : 0};
  if (var)
    hipLaunchKernelGGL((k_residual64_2r<true, true>), g, blk, 0, st, L, f, x64, e, r32, shift, active64, nrhs, partial,
                       ctr, xu);
  else
    hipLaunchKernelGGL((k_residual64_2r<false, true>), g, blk, 0, st, L, f, x64, e, r32, shift, active64, nrhs,
                       partial, ctr, xu);
  hipLaunchKernelGGL(k_update_seg_rows, dim3(1, 2 * nseg, nsys), blk, 0, st, L.N, L.n, x64, e, active64, xu);
  return true;
}

int residual_blocks(int dim, int n, long long nsys) {
  if (residual_rows(dim, n, nsys)) return (n + kRes2rRows - 1) / kRes2rRows;
  if (dim == 3) return stencil_blocks(dim, n);
  constexpr int rows_per_block = (kBlock / kRes2Cols) * kRes2Rows;
  return ((n + kRes2Cols - 1) / kRes2Cols) * ((n + rows_per_block - 1) / rows_per_block);
}

void launch_x_from_e(const LevelDev<double>& L, int dim, const float* e, double* x64, const int* active64, int nsys,
                     hipStream_t st, const float* pa, const float* pb, const double* alpha, const int* iters) {
  (void)dim;
  hipLaunchKernelGGL(k_x_from_e, flat_grid(L.N, nsys), dim3(256), 0, st, L.N, e, x64, active64, pa, pb, alpha,
                     iters);
}

void launch_combine(long long N, const double* x, const double* w, const CombineTerms& t, int nout, int nrhs,
                    int stride, double* u, hipStream_t st, unsigned long long* ctr, const double* base, double base_w,
                    bool w_per_system, const double* pa, const double* pb, const double* alpha, const int* iters,
                    double* partial, double* norms) {
  const int nb = combine_blocks(N);
  hipLaunchKernelGGL(k_combine, dim3((unsigned)nb, nrhs, nout), dim3(256), 0, st, N, x, w, t, stride, u, base, base_w,
                     ctr, w_per_system ? 1 : 0, pa, pb, alpha, iters, partial);
  if (partial && norms) launch_row_sum(partial, nb, nout * nrhs, norms, st);
}

void launch_row_sum(const double* partial, int nblk, int rows, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_row_sum, dim3(rows), dim3(nblk > 256 ? 1024 : 256), 0, st, partial, nblk, out);
}

int combine_blocks(long long N) { return (int)((N + 256 * kCombineItems - 1) / (256 * kCombineItems)); }

void launch_apply64(int dim, bool var, const LevelDev<double>& L, const double* x, double* y, double shift, int nvec,
                    hipStream_t st) {
  const dim3 g = point_grid(dim, L.n, nvec), blk(kTileX, kTileY);
#define K_AP(D, V, dummy) hipLaunchKernelGGL((k_apply64<D, V>), g, blk, 0, st, L, x, y, shift)
  BURA_DISPATCH_DV(dim, var, K_AP, 0);
#undef K_AP
}

void launch_scalars(int op, const double* partial, int nblk, int nsys, SysState S, double tol, int max_iter,
                    hipStream_t st, const Progress& pr) {
  hipLaunchKernelGGL(k_scalars, dim3(nsys), dim3(256), 0, st, op, partial, nblk, S, tol, max_iter, pr);
}

// Terms of one right-hand-side slot of a slot plan (systems j R + slot,
// j < K): weights, shifts (FP64 and FP32), tolerances; resets the systems'
// counters and marks the used ones (j < nterms) in init.
__global__ void k_slot_terms(SlotTermsDev v, double* __restrict__ w, double* __restrict__ s64,
                             float* __restrict__ s32, double* __restrict__ tol, int* __restrict__ init,
                             int* __restrict__ total_iters, int* __restrict__ outer, int* __restrict__ flags,
                             int* __restrict__ active, int* __restrict__ active64) {
  const int j = threadIdx.x;
  if (j >= v.K) return;
  const long long sys = (long long)j * v.R + v.slot;
  const bool used = j < v.nterms;
  w[sys] = used ? v.w[j] : 0.0;
  s64[sys] = used ? v.s[j] : 0.0;
  if (s32) s32[sys] = used ? (float)v.s[j] : 0.0f;
  tol[sys] = v.tol;
  init[sys] = used ? 1 : 0;
  total_iters[sys] = 0;
  outer[sys] = 0;
  flags[sys] = 0;
  active[sys] = 0;
  active64[sys] = 0;
}

// active64 of the systems just initialised (their outer test ran on init)
__global__ void k_merge_init(int* __restrict__ init, int* __restrict__ active64, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (init[i]) {
    active64[i] = init[i];
    init[i] = 0;
  }
}

void launch_slot_terms(const SlotTermsDev& v, double* w, double* s64, float* s32, double* tol, int* init,
                       int* total_iters, int* outer, int* flags, int* active, int* active64, hipStream_t st) {
  hipLaunchKernelGGL(k_slot_terms, dim3(1), dim3(64), 0, st, v, w, s64, s32, tol, init, total_iters, outer, flags,
                     active, active64);
}

void launch_merge_init(int* init, int* active64, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_merge_init, dim3((n + 255) / 256), dim3(256), 0, st, init, active64, n);
}

__global__ void k_fill_int(int* __restrict__ p, long long n, int v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ __launch_bounds__(256) void k_begin(SysState S, int nsys, int R, int nrhs, SlotUpload up) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nsys) begin_system(S, i, nsys, R, nrhs, up);
}

void launch_begin(const SysState& S, int nsys, int R, int nrhs, const SlotUpload& up, hipStream_t st) {
  hipLaunchKernelGGL(k_begin, dim3((nsys + 255) / 256), dim3(256), 0, st, S, nsys, R, nrhs, up);
}

void launch_fill_int(int* p, long long n, int v, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_int, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
}

// Fill with zero bytes: 16-byte stores over the 16-byte-aligned body, single
// bytes for the unaligned head and tail.
__global__ void k_zero(unsigned char* p, size_t bytes) {
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t head = std::min<size_t>((16 - ((uintptr_t)p & 15)) & 15, bytes);
  const size_t words = (bytes - head) / 16;
  uint4* body = (uint4*)(p + head);
  for (size_t i = tid; i < words; i += stride) body[i] = make_uint4(0u, 0u, 0u, 0u);
  const size_t tail0 = head + words * 16;
  for (size_t i = tid; i < head + (bytes - tail0); i += stride) p[i < head ? i : tail0 + (i - head)] = 0;
}

// One read and one write of every byte: 16-byte vector accesses over the body,
// grid-stride over 2048 workgroups x 256 threads (8 per CU), bytes for the tail.
// One 16-byte word per thread and no loop: every wave has its load in flight
// at once.  On 2 GiB this reaches 6.1 TB/s; a grid-stride loop over 2048
// workgroups reached 4.7 TB/s (each wave then waits for one load at a time).
__global__ __launch_bounds__(256) void k_stream_copy(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                     size_t words, unsigned char* __restrict__ dtail,
                                                     const unsigned char* __restrict__ stail, int tail) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) dst[i] = src[i];
  if (i < (size_t)tail) dtail[i] = stail[i];
}

void launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
  if (bytes == 0) return;
  const size_t words = bytes / 16;
  const int tail = (int)(bytes - words * 16);
  const size_t blocks = std::max<size_t>(1, (words + 255) / 256);
  hipLaunchKernelGGL(k_stream_copy, dim3((unsigned)blocks), dim3(256), 0, st, (uint4*)dst, (const uint4*)src, words,
                     (unsigned char*)dst + words * 16, (const unsigned char*)src + words * 16, tail);
}

void launch_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return;
  const size_t blocks = std::min<size_t>((bytes + 255) / 256, 4096);
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, st, (unsigned char*)p, bytes);
}

}  // namespace bura
