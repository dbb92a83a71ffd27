// Direct solution of the constant-coefficient shifted systems in the sine
// basis, on the FP64 matrix cores (gfx950).
//
// On the unit square / cube with constant coefficients the scaled operator is
// diagonal in the orthonormal sine basis S (S = S^T = S^-1 per axis, the
// closed form the method's own experiments start from, Sections 5.1 and 5.3):
// (A + s I)^-1 f = S (Lambda + s)^-1 S f, S applied along every axis.  An
// application of S along one axis is a matrix product, so the whole solve of a
// shifted system is dim products forward (shared by every pole of a right-hand
// side) and dim products back.  The result is the starting iterate of the
// solve: its FP64 residual f - (A + s) x is formed and tested like that of any
// other iterate, and a system over its tolerance goes on into the multigrid
// solver from there.
//
// The basis vectors are even or odd about the middle of the axis, so a
// transform of n values splits into two of n/2: forward, the sums u_j +
// u_{n+1-j} give the odd-numbered coefficients and the differences the even
// ones; back, the two halves a_j, b_j give u_j = a_j + b_j and u_{n+1-j} =
// a_j - b_j.  That halves the products (n^2 instead of 2 n^2 flops per line).
// Coefficients are kept in the split order (odd ones first) throughout.
#include "bura_internal.h"

#include <algorithm>

namespace bura {

namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kSineThreads = 256;   // four waves, 2 x 2 over the tile
constexpr int kSineK = 16;          // transformed-axis values staged per step

// One transform along one axis of a batch of grids.
struct SinePass {
  const double* in;
  double* out;
  const double* t0;      // matrix of the first half, [k][m], hp x hp, zero padded
  const double* t1;      // of the second half
  int n, h1, h0, hp;     // points per axis, length of the halves ((n+1)/2, n/2), padded length
  int tiles_m, tiles_c;  // tiles along the outputs of the axis and across the lines
  long long groups;      // batches * tiles_c
  long long in_stride, out_stride;   // elements between two batches
  long long ld;          // lines along columns: elements between neighbours on the axis
  long long lines;       // lines per batch
  int planes;            // batches per system
  int rhs_of;            // > 0: the input of system s is right-hand side s % rhs_of
  const int* gate;       // per system: 0 skip, 1 transform, 2 write zeros in the last pass; nullptr: 1
  int zero;              // the last pass
  const double* mu;      // eigenvalues of the 1D second difference in the split order
  int axes;              // axes across the lines of the scaled pass (1 in 2D, 2 in 3D)
  double wc;             // face weight of the scaled operator
  const double* shift;
  double* partial;       // forward row pass: |in|^2 per (batch, row tile)
  unsigned long long* ctr;
};

// 1/d to rounding: the hardware estimate and two Newton steps r (2 - d r).
// (An IEEE division per scaled value would cost as much as the products of a
// 64-wide tile; this is 5 instructions.)
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return r;
}

// D = M x lines for a tile of TM outputs x TM lines of both halves.
//
// ROW: the lines are rows (the axis is contiguous): D rows are lines, D columns
//   outputs; otherwise the lines are columns and D columns are lines.  Either
//   way the D columns are contiguous in memory (stores of 128 bytes).
// INV: coefficients to values, else values to coefficients.
// SCALE (inverse, columns): the coefficients are divided by the eigenvalue of
//   the system as they are staged.
//
// Bound by the FP64 matrix rate (n/2 flops per byte and pass): a wave owns
// 16 WT x 16 WT outputs of both halves in registers (v_mfma_f64_16x16x4) and
// reads WT + WT values per half and step of 4, so LDS moves an eighth of what
// it could; the next kSineK values are loaded into registers while the current
// ones are multiplied.  WT = 2 (64 x 64 tiles); WT = 1 (32 x 32) where 64 x 64
// tiles would leave CUs idle.  The sum over the axis runs in the same order in
// both, so a result does not depend on the tile.
template <bool ROW, bool INV, bool SCALE, int WT>
__global__ __launch_bounds__(kSineThreads) void k_sine(SinePass a) {
  constexpr int TM = 32 * WT, KC = kSineK;
  // rows of the staged matrix are 128 bytes off a multiple of the 256 bytes of
  // a bank cycle, so the four k of a step sit on different banks
  constexpr int LM = TM + 16, LR = KC + 1;
  constexpr int ND = TM * KC / kSineThreads;
  __shared__ double sm[2][KC * LM];
  __shared__ double sd[2][ROW ? TM * LR : KC * LM];
  // the output tiles of one set of lines go to one XCD (workgroups are dealt
  // to the 8 XCDs round-robin), whose L2 then serves the lines again
  const long long id = blockIdx.x;
  const long long q = id >> 3;
  const int mt = (int)(q % a.tiles_m);
  const long long grp = (q / a.tiles_m) * 8 + (id & 7);
  if (grp >= a.groups) return;
  const long long batch = grp / a.tiles_c;
  const int ct = (int)(grp - batch * a.tiles_c);
  const int sys = (int)(batch / a.planes);
  const int g = a.gate ? a.gate[sys] : 1;
  if (g == 0 || (g == 2 && !a.zero)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  const int m0 = mt * TM;
  const long long c0 = (long long)ct * TM;
  const long long ib = a.rhs_of > 0 ? (long long)(sys % a.rhs_of) : batch;
  const double* __restrict__ in = a.in + ib * a.in_stride;
  double* __restrict__ out = a.out + batch * a.out_stride;
  const int n = a.n, h1 = a.h1, h0 = a.h0;
  if (a.ctr && mt == 0 && tid == 0) {
    const long long ln = min((long long)TM, a.lines - c0);
    atomicAdd(a.ctr, (unsigned long long)(2 * ln * n) * 8ULL);
  }

  double4_t acc[2][WT][WT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int x = 0; x < WT; ++x)
#pragma unroll
      for (int y = 0; y < WT; ++y) acc[h][x][y] = (double4_t){0.0, 0.0, 0.0, 0.0};
  double ssq = 0.0;
  // the eigenvalue share of a column's other axes and the shift (the column of
  // a thread's staged values is the same in every step)
  double muc = 0.0;
  if (SCALE) {
    const long long c = min(c0 + (long long)(tid % TM), a.lines - 1);
    muc = a.axes == 1 ? a.mu[c] : a.mu[c / n] + a.mu[c % n];
    muc = a.wc * muc + a.shift[sys];
  }

  double d0[ND], d1[ND], q0[ND], q1[ND];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < ND; ++u) {
      const int idx = tid + kSineThreads * u;
      const int kk = k0 + (ROW ? idx % KC : idx / TM);
      const long long c = c0 + (ROW ? idx / KC : idx % TM);
      const bool on = c < a.lines;
      const int p0 = kk, p1 = INV ? h1 + kk : n - 1 - kk;
      const bool on0 = on && kk < h1, on1 = on && kk < h0;
      d0[u] = 0.0;
      d1[u] = 0.0;
      if (ROW) {
        if (on0) d0[u] = in[c * n + p0];
        if (on1) d1[u] = in[c * n + p1];
      } else {
        if (on0) d0[u] = in[(long long)p0 * a.ld + c];
        if (on1) d1[u] = in[(long long)p1 * a.ld + c];
      }
      const int mk = k0 + idx / TM, mm = m0 + idx % TM;
      q0[u] = a.t0[(long long)mk * a.hp + mm];
      q1[u] = a.t1[(long long)mk * a.hp + mm];
    }
  };
  auto stage = [&](int k0) {
#pragma unroll
    for (int u = 0; u < ND; ++u) {
      const int idx = tid + kSineThreads * u;
      const int kk = ROW ? idx % KC : idx / TM;
      const int cc = ROW ? idx / KC : idx % TM;
      double v0 = d0[u], v1 = d1[u];
      if (!INV) {
        if (ROW && a.partial) ssq += v0 * v0 + v1 * v1;
        // the middle value of an odd n has no partner: v1 = 0 there, and the
        // second half has no such input
        const double e = v0 + v1;
        v1 = k0 + kk < h0 ? v0 - v1 : 0.0;
        v0 = e;
      }
      if (SCALE) {
        if (k0 + kk < h1) v0 *= recip(fma(a.wc, a.mu[k0 + kk], muc));
        if (k0 + kk < h0) v1 *= recip(fma(a.wc, a.mu[h1 + k0 + kk], muc));
      }
      const int at = ROW ? cc * LR + kk : kk * LM + cc;
      sd[0][at] = v0;
      sd[1][at] = v1;
      const int mat = (idx / TM) * LM + idx % TM;
      sm[0][mat] = q0[u];
      sm[1][mat] = q1[u];
    }
  };
  // waves 2 x 2: ri D rows, rj D columns of this wave within the tile
  const int ri = (wave >> 1) * 16 * WT, rj = (wave & 1) * 16 * WT;
  const int nk = g == 1 ? (h1 + KC - 1) / KC : 0;
  // back, the sums start at the highest coefficients: a solution is dominated by
  // its lowest ones, and each step rounds relative to the sum so far
  auto at = [&](int t) { return (INV ? nk - 1 - t : t) * KC; };
  if (nk > 0) load(at(0));
  for (int t = 0; t < nk; ++t) {
    if (t) __syncthreads();   // every read of the previous values is done
    stage(at(t));
    __syncthreads();
    if (t + 1 < nk) load(at(t + 1));
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int kr = 4 * (INV ? KC / 4 - 1 - s : s) + lk;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        double av[WT], bv[WT];
#pragma unroll
        for (int x = 0; x < WT; ++x) {
          av[x] = ROW ? sd[h][(ri + 16 * x + l16) * LR + kr] : sm[h][kr * LM + ri + 16 * x + l16];
          bv[x] = ROW ? sm[h][kr * LM + rj + 16 * x + l16] : sd[h][kr * LM + rj + 16 * x + l16];
        }
#pragma unroll
        for (int x = 0; x < WT; ++x)
#pragma unroll
          for (int y = 0; y < WT; ++y)
            acc[h][x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[x], bv[y], acc[h][x][y], 0, 0, 0);
      }
    }
  }
  // element v of a lane: D row 4 v + lane / 16, D column lane % 16
#pragma unroll
  for (int x = 0; x < WT; ++x)
#pragma unroll
    for (int y = 0; y < WT; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int dr = ri + 16 * x + 4 * v + lk, dc = rj + 16 * y + l16;
        const int m = m0 + (ROW ? dc : dr);
        const long long c = c0 + (ROW ? dr : dc);
        if (c >= a.lines) continue;
        const double p = acc[0][x][y][v], r = acc[1][x][y][v];
        auto put = [&](int pos, double val) {
          if (ROW) out[c * n + pos] = val;
          else out[(long long)pos * a.ld + c] = val;
        };
        if (!INV) {
          if (m < h1) put(m, p);
          if (m < h0) put(h1 + m, r);
        } else if (m < h0) {
          put(m, p + r);
          put(n - 1 - m, p - r);
        } else if (m < h1) {
          put(m, p);
        }
      }
  if (ROW && !INV && a.partial && mt == 0) {
    // fixed-order block sum of the squares
    __shared__ double sh[kSineThreads / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ssq += __shfl_xor(ssq, o, 64);
    if (lane == 0) sh[wave] = ssq;
    __syncthreads();
    if (tid == 0) a.partial[grp] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  }
}

// The matrices of the four half transforms and the 1D eigenvalues.
__global__ __launch_bounds__(256) void k_sine_tables(int n, int h1, int h0, int hp, double* tab, double* mu) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long hh = (long long)hp * hp;
  if (idx < hh) {
    const int r = (int)(idx / hp), c = (int)(idx % hp);
    const double sc = sqrt(2.0 / (n + 1));
    const long long N2 = 2LL * (n + 1);
    // sqrt(2/(n+1)) sin(pi j k / (n+1)) for value j and coefficient k (1-based)
    auto S = [&](long long j, long long k) { return sc * sinpi((double)((j * k) % N2) / (n + 1)); };
    tab[idx] = r < h1 && c < h1 ? S(r + 1, 2 * c + 1) : 0.0;            // forward, first half: [value][coefficient]
    tab[hh + idx] = r < h0 && c < h0 ? S(r + 1, 2 * c + 2) : 0.0;
    tab[2 * hh + idx] = r < h1 && c < h1 ? S(c + 1, 2 * r + 1) : 0.0;   // back: [coefficient][value]
    tab[3 * hh + idx] = r < h0 && c < h0 ? S(c + 1, 2 * r + 2) : 0.0;
  }
  if (idx < n) {
    const long long k = idx < h1 ? 2 * idx + 1 : 2 * (idx - h1) + 2;
    const double sn = sinpi((double)k / (2.0 * (n + 1)));
    mu[idx] = 4.0 * sn * sn;
  }
}

template <bool ROW, bool INV, bool SCALE>
void run_pass(SinePass a, long long batches, hipStream_t st) {
  // 64 x 64 tiles where they make two workgroups per CU, else 32 x 32 (as
  // many as four times the workgroups: small grids are bound by the latency of
  // one workgroup's chain, not by the matrix rate)
  auto grid = [&](int tm) {
    a.tiles_m = (a.h1 + tm - 1) / tm;
    a.tiles_c = (int)((a.lines + tm - 1) / tm);
    a.groups = batches * a.tiles_c;
    return (unsigned)(((a.groups + 7) / 8) * 8 * a.tiles_m);
  };
  const unsigned big = grid(64);
  if (big >= 512u) {
    hipLaunchKernelGGL((k_sine<ROW, INV, SCALE, 2>), dim3(big), dim3(kSineThreads), 0, st, a);
  } else {
    const unsigned small = grid(32);
    hipLaunchKernelGGL((k_sine<ROW, INV, SCALE, 1>), dim3(small), dim3(kSineThreads), 0, st, a);
  }
}

}  // namespace

int sine_half(int n) { return (((n + 1) / 2) + 63) / 64 * 64; }

size_t sine_table_doubles(int n) { return 4 * (size_t)sine_half(n) * sine_half(n) + (size_t)n; }

void launch_sine_tables(int n, double* tab, hipStream_t st) {
  const int hp = sine_half(n);
  const long long hh = (long long)hp * hp;
  hipLaunchKernelGGL(k_sine_tables, dim3((unsigned)((std::max<long long>(hh, n) + 255) / 256)), dim3(256), 0, st, n,
                     (n + 1) / 2, n / 2, hp, tab, tab + 4 * hh);
}

int sine_norm_blocks(int dim, int n, int nrhs) {
  const long long rows = dim == 3 ? (long long)n * n : n;
  const int hp = (n + 1) / 2;
  const long long t64 = (rows + 63) / 64;
  const long long big = ((nrhs * t64 + 7) / 8) * 8 * ((hp + 63) / 64);
  return (int)(big >= 512 ? t64 : (rows + 31) / 32);
}

void launch_sine_forward(const SineSolve& s, hipStream_t st, unsigned long long* ctr, double* partial) {
  const int n = s.n, hp = sine_half(n);
  const size_t hh = (size_t)hp * hp;
  const long long nn = (long long)n * n, N = s.dim == 3 ? nn * n : nn;
  SinePass a{};
  a.n = n;
  a.h1 = (n + 1) / 2;
  a.h0 = n / 2;
  a.hp = hp;
  a.planes = 1;
  a.t0 = s.tab;
  a.t1 = s.tab + hh;
  a.ctr = ctr;
  a.ld = n;
  // x: f -> work
  a.in = s.f;
  a.out = s.work;
  a.in_stride = a.out_stride = N;
  a.lines = N / n;
  a.partial = partial;
  run_pass<true, false, false>(a, s.nrhs, st);
  a.partial = nullptr;
  // y: work -> x
  a.in = s.work;
  a.out = s.x;
  a.lines = n;
  a.in_stride = a.out_stride = nn;
  run_pass<false, false, false>(a, s.dim == 3 ? (long long)s.nrhs * n : s.nrhs, st);
  if (s.dim == 3) {
    // z: x -> work
    a.in = s.x;
    a.out = s.work;
    a.ld = nn;
    a.lines = nn;
    a.in_stride = a.out_stride = N;
    run_pass<false, false, false>(a, s.nrhs, st);
  }
}

void launch_sine_back(const SineSolve& s, hipStream_t st, unsigned long long* ctr) {
  const int n = s.n, hp = sine_half(n);
  const size_t hh = (size_t)hp * hp;
  const long long nn = (long long)n * n, N = s.dim == 3 ? nn * n : nn;
  SinePass a{};
  a.n = n;
  a.h1 = (n + 1) / 2;
  a.h0 = n / 2;
  a.hp = hp;
  a.planes = 1;
  a.t0 = s.tab + 2 * hh;
  a.t1 = s.tab + 3 * hh;
  a.mu = s.tab + 4 * hh;
  a.axes = s.dim - 1;
  a.wc = s.wc;
  a.shift = s.shift;
  a.gate = s.gate;
  a.ctr = ctr;
  // the slowest axis, with the division by the eigenvalues: one right-hand
  // side's coefficients to every system of it
  a.rhs_of = s.stride;
  a.in = s.dim == 3 ? s.work : s.x;
  a.out = s.dim == 3 ? s.x : s.work;
  a.ld = s.dim == 3 ? nn : n;
  a.lines = s.dim == 3 ? nn : n;
  a.in_stride = a.out_stride = N;
  run_pass<false, true, true>(a, s.nsys, st);
  a.rhs_of = 0;
  if (s.dim == 3) {
    // y, plane by plane: x -> work
    a.in = s.x;
    a.out = s.work;
    a.ld = n;
    a.lines = n;
    a.planes = n;
    a.in_stride = a.out_stride = nn;
    run_pass<false, true, false>(a, (long long)s.nsys * n, st);
    a.planes = 1;
  }
  // x: work -> x
  a.in = s.work;
  a.out = s.x;
  a.ld = n;
  a.lines = N / n;
  a.in_stride = a.out_stride = N;
  a.zero = 1;
  run_pass<true, true, false>(a, s.nsys, st);
}

}  // namespace bura
