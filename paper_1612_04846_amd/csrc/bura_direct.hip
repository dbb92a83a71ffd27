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
constexpr int kFftMin = 64;         // smallest n + 1 = 2^p that runs as fast Fourier transforms

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

// --------------------------------------------------------------------------
// n + 1 = 2^p: the same transform by fast Fourier transforms
//
// Two lines a, b are one complex sequence z = a + i b, extended to length
// L = 2 (n + 1) as an odd sequence; its Fourier transform is Z_k = 2 S b_k -
// 2 i S a_k.  That is twice the arithmetic of a transform that used the odd
// symmetry, but the pass stays bound by its two memory passes (16 bytes a
// value): 5 L log2 L flops per two lines against the n^2 / 2 of the products.
//
// A thread holds 16 complex values: radix-16 steps, the last one L / 256 (L /
// 16 for L = 128), in the self-sorting order, the values exchanged through LDS
// between steps, real parts first and then imaginary parts (half the LDS of
// complex values, so two workgroups of 512 threads fit a CU).
//
// What bounds it is the latency of those steps: at 1023^2 and 30 systems the
// arithmetic alone is about 50 us a pass and the traffic 50 (the scaled pass,
// which only writes) or 100.  With every value loaded and scaled at both of its
// places and 130 - 177 registers (2 - 3 waves per SIMD) the passes took 245 and
// 140 us; one load per value, LDS positions that are constants away from one
// register and twiddle powers formed in pairs leave 98 - 116 registers, 4 waves,
// and 121 - 142, by the card, and 110 us (255^3, 9 systems: 1030, 717 and 660
// -> 803, 527 and 467).
// --------------------------------------------------------------------------
struct FftPass {
  const double* in;
  double* out;
  const double2* tw;     // exp(-2 pi i m / L), m < L
  int n;
  int tiles;             // workgroups across the lines of a batch
  long long groups;      // batches * tiles
  long long per;         // groups per XCD
  long long in_stride, out_stride, ld, lines;
  int planes, rhs_of;
  int by_tile;           // scaled passes: the systems of a tile side by side
  const int* gate;
  int zero;
  const double* mu;      // 1D eigenvalues in the split order of the products
  int axes;
  double wc;
  const double* shift;
  double* partial;
  unsigned long long* ctr;
};

// two neighbouring values of an odd row length: 8-byte aligned
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

struct cplx {
  double x, y;
};
__device__ __forceinline__ cplx operator+(cplx a, cplx b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx operator-(cplx a, cplx b) { return {a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cplx operator*(cplx a, cplx b) {
  return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ cplx mul_mi(cplx a) { return {a.y, -a.x}; }   // -i a

// Fourier transforms of R values, v[s], v[s + d], v[s + 2 d], ..., in place and
// in order
template <int R>
__device__ __forceinline__ void dft(cplx* v, int s, int d) {
  if constexpr (R == 2) {
    const cplx a = v[s], b = v[s + d];
    v[s] = a + b;
    v[s + d] = a - b;
  } else if constexpr (R == 4) {
    const cplx a = v[s] + v[s + 2 * d], b = v[s] - v[s + 2 * d];
    const cplx c = v[s + d] + v[s + 3 * d], e = mul_mi(v[s + d] - v[s + 3 * d]);
    v[s] = a + c;
    v[s + d] = b + e;
    v[s + 2 * d] = a - c;
    v[s + 3 * d] = b - e;
  } else if constexpr (R == 8) {
    const double h = 0.70710678118654752440;
    dft<4>(v, s, 2 * d);       // even positions
    dft<4>(v, s + d, 2 * d);   // odd positions
    cplx o1 = v[s + 3 * d], o2 = v[s + 5 * d], o3 = v[s + 7 * d];
    o1 = {h * (o1.x + o1.y), h * (o1.y - o1.x)};
    o2 = mul_mi(o2);
    o3 = {h * (o3.y - o3.x), -h * (o3.x + o3.y)};
    const cplx e0 = v[s], e1 = v[s + 2 * d], e2 = v[s + 4 * d], e3 = v[s + 6 * d], o0 = v[s + d];
    v[s] = e0 + o0;
    v[s + d] = e1 + o1;
    v[s + 2 * d] = e2 + o2;
    v[s + 3 * d] = e3 + o3;
    v[s + 4 * d] = e0 - o0;
    v[s + 5 * d] = e1 - o1;
    v[s + 6 * d] = e2 - o2;
    v[s + 7 * d] = e3 - o3;
  } else if constexpr (R == 16) {
    const double c1 = 0.92387953251128675613, s1 = 0.38268343236508977173, h = 0.70710678118654752440;
#pragma unroll
    for (int q = 0; q < 4; ++q) dft<4>(v, s + q * d, 4 * d);
    // v[q + 4 k] is coefficient k of column q: times exp(-2 pi i q k / 16)
    auto tw = [&](int q, int k, double cr, double ci) {
      cplx& a = v[s + (q + 4 * k) * d];
      a = a * cplx{cr, ci};
    };
    tw(1, 1, c1, -s1);
    tw(1, 2, h, -h);
    tw(1, 3, s1, -c1);
    tw(2, 1, h, -h);
    v[s + 10 * d] = mul_mi(v[s + 10 * d]);
    tw(2, 3, -h, -h);
    tw(3, 1, s1, -c1);
    tw(3, 2, -h, -h);
    tw(3, 3, -c1, s1);
#pragma unroll
    for (int k = 0; k < 4; ++k) dft<4>(v, s + 4 * k * d, d);
    // v[4 k + m] is coefficient k + 4 m: transpose
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int m = k + 1; m < 4; ++m) {
        const cplx a = v[s + (4 * k + m) * d];
        v[s + (4 * k + m) * d] = v[s + (4 * m + k) * d];
        v[s + (4 * m + k) * d] = a;
      }
  }
}

// w^1, w^2, w^4, w^8 (as far as R needs them) for the twiddles w^i, i < R, of
// table step m
template <int R>
struct Twiddle {
  cplx w[4];
  __device__ __forceinline__ void load(const double2* __restrict__ tw, int m, int mask) {
#pragma unroll
    for (int b = 0; (1 << b) < R; ++b) {
      const double2 a = tw[(m << b) & mask];
      w[b] = {a.x, a.y};
    }
  }
  // v[s + i d] *= w^i (at most three roundings; w^i and w^{i + 8} together, so
  // that few powers are held at a time)
  __device__ __forceinline__ void apply(cplx* v, int s, int d) const {
    auto at = [&](int i, cplx p) {
      if (i < R) v[s + i * d] = v[s + i * d] * p;
      if (i + 8 < R) v[s + (i + 8) * d] = v[s + (i + 8) * d] * (w[3] * p);
    };
    at(1, w[0]);
    if constexpr (R > 2) {
      at(2, w[1]);
      const cplx w3 = w[1] * w[0];
      at(3, w3);
      if constexpr (R > 4) {
        at(4, w[2]);
        at(5, w[2] * w[0]);
        at(6, w[2] * w[1]);
        at(7, w[2] * w3);
      }
      if constexpr (R > 8) v[s + 8 * d] = v[s + 8 * d] * w[3];
    }
  }
};

// Workgroup shape: T = L/16 threads per pair of lines.  Rows: 256 threads (at
// least one pair).  Columns: pairs side by side so that a row of the tile is
// 128 bytes (64 at L = 2048, 32 at 4096, where LDS holds no more).
template <int LOG>
constexpr int fft_pairs(bool row) {
  constexpr int T = (1 << LOG) / 16;
  return row ? (T >= 256 ? 1 : 256 / T) : (LOG <= 8 ? 16 : LOG <= 10 ? 8 : LOG == 11 ? 4 : 2);
}

template <int LOG, bool ROW, bool SCALE>
__global__ __launch_bounds__((1 << LOG) / 16 * fft_pairs<LOG>(ROW)) __attribute__((amdgpu_waves_per_eu(4))) void
k_sine_fft(FftPass a) {
  constexpr int L = 1 << LOG, N = L / 2, T = L / 16, P = fft_pairs<LOG>(ROW);
  constexpr int RL = LOG == 7 ? 8 : (L / 256);   // the last step's radix (1: there is none)
  constexpr int LP = L + L / 16;   // a line of padded positions (see below)
  __shared__ double sh[LP * P];
  const long long id = blockIdx.x;
  // neighbouring tiles on one XCD: a tile row of columns may be half a line
  const long long grp = (id & 7) * a.per + (id >> 3);
  if (grp >= a.groups) return;
  const long long nb = a.groups / a.tiles;
  const long long batch = SCALE && a.by_tile ? grp % nb : grp / a.tiles;
  const int tile = (int)(SCALE && a.by_tile ? grp / nb : grp - batch * a.tiles);
  const int sys = (int)(batch / a.planes);
  const int g = a.gate ? a.gate[sys] : 1;
  if (g == 0 || (g == 2 && !a.zero)) return;
  const int tid = threadIdx.x;
  const int pair = ROW ? tid / T : tid % P, t = ROW ? tid % T : tid / P;
  const long long l0 = ((long long)tile * P + pair) * 2;   // lines l0 and l0 + 1
  const bool on0 = l0 < a.lines, on1 = l0 + 1 < a.lines;
  const long long ib = a.rhs_of > 0 ? (long long)(sys % a.rhs_of) : batch;
  const double* __restrict__ in = a.in + ib * a.in_stride;
  double* __restrict__ out = a.out + batch * a.out_stride;
  const int n = a.n;
  if (a.ctr && tid == 0) {
    const long long ln = min((long long)2 * P, a.lines - (long long)tile * P * 2);
    atomicAdd(a.ctr, (unsigned long long)(2 * ln * n) * 8ULL);
  }
  // value j (1-based) of a line
  auto addr = [&](int j, long long l) { return ROW ? l * n + (j - 1) : (long long)(j - 1) * a.ld + l; };
  if (g == 2) {
    for (int j = t; j < N; j += T) {
      if (j >= 1 && on0) out[addr(j, l0)] = 0.0;
      if (j >= 1 && on1) out[addr(j, l0 + 1)] = 0.0;
    }
    return;
  }
  double mu0 = 0.0, mu1 = 0.0;
  if (SCALE) {
    // the split order of the eigenvalue table: odd numbers first
    auto mu_at = [&](long long k) { return a.mu[(k & 1) ? (k - 1) / 2 : N / 2 + k / 2 - 1]; };
    auto across = [&](long long l) {
      l = min(l, a.lines - 1);
      return a.axes == 1 ? mu_at(l + 1) : mu_at(l / n + 1) + mu_at(l % n + 1);
    };
    mu0 = fma(a.wc, across(l0), a.shift[sys]);
    mu1 = fma(a.wc, across(l0 + 1), a.shift[sys]);
  }
  // The odd extension z_j = x_j, z_{L-j} = -x_j, 0 at 0 and N: this thread's
  // values t + i T.  The first half (i < 8) is loaded; the second half is the
  // first half of other threads, mirrored, and comes through LDS (loaded and
  // scaled twice, a scaled pass took 1.7 times as long).  Loads are clamped to
  // a line and a value that exist (a last line without a partner takes the one
  // before it along): what is not on the grid is 0 at value 0, and is not
  // stored otherwise.
  cplx v[16];
  const long long step = ROW ? 1 : a.ld;
  const double* __restrict__ p0;
  const double* __restrict__ p1;
  {
    const long long c0 = min(l0, a.lines - 1), c1 = min(l0 + 1, a.lines - 1);
    const long long q = (long long)(t - 1) * step;   // value t (value 0: see below)
    p0 = in + (ROW ? c0 * n : (on1 ? c0 : c1 - 1)) + q;
    p1 = in + (ROW ? c1 * n : 0) + q;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const long long o = i == 0 && t == 0 ? step : (long long)i * T * step;
    if (ROW) {
      v[i] = {p0[o], p1[o]};
    } else {
      const f64x2u w = *reinterpret_cast<const f64x2u*>(p0 + o);
      v[i] = {on1 ? w[0] : w[1], w[1]};
    }
    if (i == 0 && t == 0) v[i] = {0.0, 0.0};
  }
  // the workgroup's sum of squares, in fixed order (before the transform, so
  // that nothing of it stays in registers)
  constexpr int NW = (T * P + 63) / 64;
  __shared__ double sw[NW];
  if (ROW && !SCALE) {
    double ssq = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) ssq += (on0 ? v[i].x * v[i].x : 0.0) + (on1 ? v[i].y * v[i].y : 0.0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ssq += __shfl_xor(ssq, o, 64);
    if ((tid & 63) == 0) sw[tid >> 6] = ssq;
  }
  if (SCALE) {
    // value j = t + i T has the parity of t (T is even)
    const double* __restrict__ pm = a.mu + ((t & 1) ? (t - 1) / 2 : N / 2 + t / 2 - 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const double m = pm[i * (T / 2)];
      v[i].x *= recip(fma(a.wc, m, mu0));
      v[i].y *= recip(fma(a.wc, m, mu1));
      // (all the reciprocals at once do not fit the registers of 4 waves)
      if (i & 1) __builtin_amdgcn_sched_barrier(0);
    }
  }
  // Value q of a pair is at position q + q / 16 of its line in LDS: the strided
  // accesses of a step fall in different banks, and every access of a thread
  // is a constant away from one position (all the constants here are
  // multiples of 16 or below the next one), so that few registers hold
  // addresses.  C: what a position of a line is worth in LDS.
  constexpr int C = ROW ? 1 : P;
  auto pos = [](int q) constexpr { return q + q / 16; };
  double* const line = sh + (ROW ? pair * LP : pair);
  {
    double* w = line + pos(t) * C;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      w[pos(i * T) * C] = v[i].x;
      w[pos(N + i * T) * C] = v[i].y;
    }
    __syncthreads();
    // value L - (t + i T), which is value 0 for t = 0, i = 8
    const double* r = line - (t + (t + 15) / 16) * C;
#pragma unroll
    for (int i = 8; i < 16; ++i) {
      // (T = 8: L - i T is an odd multiple of 8 for odd i, and t < 8)
      const double* ri = i == 8 && t == 0 ? line - pos(N) * C : (L - i * T) % 16 ? line - t * C : r;
      v[i] = {-ri[pos(L - i * T) * C], -ri[pos(N + L - i * T) * C]};
    }
  }
  // hand the values over: value i goes to put + its constant, what comes back
  // is at get + its constant
  auto exchange = [&](int put, auto put_c, int get, auto get_c) {
    double* w = line + put * C;
    const double* r = line + get * C;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) w[put_c(i) * C] = v[i].x;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i].x = r[get_c(i) * C];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) w[put_c(i) * C] = v[i].y;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i].y = r[get_c(i) * C];
  };
  dft<16>(v, 0, 1);
  constexpr int M = 16 / RL;   // the last step's transforms per thread
  if constexpr (LOG >= 8) {
    const int k = t & 15;
    Twiddle<16> w;
    w.load(a.tw, k * (L / 256), L - 1);
    exchange(t * 17, [](int i) { return i; }, pos(t), [&](int i) { return pos(i * T); });
    w.apply(v, 0, 1);
    dft<16>(v, 0, 1);
    if constexpr (RL > 1)
      exchange((t >> 4) * pos(256) + k, [&](int i) { return pos(i * 16); }, pos(t),
               [&](int i) { return pos((i / RL) * T + (i % RL) * 256); });
  } else {
    // (T = 8: value t + 8 c + 16 i, of position t + 8 c + 17 i)
    exchange(t * 17, [](int i) { return i; }, t, [&](int i) { return (i / RL) * T + (i % RL) * 17; });
  }
  if constexpr (RL > 1) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      Twiddle<RL> w;
      w.load(a.tw, t + m * T, L - 1);
      w.apply(v, m * RL, 1);
      dft<RL>(v, m * RL, 1);
    }
  }
  // coefficient k of value i; those past N repeat the first half (known when
  // compiling, so the last step does not form them)
  const double sc = 0.5 * sqrt(2.0 / N);
  const int k0 = RL > 1 ? t : (t >> 4) * 256 + (t & 15);
  auto put = [&](auto store) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      constexpr int NS = L / RL;
      if (RL > 1 ? (i % RL) >= RL / 2 : i >= 8) continue;
      if (i == 0 && k0 == 0) continue;
      store((RL > 1 ? (i / RL) * T + (i % RL) * NS : i * 16) * step, -sc * v[i].y, sc * v[i].x);
    }
  };
  double* const o0 = out + (k0 - 1) * step + l0 * (ROW ? n : 1);
  if (!ROW && on1) {
    put([&](long long o, double x, double y) { *reinterpret_cast<f64x2u*>(o0 + o) = f64x2u{x, y}; });
  } else {
    if (on0) put([&](long long o, double x, double) { o0[o] = x; });
    if (ROW && on1) put([&](long long o, double, double y) { o0[n + o] = y; });
  }
  if (ROW && !SCALE && a.partial && tid == 0) {
    double tot = 0.0;
    for (int w = 0; w < NW; ++w) tot += sw[w];
    a.partial[grp] = tot;
  }
}

__global__ __launch_bounds__(256) void k_fft_table(int L, double2* tw) {
  const int m = blockIdx.x * 256 + threadIdx.x;
  if (m >= L) return;
  double s, c;
  sincospi(2.0 * m / L, &s, &c);
  tw[m] = make_double2(c, -s);
}

template <int LOG, bool ROW, bool SCALE>
void run_fft_log(FftPass a, long long batches, hipStream_t st) {
  constexpr int P = fft_pairs<LOG>(ROW);
  a.tiles = (int)((a.lines + 2 * P - 1) / (2 * P));
  a.groups = batches * a.tiles;
  a.per = (a.groups + 7) / 8;
  hipLaunchKernelGGL((k_sine_fft<LOG, ROW, SCALE>), dim3((unsigned)(8 * a.per)), dim3((1 << LOG) / 16 * P), 0, st, a);
}

template <bool ROW, bool SCALE>
void run_fft(const SinePass& p, const double2* tw, long long batches, hipStream_t st) {
  FftPass a{};
  a.in = p.in;
  a.out = p.out;
  a.tw = tw;
  a.n = p.n;
  a.in_stride = p.in_stride;
  a.out_stride = p.out_stride;
  a.ld = p.ld;
  a.lines = p.lines;
  a.planes = p.planes;
  a.rhs_of = p.rhs_of;
  // A scaled pass reads the same coefficients for every system of a right-hand
  // side.  In 3D, where they are more than the L2s hold (32 MB), the systems of
  // a tile go side by side and read them once: 255^3, 9 systems 803 -> 566 us.
  // In 2D they stay in the caches and a system's neighbouring tiles, which
  // share lines of memory, have to be close: 1023^2, 30 systems by tiles 149 us
  // against 121.
  a.by_tile = p.axes == 2 && p.in_stride * 8 > (32LL << 20);
  a.gate = p.gate;
  a.zero = p.zero;
  a.mu = p.mu;
  a.axes = p.axes;
  a.wc = p.wc;
  a.shift = p.shift;
  a.partial = p.partial;
  a.ctr = p.ctr;
  switch (p.n + 1) {
    case 64: run_fft_log<7, ROW, SCALE>(a, batches, st); break;
    case 128: run_fft_log<8, ROW, SCALE>(a, batches, st); break;
    case 256: run_fft_log<9, ROW, SCALE>(a, batches, st); break;
    case 512: run_fft_log<10, ROW, SCALE>(a, batches, st); break;
    case 1024: run_fft_log<11, ROW, SCALE>(a, batches, st); break;
    case 2048: run_fft_log<12, ROW, SCALE>(a, batches, st); break;
  }
}

// one pass of either kind
template <bool ROW, bool INV, bool SCALE>
void pass(const SinePass& a, const double2* tw, long long batches, hipStream_t st) {
  if (tw) run_fft<ROW, SCALE>(a, tw, batches, st);
  else run_pass<ROW, INV, SCALE>(a, batches, st);
}

// grids whose transforms are fast Fourier transforms
bool by_fft(int n) {
  const int N = n + 1;
  return (N & n) == 0 && N >= kFftMin && N <= 2048;
}

// lines per workgroup of the forward row pass
int fft_row_lines(int n) {
  const int T = (n + 1) / 8;
  return 2 * (T >= 256 ? 1 : 256 / T);
}

// --------------------------------------------------------------------------
// The residual test and the combine (see launch_check)
//
// Bound by one read of every system's x (8 bytes a point): a thread owns a
// block of points, keeps f and the sums of the outputs there in registers and
// goes through the terms of its output, so x is read once for both.  The
// separate passes read it twice, and the residual pass of the refinement also
// writes r and e, which only a system over its tolerance needs (1023^2, 30
// systems: 139 + 69 -> 109 us; 255^3, 9 systems: 803 + 260 -> 611 us).
// --------------------------------------------------------------------------
constexpr int kCheckRows = 4;   // rows per thread

// the sums of a workgroup's four waves over each term's points, one barrier
// for all terms
struct CheckSums {
  double* wave;   // [term][4] in LDS
  __device__ __forceinline__ void add(int slot, double v) const {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    if ((tid & 63) == 0) wave[slot * 4 + (tid >> 6)] = v;
  }
  __device__ __forceinline__ double total(int slot) const {
    const double* w = wave + slot * 4;
    return (w[0] + w[1]) + (w[2] + w[3]);
  }
};

// 2D: the next term's loads are in flight while a term is used.  3D: one plane
// per workgroup, and each XCD (workgroups are dealt to the 8 XCDs round-robin)
// keeps a range of rows and walks the planes, so the planes above and below
// come from its L2 (10 terms x 3 planes x 1/8 of 255^2 points: 2 of 4 MB).
template <int DIM, bool COMB>
__global__ __launch_bounds__(256) void k_check(CheckArgs a, CombineTerms t) {
  constexpr int R = kCheckRows;
  __shared__ double wave_sums[(BURA_MAX_TERMS + 1) * 4];
  const CheckSums sums{wave_sums};
  const int n = a.n;
  const int z = blockIdx.z;
  const int out = COMB ? z / a.nrhs : 0, r = COMB ? z % a.nrhs : z % a.stride;
  const int jb = COMB ? t.begin[out] : z / a.stride, je = COMB ? t.begin[out + 1] : jb + 1;
  const int xt = (n + blockDim.x - 1) / blockDim.x, yt = (n + blockDim.y * R - 1) / (blockDim.y * R);
  const int tiles = xt * yt;
  int tile = blockIdx.x, k = 0;
  if (DIM == 3) {
    const int per = (tiles + 7) / 8, q = blockIdx.x >> 3;
    k = q / per;
    tile = (blockIdx.x & 7) * per + q % per;
    if (tile >= tiles) return;
  }
  const int blk = k * tiles + tile, nblk = DIM == 3 ? tiles * n : tiles;
  const int by = tile / xt;
  const int i = (tile - by * xt) * blockDim.x + threadIdx.x, j0 = (by * blockDim.y + threadIdx.y) * R;
  const bool on = i < n && j0 < n;
  const int ic = min(i, n - 1);
  const long long nn = (long long)n * n, pk = k * nn;
  // in-plane offsets of the rows j0 - 1 .. j0 + R, on the grid
  int row[R + 2];
#pragma unroll
  for (int q = 0; q < R + 2; ++q) row[q] = min(max(j0 - 1 + q, 0), n - 1) * n;
  const int il = max(ic - 1, 0), ir = min(ic + 1, n - 1);
  const long long pb = (k > 0 ? k - 1 : 0) * nn, pa = min(k + 1, n - 1) * nn;
  if (!COMB && !a.active[z]) return;
  if (a.ctr && blk == 0 && threadIdx.x == 0 && threadIdx.y == 0)
    atomicAdd(a.ctr, (unsigned long long)a.N * 8ULL * ((je - jb) + 1 + (COMB ? 1 : 0)));
  double fv[R], acc[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const long long p = (long long)r * a.N + pk + row[q + 1] + ic;
    fv[q] = a.f[p];
    acc[q] = COMB && a.base ? a.base_w * a.base[p] : 0.0;
  }
  const double wc = a.wc;
  struct Block {   // the points of a thread and their neighbours
    double c[R + 2], l[R], r[R], b[DIM == 3 ? R : 1], f[DIM == 3 ? R : 1];
  };
  auto load = [&](int j, Block& p) {
    const double* __restrict__ xs = a.x + ((long long)j * a.stride + r) * a.N;
#pragma unroll
    for (int q = 0; q < R + 2; ++q) p.c[q] = xs[pk + row[q] + ic];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      p.l[q] = xs[pk + row[q + 1] + il];
      p.r[q] = xs[pk + row[q + 1] + ir];
      if (DIM == 3) {
        p.b[DIM == 3 ? q : 0] = xs[pb + row[q + 1] + ic];
        p.f[DIM == 3 ? q : 0] = xs[pa + row[q + 1] + ic];
      }
    }
  };
  auto term = [&](int j, const Block& p) {
    const long long sys = (long long)j * a.stride + r;
    const bool act = a.active[sys] != 0;
    const double wv = COMB ? (a.wsys ? a.w[sys] : a.w[j]) : 0.0;
    // per-system weights: a zero weight marks an unused slot, whose x does not count
    const bool used = COMB && !(a.wsys && wv == 0.0);
    if (!act && !used) return;
    const double s = a.shift[sys];
    double rr = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const double c = p.c[q + 1];
      const double dn = j0 + q > 0 ? p.c[q] : 0.0, up = j0 + q + 1 < n ? p.c[q + 2] : 0.0;
      const double lv = i > 0 ? p.l[q] : 0.0, rv = i < n - 1 ? p.r[q] : 0.0;
      double d = (c - lv) + (c - rv) + (c - dn) + (c - up);
      if (DIM == 3)
        d += (c - (k > 0 ? p.b[DIM == 3 ? q : 0] : 0.0)) + (c - (k + 1 < n ? p.f[DIM == 3 ? q : 0] : 0.0));
      const double res = fv[q] - (wc * d + s * c);
      if (on && j0 + q < n) rr += res * res;
      if (used) acc[q] += wv * c;
    }
    if (act) sums.add(j - jb, rr);
  };
  Block cur;
  if (DIM == 2 && COMB) {
    Block next;
    load(jb, cur);
    for (int j = jb; j < je; j += 2) {
      if (j + 1 < je) load(j + 1, next);
      term(j, cur);
      if (j + 1 >= je) break;
      if (j + 2 < je) load(j + 2, cur);
      term(j + 1, next);
    }
  } else {
    for (int j = jb; j < je; ++j) {
      load(j, cur);
      term(j, cur);
    }
  }
  double uu = 0.0;
  if (COMB && on) {
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (j0 + q < n) {
        a.u[(long long)z * a.N + pk + row[q + 1] + ic] = acc[q];
        uu += acc[q] * acc[q];
      }
  }
  if (COMB && a.upartial) sums.add(BURA_MAX_TERMS, uu);
  __syncthreads();
  const int tid = threadIdx.x + threadIdx.y * blockDim.x;
  if (tid < je - jb) {
    const long long sys = (long long)(jb + tid) * a.stride + r;
    if (a.active[sys]) a.partial[sys * nblk + blk] = sums.total(tid);
  }
  if (COMB && a.upartial && tid == 64) a.upartial[(size_t)z * nblk + blk] = sums.total(BURA_MAX_TERMS);
}

dim3 check_block(int n) {
  const int x = n >= 192 ? 256 : (n >= 96 ? 128 : 64);
  return dim3(x, 256 / x);
}

int check_tiles(int n) {
  const dim3 b = check_block(n);
  return ((n + b.x - 1) / b.x) * ((n + b.y * kCheckRows - 1) / (b.y * kCheckRows));
}

}  // namespace

int check_blocks(int dim, int n) { return check_tiles(n) * (dim == 3 ? n : 1); }

// The terms of an output go one after the other there, about 1.3 us each on a
// grid too small to hide their loads: from about one workgroup per CU on the
// one pass is the shorter (511^2, 256 workgroups, 9 terms: 15 against 11 + 7 us;
// 63^3, 252: 23 against 28; 127^2, 16 workgroups, 10 terms: 15 against 4 + 5).
bool check_combines(int dim, int n, int rows) { return (long long)check_blocks(dim, n) * rows >= 200; }

void launch_check(int dim, const CheckArgs& a, const CombineTerms& t, int nout, int nsys, hipStream_t st) {
  const dim3 b = check_block(a.n);
  const int tiles = check_tiles(a.n);
  const dim3 g(dim == 3 ? (tiles + 7) / 8 * 8 * a.n : tiles, 1, a.u ? nout * a.nrhs : nsys);
#define BURA_CHECK(D, C) hipLaunchKernelGGL((k_check<D, C>), g, b, 0, st, a, t)
  if (dim == 3) {
    if (a.u) BURA_CHECK(3, true);
    else BURA_CHECK(3, false);
  } else {
    if (a.u) BURA_CHECK(2, true);
    else BURA_CHECK(2, false);
  }
#undef BURA_CHECK
}

int sine_half(int n) { return (((n + 1) / 2) + 63) / 64 * 64; }

// the 1D eigenvalues, then the twiddle factors or the four half matrices
static size_t mu_doubles(int n) { return ((size_t)n + 1) / 2 * 2; }

size_t sine_table_doubles(int n) {
  return mu_doubles(n) + (by_fft(n) ? 4 * (size_t)(n + 1) : 4 * (size_t)sine_half(n) * sine_half(n));
}

void launch_sine_tables(int n, double* tab, hipStream_t st) {
  const bool fft = by_fft(n);
  const int hp = sine_half(n);
  const long long hh = fft ? 0 : (long long)hp * hp;
  double* mats = tab + mu_doubles(n);
  hipLaunchKernelGGL(k_sine_tables, dim3((unsigned)((std::max<long long>(hh, n) + 255) / 256)), dim3(256), 0, st, n,
                     (n + 1) / 2, n / 2, fft ? 0 : hp, mats, tab);
  if (fft)
    hipLaunchKernelGGL(k_fft_table, dim3((2 * (n + 1) + 255) / 256), dim3(256), 0, st, 2 * (n + 1), (double2*)mats);
}

int sine_norm_blocks(int dim, int n, int nrhs) {
  const long long rows = dim == 3 ? (long long)n * n : n;
  if (by_fft(n)) return (int)((rows + fft_row_lines(n) - 1) / fft_row_lines(n));
  const int hp = (n + 1) / 2;
  const long long t64 = (rows + 63) / 64;
  const long long big = ((nrhs * t64 + 7) / 8) * 8 * ((hp + 63) / 64);
  return (int)(big >= 512 ? t64 : (rows + 31) / 32);
}

int sine_norm_max_blocks(int dim, int n) {
  const long long rows = dim == 3 ? (long long)n * n : n;
  const int lines = by_fft(n) ? fft_row_lines(n) : 32;
  return (int)((rows + lines - 1) / lines);
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
  const double2* tw = by_fft(n) ? (const double2*)(s.tab + mu_doubles(n)) : nullptr;
  a.t0 = s.tab + mu_doubles(n);
  a.t1 = a.t0 + hh;
  a.ctr = ctr;
  a.ld = n;
  // x: f -> work
  a.in = s.f;
  a.out = s.work;
  a.in_stride = a.out_stride = N;
  a.lines = N / n;
  a.partial = partial;
  pass<true, false, false>(a, tw, s.nrhs, st);
  a.partial = nullptr;
  // y: work -> x
  a.in = s.work;
  a.out = s.x;
  a.lines = n;
  a.in_stride = a.out_stride = nn;
  pass<false, false, false>(a, tw, s.dim == 3 ? (long long)s.nrhs * n : s.nrhs, st);
  if (s.dim == 3) {
    // z: x -> work
    a.in = s.x;
    a.out = s.work;
    a.ld = nn;
    a.lines = nn;
    a.in_stride = a.out_stride = N;
    pass<false, false, false>(a, tw, s.nrhs, st);
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
  const double2* tw = by_fft(n) ? (const double2*)(s.tab + mu_doubles(n)) : nullptr;
  a.t0 = s.tab + mu_doubles(n) + 2 * hh;
  a.t1 = a.t0 + hh;
  a.mu = s.tab;
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
  pass<false, true, true>(a, tw, s.nsys, st);
  a.rhs_of = 0;
  if (s.dim == 3) {
    // y, plane by plane: x -> work
    a.in = s.x;
    a.out = s.work;
    a.ld = n;
    a.lines = n;
    a.planes = n;
    a.in_stride = a.out_stride = nn;
    pass<false, true, false>(a, tw, (long long)s.nsys * n, st);
    a.planes = 1;
  }
  // x: work -> x
  a.in = s.work;
  a.out = s.x;
  a.ld = n;
  a.lines = N / n;
  a.in_stride = a.out_stride = N;
  a.zero = 1;
  pass<true, true, false>(a, tw, s.nsys, st);
}

}  // namespace bura
