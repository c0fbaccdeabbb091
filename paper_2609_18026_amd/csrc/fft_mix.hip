// Mixed-radix FFTs for the lengths n = R1 R2 (R1, R2 of 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16) other than
// 256: a line is transformed in two passes held in registers, a radix-R1 pass, one exchange through
// LDS and a radix-R2 pass,
//   X[k1 + R1 k2] = sum_{n2} w_n^(k1 n2) w_R2^(k2 n2) sum_{n1} w_R1^(k1 n1) x[R2 n1 + n2],
// where the Stockham passes of radices 2 to 5 in kernels.hip move every sample through LDS four to
// seven times (they stay for the lengths with no such pair: 125, 162, 200, 216, 243 and 250 below
// 256, and most lengths above).
//
// Kernels: the z transforms over contiguous lines, up to six fields in one launch, and the azimuthal
// stages on groups of lines (the scalar transforms and nonlinear terms, and the vector stage of the
// toroidal-poloidal RHS).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dev_common.h"
#include "dft_reg.h"
#include "mlg_internal.h"

namespace mlg {
namespace {

using namespace ::mlg::dev;

// v[c] *= w_n^(e c), c = 1 .. R - 1, w_n = exp(-2 pi i / n) (conjugated for the inverse), c e < n.  Every factor comes from
// the table: factors formed as products of the powers 1, 2, 4, 8 left up to 15% more rounding error in a transform (root mean
// square over white lines: 1.81e-16 at n = 48 against 1.59e-16 with the LDS passes).
template <int R, bool INV>
__device__ __forceinline__ void twiddle_tab(double2 (&v)[R], const double2* __restrict__ tw, int e) {
#pragma unroll
  for (int c = 1; c < R; ++c) {
    const double2 w = tw[c * e];
    v[c] = cmul(v[c], INV ? cconj(w) : w);
  }
}

// The lengths served, as R1 >= R2 with R1 as small as possible: one kernel instance per length, so that each
// takes the registers of its own radices.  MIX_PAIRS: R2 <= 10, all stages; MIX_WIDE: the rest, which the
// vector stage (three pairs of R2 values per lane) leaves to the kernel in kernels.hip.
#define MIX_PAIRS(X) \
  X(2, 2) X(3, 2) X(4, 2) X(3, 3) X(5, 2) X(4, 3) X(5, 3) X(4, 4) X(6, 3) X(5, 4) X(6, 4) X(5, 5) X(9, 3) \
  X(6, 5) X(8, 4) X(6, 6) X(8, 5) X(9, 5) X(8, 6) X(10, 5) X(9, 6) X(10, 6) X(8, 8) X(9, 8) X(15, 5) X(10, \
  8) X(9, 9) X(10, 9) X(12, 8) X(10, 10) X(12, 9) X(12, 10) X(16, 8) X(15, 9) X(16, 9) X(15, 10) X(16, 10)
#define MIX_WIDE(X) \
  X(15, 12) X(16, 12) X(15, 15) X(16, 15)

// ---------------------------------------------------------------- z transforms
// Contiguous lines, lb lines per block.  Lane (line, n2) of the first pass loads x[n2 + R2 n1] straight
// into registers; lane (line, k1) of the second stores X[k1 + R1 k2].  In LDS a line is R1 rows of RS
// (R2 rounded up to odd) entries, so that the rows read by neighbouring lanes start in different
// banks.  In place when in == out: every line belongs to one block, which has read it before the
// barrier and writes it after.  Bound by memory: at 128^3 the six inverse transforms of the vector term take
// 24 us (113 MB, 4.7 TB/s, the rate of a plain copy) against 72 us in six launches of zfft_kernel.
struct ZMix {
  int lb, mask_m, mask_k, kept_only;  // kept slots: |k| <= mask_k
  int64_t rows, per_field;
  const int32_t* row_m;
  // the proxy parts (Eq. logproxy) join the slot 0 of the order 0 rows (node: rinv, q of the nr nodes; nr = 0: none;
  // as a launch of its own this took 4 us a step)
  const double* node;
  int nr;
  LogProxy proxy;
  const double2* in[6];
  double2* out[6];
};

template <int R1, int R2, bool INV>
__global__ __launch_bounds__(256) void zmix_kernel(ZMix a, const double2* __restrict__ twg) {
  extern __shared__ double2 smem[];
  constexpr int n = R1 * R2, RS = R2 | 1;
  const int lb = a.lb;
  double2* T = smem;
  double2* tw = smem + lb * R1 * RS;
  const int64_t nf = gridDim.x / a.per_field;
  const int64_t f = blockIdx.x % nf;
  const int64_t r0 = (int64_t)(blockIdx.x / nf) * lb;
  const double2* __restrict__ in = a.in[f];
  double2* __restrict__ out = a.out[f];
  const int kp = a.mask_k;
  for (int t = threadIdx.x; t < n; t += 256) tw[t] = twg[t];
  __syncthreads();
  for (int e = threadIdx.x; e < lb * R2; e += 256) {
    const int line = e / R2, n2 = e % R2;
    const int64_t row = r0 + line;
    const bool ok = row < a.rows && !(a.row_m && a.row_m[row < a.rows ? row : 0] > a.mask_m);  // else zero
    const double2* x = in + row * n;
    double2 v[R1];
#pragma unroll
    for (int c = 0; c < R1; ++c) {
      const int kk = n2 + c * R2;
      v[c] = make_double2(0.0, 0.0);
      if (ok && (!INV || kk <= kp || kk >= n - kp)) v[c] = x[kk];
    }
    if (INV && n2 == 0 && row < a.nr) v[0].x += proxy_part(a.proxy, (int)f, a.node[row], a.node[a.nr + row]);
    Dft<R1, INV>::run(v);
    twiddle_tab<R1, INV>(v, tw, n2);
    double2* d = T + line * (R1 * RS) + n2;
#pragma unroll
    for (int c = 0; c < R1; ++c) d[c * RS] = v[c];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < lb * R1; e += 256) {
    const int line = e / R1, k1 = e % R1;
    const int64_t row = r0 + line;
    if (row >= a.rows) continue;
    const double2* d = T + line * (R1 * RS) + k1 * RS;
    double2 v[R2];
#pragma unroll
    for (int c = 0; c < R2; ++c) v[c] = d[c];
    Dft<R2, INV>::run(v);
    const bool dead = !INV && a.row_m && a.row_m[row] > a.mask_m;
    double2* y = out + row * n;
#pragma unroll
    for (int c = 0; c < R2; ++c) {
      const int kk = k1 + c * R1;
      if (INV) {
        y[kk] = v[c];
      } else if (!dead && (kk <= kp || kk >= n - kp)) {
        y[kk] = cscale(v[c], 1.0 / n);
      } else if (!a.kept_only) {
        y[kk] = make_double2(0.0, 0.0);
      }
    }
  }
}

// ---------------------------------------------------------------- azimuthal stages
// Line q = i N_z + l; physical samples at (l N_r + i) N_phi + j; harmonic m at m * nlines + q.  A block
// takes 2^lbs lines (or pairs of lines); in LDS entry (k, line) sits at k * row + line, so the lanes of
// every access run over the lines first: 16-byte entries side by side, whatever the order k.
struct PhiMix {
  int n, lbs, nr, nz;
  int min_, mout;       // orders read (the others enter as zero) and orders written
  int64_t nlines;
};

__device__ __forceinline__ int64_t phys_off(const PhiMix& g, int64_t q) {
  const int64_t i = q / g.nz, l = q - i * g.nz;
  return (l * g.nr + i) * g.n;
}

// First pass (radix R of n = R S): lane (n2, line) reads x[n2 + S n1] from X and writes row k1, entry n2
// of Y; second pass in second_pass: lane (k1, line) reads row k1 of length R2 and leaves X[k1 + R1 k2].
template <int R, bool INV>
__device__ __forceinline__ void mix_first(const double2* X, double2* Y, int S, int n2, int line, int row,
                                          const double2* tw) {
  double2 v[R];
#pragma unroll
  for (int c = 0; c < R; ++c) v[c] = X[(n2 + c * S) * row + line];
  Dft<R, INV>::run(v);
  twiddle_tab<R, INV>(v, tw, n2);
#pragma unroll
  for (int c = 0; c < R; ++c) Y[(c * S + n2) * row + line] = v[c];
}

struct Six {
  double2* f[6];
};

// Vector stage: six harmonic fields -> nodal u, w -> N = (U + u) x w -> harmonics of N_r / r, N_phi / r,
// N_z over fields 0, 1, 2 (see phi_vec256_kernel, of which this is the form for the other lengths).  A
// block holds 2^lbs lines, R1 lanes per line; pairs of fields travel as one complex line.  The
// inverse transforms end with their radix-R2 pass and leave X[k1 + R1 k2] in lane k1: the input of
// the forward transforms' first pass taken with the radices in the other order, so the nodal values
// stay in registers from the inverse to the forward transform.  The next pair's harmonics are
// loaded into registers while the current pair is transformed.  R2 <= R1 keeps the three pairs' values
// (12 R2 registers) small.
// Bound by memory: 6 fields read and 3 written on the kept orders, in pieces of 16 2^lbs bytes: at 128^3
// 101 MB in 35 us (2.9 TB/s) against 142 us with phi_vec_kernel, at 200 x 128 x 128 50 against 216 us.
template <int R1, int R2, bool TAPS>
__global__ __launch_bounds__(128) void phi_vec_mix_kernel(PhiMix g, const double2* __restrict__ twg, Six fs,
                                                          const double* __restrict__ rinv, double Ux, double Uy,
                                                          double Uz, double* __restrict__ taps) {
  extern __shared__ double2 smem[];
  constexpr int n = R1 * R2;
  const int lb = 1 << g.lbs;
  double2* Z = smem;                 // [n][lb]
  double2* T = smem + (n << g.lbs);  // [n][lb]
  double2* tw = T + (n << g.lbs);
  const int tid = threadIdx.x, ll = tid & (lb - 1), k1 = tid >> g.lbs;  // blockDim = lb R1
  const int64_t q0 = (int64_t)blockIdx.x << g.lbs, q = q0 + ll;
  const bool valid = q < g.nlines;
  constexpr int NP = (R2 + 1) / 2;  // orders below n / 2 per lane and field
  double2 pa[NP], pb[NP];
  auto load = [&](const double2* __restrict__ fa, const double2* __restrict__ fb) {
#pragma unroll
    for (int it = 0; it < NP; ++it) {
      const int m = k1 + it * R1;
      const bool ok = valid && m < g.min_;
      const int64_t o = ok ? (int64_t)m * g.nlines + q : 0;
      pa[it] = ok ? fa[o] : make_double2(0.0, 0.0);
      pb[it] = ok ? fb[o] : make_double2(0.0, 0.0);
    }
  };
  // the pair's Hermitian spectrum A + i B at the orders read; the other entries stay zero
  auto store = [&]() {
#pragma unroll
    for (int it = 0; it < NP; ++it) {
      const int m = k1 + it * R1;
      if (m >= g.min_) continue;
      const double2 a = pa[it], b = pb[it];
      if (m == 0) {
        Z[ll] = make_double2(a.x, b.x);
      } else {
        Z[(m << g.lbs) + ll] = make_double2(a.x - b.y, a.y + b.x);
        Z[((n - m) << g.lbs) + ll] = make_double2(a.x + b.y, -a.y + b.x);
      }
    }
  };
  load(fs.f[0], fs.f[1]);
  for (int e = tid; e < n; e += blockDim.x) tw[e] = twg[e];
  for (int k = g.min_ + k1; k <= n - g.min_; k += R1) Z[(k << g.lbs) + ll] = make_double2(0.0, 0.0);
  double2 x[3][R2];
#pragma unroll
  for (int pr = 0; pr < 3; ++pr) {
    store();
    if (pr < 2) load(fs.f[2 * pr + 2], fs.f[2 * pr + 3]);
    __syncthreads();
    if (k1 < R2) mix_first<R1, true>(Z, T, R2, k1, ll, lb, tw);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < R2; ++c) x[pr][c] = T[((k1 * R2 + c) << g.lbs) + ll];
    Dft<R2, true>::run(x[pr]);
  }
  // nodal cross product at phi_j, j = k1 + R1 c: cos(phi_j) = tw[j].x, sin(phi_j) = -tw[j].y
  const double ri = valid ? rinv[q / g.nz] : 0.0;
  const int64_t pe = g.nlines * n;
#pragma unroll
  for (int c = 0; c < R2; ++c) {
    const int j = k1 + c * R1;
    const double2 t = tw[j];
    const double cphi = t.x, sphi = -t.y;
    const double ur = x[0][c].x, up = x[0][c].y, uz = x[1][c].x, wr = x[1][c].y, wp = x[2][c].x, wz = x[2][c].y;
    const double Ur = ur + Ux * cphi + Uy * sphi;
    const double Up = up - Ux * sphi + Uy * cphi;
    const double Uzz = uz + Uz;
    const double Nr = Up * wz - Uzz * wp;
    const double Np = Uzz * wr - Ur * wz;
    const double Nz = Ur * wp - Up * wr;
    if (TAPS && valid) {
      const int64_t o = phys_off(g, q) + j;
      taps[0 * pe + o] = ur; taps[1 * pe + o] = up; taps[2 * pe + o] = uz;
      taps[3 * pe + o] = wr; taps[4 * pe + o] = wp; taps[5 * pe + o] = wz;
      taps[6 * pe + o] = Nr; taps[7 * pe + o] = Np; taps[8 * pe + o] = Nz;
    }
    x[0][c] = make_double2(Nr * ri, Np * ri);
    x[1][c] = make_double2(Nz, 0.0);
  }
  // forward: radix R2, then radix R1 on rows c of length R1; N_r, N_phi through Z, N_z through T
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    Dft<R2, false>::run(x[f]);
    twiddle_tab<R2, false>(x[f], tw, k1);
  }
#pragma unroll
  for (int c = 0; c < R2; ++c) Z[((c * R1 + k1) << g.lbs) + ll] = x[0][c];
  __syncthreads();  // every lane has read its last row of T
#pragma unroll
  for (int c = 0; c < R2; ++c) T[((c * R1 + k1) << g.lbs) + ll] = x[1][c];
  __syncthreads();
  // lanes 0 .. R2 - 1 take Z, the next R2 take T where the line has as many lanes, else a second round
  constexpr bool split = 2 * R2 <= R1;
#pragma unroll
  for (int round = 0; round < (split ? 1 : 2); ++round) {
    const int f = split ? k1 / R2 : round, k = split ? k1 - f * R2 : k1;
    const bool act = f < 2 && k < R2;
    double2* B = f ? T : Z;
    double2 v[R1];
    if (act) {
#pragma unroll
      for (int c = 0; c < R1; ++c) v[c] = B[((k * R1 + c) << g.lbs) + ll];
      Dft<R1, false>::run(v);
    }
    __syncthreads();
    if (act) {
#pragma unroll
      for (int c = 0; c < R1; ++c) B[((k + c * R2) << g.lbs) + ll] = v[c];
    }
  }
  __syncthreads();
  if (!valid) return;
  const double h = 0.5 / n;
  for (int m = k1; m < g.mout; m += R1) {
    const int mc = m ? n - m : 0;
    const double2 zm = Z[(m << g.lbs) + ll], zc = cconj(Z[(mc << g.lbs) + ll]);
    const double2 cm = T[(m << g.lbs) + ll], cc = cconj(T[(mc << g.lbs) + ll]);
    const double2 d = csub(zm, zc);
    const int64_t o = (int64_t)m * g.nlines + q;
    fs.f[0][o] = cscale(cadd(zm, zc), h);
    fs.f[1][o] = make_double2(h * d.y, -h * d.x);
    fs.f[2][o] = cscale(cadd(cm, cc), h);
  }
}

// ---------------------------------------------------------------- scalar azimuthal stages
// The backward transform and the nonlinear terms.  Two real lines (2p, 2p + 1) travel as one complex line
// a + i b; a block takes 2^lbs pairs, R1 lanes per pair.  The LDS rows hold one entry more than the block has
// pairs where the physical side reads them along j, so that neighbouring j start in different banks.
// (The forward transform stays with phi_forward_kernel: its rounding is the floor of a transformed field's
// smallest coefficients, which the projection's solves amplify, and another order of the same sums moved the
// vector term of such a field by 2e-7 of its root mean square, in single coefficients, at 128^3.)

// physical offsets of the lines qa and qa + 1 (N_r N_z fits 32 bits: N_r <= 4096, N_z <= 1024)
__device__ __forceinline__ void pair_offs(const PhiMix& g, int64_t qa, int64_t& oa, int64_t& ob) {
  const uint32_t q = (uint32_t)qa, i = q / (uint32_t)g.nz, l = q - i * (uint32_t)g.nz;
  const bool wrap = l + 1 == (uint32_t)g.nz;
  oa = ((int64_t)l * g.nr + i) * g.n;
  ob = ((int64_t)(wrap ? 0 : l + 1) * g.nr + i + (wrap ? 1 : 0)) * g.n;
}

// the pair spectrum of the block's lines in Z (orders below min_, the others zero)
template <int n, int R1>
__device__ __forceinline__ void gather_pairs(const PhiMix& g, const double2* __restrict__ mixed, double2* Z, int row,
                                             int64_t q0, int pr, int k1) {
  const int64_t qa = q0 + 2 * pr;
  for (int m = k1; m < g.min_; m += R1) {
    const double2* f = mixed + (int64_t)m * g.nlines + qa;
    const double2 a = qa < g.nlines ? f[0] : make_double2(0.0, 0.0);
    const double2 b = qa + 1 < g.nlines ? f[1] : make_double2(0.0, 0.0);
    if (m == 0) {
      Z[pr] = make_double2(a.x, b.x);
    } else {
      Z[m * row + pr] = make_double2(a.x - b.y, a.y + b.x);
      Z[(n - m) * row + pr] = make_double2(a.x + b.y, -a.y + b.x);
    }
  }
  for (int k = g.min_ + k1; k <= n - g.min_; k += R1) Z[k * row + pr] = make_double2(0.0, 0.0);
}

// the harmonics of both lines of every pair from its spectrum in Z (orders below mout; from min_ on zero)
template <int n, int R1>
__device__ __forceinline__ void scatter_pairs(const PhiMix& g, double2* __restrict__ mixed, const double2* Z, int row,
                                              int64_t q0, int pr, int k1) {
  const int64_t qa = q0 + 2 * pr;
  if (qa >= g.nlines) return;
  const double h = 0.5 / n;
  for (int m = k1; m < g.mout; m += R1) {
    double2 A = make_double2(0.0, 0.0), B = A;
    if (m < g.min_) {
      const double2 zm = Z[m * row + pr], zc = cconj(Z[(m ? n - m : 0) * row + pr]);
      const double2 d = csub(zm, zc);
      A = cscale(cadd(zm, zc), h);
      B = make_double2(h * d.y, -h * d.x);
    }
    double2* f = mixed + (int64_t)m * g.nlines + qa;
    f[0] = A;
    if (qa + 1 < g.nlines) f[1] = B;
  }
}

template <int R1, int R2>
__global__ __launch_bounds__(256) void phi_bwd_mix_kernel(PhiMix g, const double2* __restrict__ twg,
                                                          const double2* __restrict__ mixed, double* __restrict__ phys) {
  extern __shared__ double2 smem[];
  constexpr int n = R1 * R2;
  const int lb = 1 << g.lbs, row = lb + 1;
  double2* Z = smem;
  double2* T = smem + n * row;
  double2* tw = T + n * row;
  const int tid = threadIdx.x, pr = tid & (lb - 1), k1 = tid >> g.lbs;
  const int64_t q0 = (int64_t)blockIdx.x << (g.lbs + 1);
  for (int e = tid; e < n; e += blockDim.x) tw[e] = twg[e];
  gather_pairs<n, R1>(g, mixed, Z, row, q0, pr, k1);
  __syncthreads();
  if (k1 < R2) mix_first<R1, true>(Z, T, R2, k1, pr, row, tw);
  __syncthreads();
  double2 x[R2];
#pragma unroll
  for (int c = 0; c < R2; ++c) x[c] = T[(k1 * R2 + c) * row + pr];
  Dft<R2, true>::run(x);
#pragma unroll
  for (int c = 0; c < R2; ++c) Z[(k1 + c * R1) * row + pr] = x[c];
  __syncthreads();
  for (int e = tid; e < (n << g.lbs); e += blockDim.x) {
    const int p = e / n, j = e - p * n;
    const double2 v = Z[j * row + p];
    const int64_t qa = q0 + 2 * p;
    int64_t oa, ob;
    pair_offs(g, qa, oa, ob);
    if (qa < g.nlines) phys[oa + j] = v.x;
    if (qa + 1 < g.nlines) phys[ob + j] = v.y;
  }
}

// Scalar nonlinear term in place: the inverse transform ends with its radix-R2 pass, u^2 or gamma u (1 - u) on
// both real lines in registers, and the forward transform starts from the same lanes with the radices in
// the other order (see phi_vec_mix_kernel).
template <int R1, int R2, int MODE>
__global__ __launch_bounds__(256) void phi_scalar_mix_kernel(PhiMix g, const double2* __restrict__ twg, double2* mixed,
                                                             double gamma) {
  extern __shared__ double2 smem[];
  constexpr int n = R1 * R2;
  const int lb = 1 << g.lbs;
  double2* Z = smem;
  double2* T = smem + (n << g.lbs);
  double2* tw = T + (n << g.lbs);
  const int tid = threadIdx.x, pr = tid & (lb - 1), k1 = tid >> g.lbs;
  const int64_t q0 = (int64_t)blockIdx.x << (g.lbs + 1);
  for (int e = tid; e < n; e += blockDim.x) tw[e] = twg[e];
  gather_pairs<n, R1>(g, mixed, Z, lb, q0, pr, k1);
  __syncthreads();
  if (k1 < R2) mix_first<R1, true>(Z, T, R2, k1, pr, lb, tw);
  __syncthreads();
  double2 x[R2];
#pragma unroll
  for (int c = 0; c < R2; ++c) x[c] = T[((k1 * R2 + c) << g.lbs) + pr];
  Dft<R2, true>::run(x);
#pragma unroll
  for (int c = 0; c < R2; ++c) {
    const double a = x[c].x, b = x[c].y;
    x[c] = MODE == MLG_RHS_U2 ? make_double2(a * a, b * b)
                              : make_double2(gamma * a * (1.0 - a), gamma * b * (1.0 - b));
  }
  Dft<R2, false>::run(x);
  twiddle_tab<R2, false>(x, tw, k1);
#pragma unroll
  for (int c = 0; c < R2; ++c) Z[((c * R1 + k1) << g.lbs) + pr] = x[c];
  __syncthreads();
  if (k1 < R2) {
    double2 v[R1];
#pragma unroll
    for (int c = 0; c < R1; ++c) v[c] = Z[((k1 * R1 + c) << g.lbs) + pr];
    Dft<R1, false>::run(v);
#pragma unroll
    for (int c = 0; c < R1; ++c) T[((k1 + c * R2) << g.lbs) + pr] = v[c];  // every lane has read its row of T
  }
  __syncthreads();
  scatter_pairs<n, R1>(g, mixed, T, lb, q0, pr, k1);
}

mlg_status check(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
  return MLG_OK;
}

}  // namespace

// n = R1 R2 of MIX_PAIRS (wide: or of MIX_WIDE); false if n is none of them
bool mix_pair(int n, bool wide, int* R1, int* R2) {
#define MIX_FIND(A, B) \
  if (n == A * B) {    \
    *R1 = A;           \
    *R2 = B;           \
    return true;       \
  }
  MIX_PAIRS(MIX_FIND)
  if (wide) {
    MIX_WIDE(MIX_FIND)
  }
#undef MIX_FIND
  return false;
}

bool zmix_ok(const mlg_plan_s* p) {
  int a, b;
  return p->prec == MLG_FP64 && mix_pair(p->nz, true, &a, &b);
}

mlg_status launch_zmix(const mlg_plan_s* p, const double* const* in, double* const* out, int nf, int64_t rows, int dir,
                       const int32_t* row_m, int mask_m, int mask_k, hipStream_t s, bool kept_only, bool proxy) {
  if (nf < 1 || nf > 6) return fail(MLG_E_ARG, "z transform: 1 to 6 fields per launch");
  ZMix a{};
  int R1, R2;
  if (!mix_pair(p->nz, true, &R1, &R2)) return fail(MLG_E_UNSUPPORTED, "z transform: length without a radix pair");
  // the largest kept |k|: the chop, never the Nyquist slot, and the mask
  int kp = std::min(p->nzc - 1, (p->nz - 1) / 2);
  if (mask_k >= 0) kp = std::min(kp, mask_k);
  a.mask_k = kp;
  a.mask_m = mask_m;
  a.row_m = row_m;
  a.kept_only = kept_only;
  a.rows = rows;
  // about one line-lane per thread, and at most 64 KB of LDS
  const int line = R1 * (R2 | 1);
  a.lb = std::min(std::max(1, 256 / R1), (4096 - p->nz) / line);
  a.per_field = (rows + a.lb - 1) / a.lb;
  for (int i = 0; i < nf; ++i) {
    a.in[i] = reinterpret_cast<const double2*>(in[i]);
    a.out[i] = reinterpret_cast<double2*>(out[i]);
  }
  if (proxy && (p->log_cpsi != 0.0 || p->log_cchi != 0.0)) {
    a.node = p->d_node;
    a.nr = p->nr;
    a.proxy = LogProxy{p->log_cpsi, p->log_cchi, p->g.ell};
  }
  const size_t shm = ((size_t)a.lb * line + p->nz) * sizeof(double2);
  const dim3 grid((unsigned)(a.per_field * nf));
  const double2* tw = reinterpret_cast<const double2*>(p->d_tw_z);
  p->timing.begin("z_fft", s);
  switch (p->nz) {
#define MIX_Z(A, B)                                                      \
  case A * B:                                                            \
    if (dir > 0) zmix_kernel<A, B, true><<<grid, 256, shm, s>>>(a, tw);  \
    else zmix_kernel<A, B, false><<<grid, 256, shm, s>>>(a, tw);         \
    break;
    MIX_PAIRS(MIX_Z) MIX_WIDE(MIX_Z)
#undef MIX_Z
  }
  p->timing.end(s);
  return check("zmix_kernel");
}

namespace {

PhiMix phi_mix(const mlg_plan_s* p, bool masked) {
  PhiMix g{};
  g.n = p->nphi;
  g.nr = p->nr;
  g.nz = p->nz;
  g.nlines = (int64_t)p->nr * p->nz;
  g.min_ = std::min(p->M, (p->nphi + 1) / 2);  // stored orders below the Nyquist order
  if (masked) g.min_ = std::min(g.min_, p->dealias_m + 1);
  g.mout = g.min_;
  return g;
}

template <int R1, int R2>
void vec_go(const PhiMix& g, const double2* tw, const Six& six, const double* node, const double* U, double* taps,
            size_t shm, hipStream_t s) {
  const unsigned blocks = (unsigned)((g.nlines + (1 << g.lbs) - 1) >> g.lbs);
  const unsigned threads = (unsigned)(R1 << g.lbs);
  if (taps)
    phi_vec_mix_kernel<R1, R2, true><<<blocks, threads, shm, s>>>(g, tw, six, node, U[0], U[1], U[2], taps);
  else
    phi_vec_mix_kernel<R1, R2, false><<<blocks, threads, shm, s>>>(g, tw, six, node, U[0], U[1], U[2], taps);
}

}  // namespace

bool phi_vec_mix_ok(const mlg_plan_s* p) {
  int a, b;
  return p->prec == MLG_FP64 && mix_pair(p->nphi, false, &a, &b);
}

mlg_status launch_phi_vec_mix(const mlg_plan_s* p, const double* U, double* const* f6, double* taps, hipStream_t s) {
  PhiMix g = phi_mix(p, p->g.dealias != 0);
  int R1, R2;
  if (!mix_pair(p->nphi, false, &R1, &R2)) return fail(MLG_E_UNSUPPORTED, "phi stage: length without a radix pair");
  g.lbs = 3;
  while (g.lbs < 5 && (R1 << g.lbs) < 64) ++g.lbs;
  const size_t shm = ((size_t)2 * (g.n << g.lbs) + g.n) * sizeof(double2);
  Six six;
  for (int i = 0; i < 6; ++i) six.f[i] = reinterpret_cast<double2*>(f6[i]);
  const double2* tw = reinterpret_cast<const double2*>(p->d_tw_phi);
  p->timing.begin("phi_fft", s);
  switch (g.n) {
#define MIX_VEC(A, B) \
  case A * B: vec_go<A, B>(g, tw, six, p->d_node, U, taps, shm, s); break;
    MIX_PAIRS(MIX_VEC)
#undef MIX_VEC
  }
  p->timing.end(s);
  return check("phi_vec_mix_kernel");
}

// pairs of lines per block: at least a wavefront, and about two blocks per CU where there are lines for them
static int pair_bits(const PhiMix& g, int R1) {
  auto fits = [&](int lbs) { return 2 * g.n * ((1 << lbs) + 1) + g.n <= 4096; };  // 64 KB of LDS
  int lbs = fits(3) ? 3 : 2;
  while (lbs < 5 && fits(lbs + 1) && ((R1 << lbs) < 64 || ((R1 << lbs) < 128 && (g.nlines >> (lbs + 1)) > 1024))) ++lbs;
  return lbs;
}

bool phi_mix_ok(const mlg_plan_s* p) {
  int a, b;
  return p->prec == MLG_FP64 && mix_pair(p->nphi, true, &a, &b);
}

mlg_status launch_phi_mix_backward(const mlg_plan_s* p, const double* mixed, double* phys, hipStream_t s) {
  PhiMix g = phi_mix(p, false);
  int R1, R2;
  if (!mix_pair(p->nphi, true, &R1, &R2)) return fail(MLG_E_UNSUPPORTED, "phi stage: length without a radix pair");
  g.lbs = pair_bits(g, R1);
  const unsigned blocks = (unsigned)((g.nlines + (2 << g.lbs) - 1) >> (g.lbs + 1));
  const unsigned threads = (unsigned)(R1 << g.lbs);
  const size_t shm = ((size_t)2 * g.n * ((1 << g.lbs) + 1) + g.n) * sizeof(double2);
  const double2* tw = reinterpret_cast<const double2*>(p->d_tw_phi);
  const double2* f = reinterpret_cast<const double2*>(mixed);
  p->timing.begin("phi_fft", s);
  switch (g.n) {
#define MIX_BWD(A, B) \
  case A * B: phi_bwd_mix_kernel<A, B><<<blocks, threads, shm, s>>>(g, tw, f, phys); break;
    MIX_PAIRS(MIX_BWD) MIX_WIDE(MIX_BWD)
#undef MIX_BWD
  }
  p->timing.end(s);
  return check("phi_bwd_mix_kernel");
}

mlg_status launch_phi_mix_scalar(const mlg_plan_s* p, int kind, double gamma, double* mixed, hipStream_t s) {
  PhiMix g = phi_mix(p, p->g.dealias != 0);
  int R1, R2;
  if (!mix_pair(p->nphi, true, &R1, &R2)) return fail(MLG_E_UNSUPPORTED, "phi stage: length without a radix pair");
  if (!p->g.dealias) g.mout = p->M;  // every stored order is written, the Nyquist order as zero
  g.lbs = pair_bits(g, R1);
  const unsigned blocks = (unsigned)((g.nlines + (2 << g.lbs) - 1) >> (g.lbs + 1));
  const unsigned threads = (unsigned)(R1 << g.lbs);
  const size_t shm = ((size_t)2 * (g.n << g.lbs) + g.n) * sizeof(double2);
  const double2* tw = reinterpret_cast<const double2*>(p->d_tw_phi);
  double2* f = reinterpret_cast<double2*>(mixed);
  p->timing.begin("phi_fft", s);
  switch (g.n) {
#define MIX_SCALAR(A, B)                                                                                    \
  case A * B:                                                                                               \
    if (kind == MLG_RHS_U2) phi_scalar_mix_kernel<A, B, MLG_RHS_U2><<<blocks, threads, shm, s>>>(g, tw, f, gamma); \
    else phi_scalar_mix_kernel<A, B, MLG_RHS_KPP><<<blocks, threads, shm, s>>>(g, tw, f, gamma);            \
    break;
    MIX_PAIRS(MIX_SCALAR) MIX_WIDE(MIX_SCALAR)
#undef MIX_SCALAR
  }
  p->timing.end(s);
  return check("phi_scalar_mix_kernel");
}

}  // namespace mlg
