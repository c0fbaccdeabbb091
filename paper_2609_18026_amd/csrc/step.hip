// Semi-implicit time stepping of ds/dt = A(s) + L s (Sec. 3.3) on the GPU.
//
// L = nu grad^2 - nu_h (-grad^2)^{p/2} (Eq. dissipation) acts per (m, k) harmonic through the
// truncated horizontal Laplacian: -grad^2 = X_m + kappa^2 with X_m = G_m diag(n(n+1)) / ell^2
// (G_m the exact Gram matrix <Pbar_n, (1-x)^2 Pbar_j>, Eq. del2h-entries).  Every step operator
// is a rational function of -grad^2:
//   FE-BE  out = Phi s + Psi A,       Phi = 1 / (1 - h L),          Psi = h / (1 - h L);
//   AB-CN  out = Phi s + Psi (3 A1 - A0), Phi = (1 + h L) / (1 - h L), Psi = h / (1 - h L),  h = dt / 2
// (Eq. abcn).  The paper factors the banded matrices I - h L per (m, k); here X_m is
// diagonalised once per m on the host, X_m = V diag(lam) V^{-1} with V = L^{-1/2} Q and
// S = L^{1/2} G L^{1/2} / ell^2 = Q diag(lam) Q^T symmetric (n >= max(m, 1), where L > 0).
// The eigenvectors do not depend on kappa, so for all k at once
//   out = V [Phi(lam + kappa^2) (V^{-1} s) + Psi(lam + kappa^2) (V^{-1} a)],
// two FP64 MFMA products per m with the scalar functions applied in between.  For m = 0 the
// n = 0 row of X is (0, b^T) (its column is zero since L_0 = 0), so X is block upper triangular
// and the n = 0 output gains b^T V diag((f(mu) - f(alpha)) / lam) V^{-1} s' terms (divided
// differences, alpha = kappa^2), evaluated in closed form without cancellation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "dev_common.h"
#include "mlg_internal.h"

namespace mlg {
bool sym_eig(int n, std::vector<double>& A, std::vector<double>& w, std::vector<double>& Q);

namespace {

using namespace ::mlg::dev;
using ld = long double;

constexpr int TM = 64;  // rows per block
constexpr int TC = 16;  // complex columns per block
constexpr int TK = 16;  // k depth per LDS stage

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f64_16x16x4f64((a), (b), (c), 0, 0, 0)

__device__ __forceinline__ int kval(int kk, int nz) { return (2 * kk < nz) ? kk : kk - nz; }

// one field of a step
struct StepField {
  const double2* s;
  const double2* a1;
  const double2* a0;   // AB-CN: A^{j-1}; FE-BE: null
  double2* out;
  double2* W;          // packed like the spectra (rows n >= n0 of each m)
  double2* W0;         // m = 0 divided-difference products [j][kk]
};

struct StepArgs {
  StepField f[2];      // one launch steps one or both potentials (nf fields)
  int nf, nrow0;
  const double* fwd;
  const double* bwd;
  const double* lam;
  const double* u;
  const int64_t* qoff;
  const int64_t* loff;
  const int64_t* off;
  int M, nrc, nz, nzc, mode, q;   // mode 0 FE-BE, 1 AB-CN; q = p / 2 (1 without hyperviscosity)
  int gx, gy, gz;                 // tiles: axial column blocks, row blocks (of each field), orders
  double h, nu, nuh, kap0;
};

__device__ __forceinline__ bool active_slot(int kk, int nz, int nzc) {
  const int k = kval(kk, nz);
  const int ka = k < 0 ? -k : k;
  return ka < nzc && !(nz % 2 == 0 && nz > 1 && k == -(nz / 2));
}

// 1 - h L(mu) with L(mu) = -nu mu - nu_h mu^q
__device__ __forceinline__ double denom(const StepArgs& a, double mu) {
  double pw = mu;
  for (int i = 1; i < a.q; ++i) pw *= mu;
  return 1.0 + a.h * (a.nu * mu + a.nuh * pw);
}

// column of an LDS row of a stage: neighbouring rows, which a wavefront reads together, use the two halves of the banks
__device__ __forceinline__ int swz(int row, int col) { return col ^ ((row & 1) << 4); }

// Z = V^{-1} [s | a] per m, then W = Phi Zs + Psi Za (and the m = 0 divided differences).  Both
// potentials go in one launch, the tiles of an order on one XCD (they share its tables), and a
// wavefront whose rows lie past the order's last leaves the products out.  Ten steps at 128 (96) x 64 x 32, where
// one field has 128 blocks for the 256 CUs: 1.40 -> 1.14 ms, the n = 0 row taken along by the second launch.
// FE-BE (MODE 0) has Phi = 1 / D and Psi = h / D, so it needs one product, of s + h a.
template <int MODE>
__global__ __launch_bounds__(256) void step_fwd_kernel(StepArgs a) {
  constexpr int NP = MODE == 1 ? 2 : 1;  // products
  Tile3 tl;
  if (!xcd_tile(a.gx, a.gy * a.nf, a.gz, tl)) return;
  const bool second = tl.y >= a.gy;
  const StepField fd = second ? a.f[1] : a.f[0];
  if (second) tl.y -= a.gy;
  const int m = tl.z;
  if (m >= a.M || m >= a.nrc) return;
  const int n0 = m == 0 ? 1 : 0;
  const int K = a.nrc - m - n0;
  const int j0 = tl.y * TM, kk0 = tl.x * TC;
  if (j0 >= K || kk0 >= a.nz) return;
  const int nz = a.nz;
  const double* __restrict__ A = a.fwd + a.qoff[m];
  const int64_t rb = (a.off[m] + n0) * nz;
  const double2* __restrict__ s = fd.s + rb;
  const double2* __restrict__ p1 = fd.a1 + rb;
  const double2* __restrict__ p0 = MODE == 1 ? fd.a0 + rb : nullptr;
  __shared__ double As[2][TK][TM];
  __shared__ double Bs[2][NP][TK][2 * TC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double4_t acc[NP][2];
#pragma unroll
  for (int p = 0; p < NP; ++p) acc[p][0] = acc[p][1] = double4_t{0.0, 0.0, 0.0, 0.0};
  // raw loads with indices clamped into the operands (no branch around a load); the AB-CN
  // combination 3 A1 - A0 and the zeros outside the operands are formed at the LDS store, so the
  // loads of the next stage stay in flight across this stage's MFMAs
  double ra[4];
  double2 rs, r1, r0v;
  auto load = [&](int k0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = tid + 256 * t;
      const int kr = e >> 6, rr = e & 63;
      const int k = k0 + kr, j = j0 + rr;
      const int kc = k < K ? k : K - 1, jc = j < K ? j : K - 1;
      ra[t] = A[(int64_t)kc * K + jc];
    }
    const int kr = tid >> 4, cc = tid & 15;
    const int k = k0 + kr, kk = kk0 + cc;
    const int kc = k < K ? k : K - 1, kkc = kk < nz ? kk : nz - 1;
    const int64_t i = (int64_t)kc * nz + kkc;
    rs = s[i];
    r1 = p1[i];
    if constexpr (MODE == 1) r0v = p0[i];
  };
  auto store = [&](int buf, int k0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = tid + 256 * t;
      const bool ok = k0 + (e >> 6) < K && j0 + (e & 63) < K;
      As[buf][e >> 6][swz(e >> 6, e & 63)] = ok ? ra[t] : 0.0;
    }
    const int kr = tid >> 4, cc = tid & 15;
    const bool ok = k0 + kr < K && kk0 + cc < nz;
    if constexpr (MODE == 1) {
      Bs[buf][0][kr][swz(kr, cc)] = ok ? rs.x : 0.0;
      Bs[buf][0][kr][swz(kr, TC + cc)] = ok ? rs.y : 0.0;
      Bs[buf][NP - 1][kr][swz(kr, cc)] = ok ? 3.0 * r1.x - r0v.x : 0.0;
      Bs[buf][NP - 1][kr][swz(kr, TC + cc)] = ok ? 3.0 * r1.y - r0v.y : 0.0;
    } else {
      Bs[buf][0][kr][swz(kr, cc)] = ok ? rs.x + a.h * r1.x : 0.0;
      Bs[buf][0][kr][swz(kr, TC + cc)] = ok ? rs.y + a.h * r1.y : 0.0;
    }
  };
  const int nk = (K + TK - 1) / TK;
  const bool rows_in = j0 + wave * 16 < K;
  load(0);
  store(0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load((kt + 1) * TK);
#pragma unroll
    for (int ks = 0; ks < TK; ks += 4) {
      if (!rows_in) break;
      const int kr = ks + (lane >> 4);
      const double av = As[buf][kr][swz(kr, wave * 16 + (lane & 15))];
      acc[0][0] = MFMA(av, Bs[buf][0][kr][swz(kr, lane & 15)], acc[0][0]);
      acc[0][1] = MFMA(av, Bs[buf][0][kr][swz(kr, TC + (lane & 15))], acc[0][1]);
      if constexpr (MODE == 1) {
        acc[NP - 1][0] = MFMA(av, Bs[buf][NP - 1][kr][swz(kr, lane & 15)], acc[NP - 1][0]);
        acc[NP - 1][1] = MFMA(av, Bs[buf][NP - 1][kr][swz(kr, TC + (lane & 15))], acc[NP - 1][1]);
      }
    }
    if (kt + 1 < nk) store(buf ^ 1, (kt + 1) * TK);
    __syncthreads();
  }
  const int kk = kk0 + (lane & 15);
  if (kk >= nz || !active_slot(kk, nz, a.nzc)) return;
  const double kap = a.kap0 * kval(kk, nz);
  const double alpha = kap * kap;
  const double* lam = a.lam + a.loff[m];
  const double Da = denom(a, alpha);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int j = j0 + wave * 16 + (lane >> 4) + 4 * v;
    if (j >= K) continue;
    const double lj = lam[j];
    const double mu = lj + alpha;
    const double D = denom(a, mu);
    const double zsr = acc[0][0][v], zsi = acc[0][1][v];
    double zar = 0.0, zai = 0.0;
    if constexpr (MODE == 1) {
      zar = acc[NP - 1][0][v];
      zai = acc[NP - 1][1][v];
    }
    const double psi = a.h / D, phi = MODE == 1 ? 2.0 / D - 1.0 : 1.0 / D;
    fd.W[rb + (int64_t)j * nz + kk] =
        MODE == 1 ? make_double2(phi * zsr + psi * zar, phi * zsi + psi * zai) : make_double2(phi * zsr, phi * zsi);
    if (m == 0) {
      // (f(mu) - f(alpha)) / lam in closed form: L(mu) - L(alpha) = lam * dl
      double sum = 0.0, mp = 1.0;
      for (int i = 0; i < a.q; ++i) {
        double ap = 1.0;
        for (int t = 0; t < a.q - 1 - i; ++t) ap *= alpha;
        sum += mp * ap;
        mp *= mu;
      }
      const double dl = -a.nu - a.nuh * sum;
      const double inv = a.h * dl / (D * Da);
      const double dphi = (MODE == 1 ? 2.0 : 1.0) * inv;
      const double dpsi = a.h * inv;
      fd.W0[(int64_t)j * nz + kk] =
          MODE == 1 ? make_double2(dphi * zsr + dpsi * zar, dphi * zsi + dpsi * zai) : make_double2(dphi * zsr, dphi * zsi);
    }
  }
}

// m = 0, n = 0: out = Phi(alpha) s0 + Psi(alpha) a0 + sum_j u_j W0[j].  A block takes R0C axial
// columns; the R0S lanes of a column sum every R0S-th j (their loads all in flight at once) and
// the partial sums are added in LDS in a fixed order.
constexpr int R0C = 16;  // columns per block
constexpr int R0S = 16;  // partial sums per column

__device__ __forceinline__ void step_row0(const StepArgs& a, const StepField& fd, int block, double2 (*part)[R0C]) {
  const int c = threadIdx.x % R0C, sl = threadIdx.x / R0C;
  const int kk = block * R0C + c;
  const int K = a.nrc - 1;
  double re = 0.0, im = 0.0;
  if (kk < a.nz) {
#pragma unroll 8
    for (int j = sl; j < K; j += R0S) {
      const double2 w = fd.W0[(int64_t)j * a.nz + kk];
      re += a.u[j] * w.x;
      im += a.u[j] * w.y;
    }
  }
  part[sl][c] = make_double2(re, im);
  __syncthreads();
  if (sl != 0 || kk >= a.nz) return;
  if (!active_slot(kk, a.nz, a.nzc)) {
    fd.out[kk] = make_double2(0.0, 0.0);
    return;
  }
  double sr = 0.0, si = 0.0;
#pragma unroll
  for (int q = 0; q < R0S; ++q) {
    sr += part[q][c].x;
    si += part[q][c].y;
  }
  const double kap = a.kap0 * kval(kk, a.nz);
  const double alpha = kap * kap;
  const double D = denom(a, alpha);
  const double psi = a.h / D;
  const double phi = a.mode == 1 ? 2.0 / D - 1.0 : 1.0 / D;
  const double2 s0 = fd.s[kk];
  double2 v = fd.a1[kk];
  if (fd.a0) v = make_double2(3.0 * v.x - fd.a0[kk].x, 3.0 * v.y - fd.a0[kk].y);
  fd.out[kk] = make_double2(phi * s0.x + psi * v.x + sr, phi * s0.y + psi * v.y + si);
}

// out rows n >= n0 = V W per m; inactive axial slots are zeroed.  The first nrow0 blocks (a multiple of
// 8, so that the others keep their XCDs) take the n = 0 rows of the fields.
__global__ __launch_bounds__(256) void step_bwd_kernel(StepArgs a) {
  __shared__ double As[2][TK][TM];
  __shared__ double Bs[2][TK][2 * TC];
  if ((int)blockIdx.x < a.nrow0) {
    static_assert(sizeof(double2) * R0S * R0C <= sizeof(As), "the partial sums fit in the table stage");
    const int per = (a.nz + R0C - 1) / R0C, f = (int)blockIdx.x / per;
    if (f < a.nf) step_row0(a, f ? a.f[1] : a.f[0], (int)blockIdx.x - f * per, reinterpret_cast<double2(*)[R0C]>(&As[0][0][0]));
    return;
  }
  Tile3 tl;
  if (!xcd_tile(a.gx, a.gy * a.nf, a.gz, tl, blockIdx.x - a.nrow0)) return;
  const bool second = tl.y >= a.gy;
  const StepField fd = second ? a.f[1] : a.f[0];
  if (second) tl.y -= a.gy;
  const int m = tl.z;
  if (m >= a.M || m >= a.nrc) return;
  const int n0 = m == 0 ? 1 : 0;
  const int K = a.nrc - m - n0;
  const int r0 = tl.y * TM, kk0 = tl.x * TC;
  if (r0 >= K || kk0 >= a.nz) return;
  const int nz = a.nz;
  const double* __restrict__ A = a.bwd + a.qoff[m];
  const int64_t rb = (a.off[m] + n0) * nz;
  const double2* __restrict__ Wm = fd.W + rb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double4_t acc[2];
  acc[0] = acc[1] = double4_t{0.0, 0.0, 0.0, 0.0};
  // raw loads with clamped indices, zeros applied at the LDS store (as in step_fwd_kernel)
  double ra[4];
  double2 rbv;
  auto load = [&](int k0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = tid + 256 * t;
      const int kr = e >> 6, rr = e & 63;
      const int k = k0 + kr, r = r0 + rr;
      const int kc = k < K ? k : K - 1, rc = r < K ? r : K - 1;
      ra[t] = A[(int64_t)kc * K + rc];
    }
    const int kr = tid >> 4, cc = tid & 15;
    const int k = k0 + kr, kk = kk0 + cc;
    const int kc = k < K ? k : K - 1, kkc = kk < nz ? kk : nz - 1;
    rbv = Wm[(int64_t)kc * nz + kkc];
  };
  auto store = [&](int buf, int k0) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int e = tid + 256 * t;
      const bool ok = k0 + (e >> 6) < K && r0 + (e & 63) < K;
      As[buf][e >> 6][swz(e >> 6, e & 63)] = ok ? ra[t] : 0.0;
    }
    const int kr = tid >> 4, cc = tid & 15;
    const bool ok = k0 + kr < K && kk0 + cc < nz;
    Bs[buf][kr][swz(kr, cc)] = ok ? rbv.x : 0.0;
    Bs[buf][kr][swz(kr, TC + cc)] = ok ? rbv.y : 0.0;
  };
  const int nk = (K + TK - 1) / TK;
  const bool rows_in = r0 + wave * 16 < K;
  load(0);
  store(0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) load((kt + 1) * TK);
#pragma unroll
    for (int ks = 0; ks < TK; ks += 4) {
      if (!rows_in) break;
      const int kr = ks + (lane >> 4);
      const double av = As[buf][kr][swz(kr, wave * 16 + (lane & 15))];
      acc[0] = MFMA(av, Bs[buf][kr][swz(kr, lane & 15)], acc[0]);
      acc[1] = MFMA(av, Bs[buf][kr][swz(kr, TC + (lane & 15))], acc[1]);
    }
    if (kt + 1 < nk) store(buf ^ 1, (kt + 1) * TK);
    __syncthreads();
  }
  const int kk = kk0 + (lane & 15);
  if (kk >= nz) return;
  const bool act = active_slot(kk, nz, a.nzc);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = r0 + wave * 16 + (lane >> 4) + 4 * v;
    if (r >= K) continue;
    fd.out[rb + (int64_t)r * nz + kk] = act ? make_double2(acc[0][v], acc[1][v]) : make_double2(0.0, 0.0);
  }
}

// N_z = 1: one column per field, as matrix-vector products (dev_common.h; the tiles above would hold one
// column of 16, and their K stages run one after the other).  N_r = 768, 2 orders, one field: the first
// product 56 -> 8.0 us, the second 36 -> 5.8 us (with the n = 0 row, 6 us before).
template <int GU>
__global__ __launch_bounds__(GT) void step_fwd1_kernel(StepArgs a) {
  constexpr int GC = GK * GU, GV = (GC + GT - 1) / GT;  // terms a chunk, vector entries a thread
  __shared__ double2 xs[GC], xa[GC];
  const int m = blockIdx.y;
  const StepField fd = blockIdx.z ? a.f[1] : a.f[0];
  const int n0 = m == 0 ? 1 : 0;
  const int K = a.nrc - m - n0;
  const int j0 = blockIdx.x * GR;
  if (j0 >= K) return;
  const int q = threadIdx.x % (GR / 2), g = threadIdx.x / (GR / 2);
  const int jl = j0 + 2 * q;
  // the pair (K - 1, K) reads on into the next table row (the tables end in a spare entry)
  const double* __restrict__ A = a.fwd + a.qoff[m] + min(jl, K - 1);
  const int64_t rb = a.off[m] + n0;
  const double2* __restrict__ s = fd.s + rb;
  const double2* __restrict__ p1 = fd.a1 + rb;
  const double2* __restrict__ p0 = (fd.a0 ? fd.a0 : fd.a1) + rb;
  const bool ab = fd.a0 != nullptr;
  const double c1 = ab ? 3.0 : 1.0;
  double z[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // V^{-1} s and V^{-1} a of row jl, of row jl + 1
  for (int k0 = 0; k0 < K; k0 += GC) {
    double2 sv[GV], x1[GV], x0[GV];
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      const int k = k0 + t * GT + threadIdx.x;
      sv[t] = k < K ? s[k] : make_double2(0.0, 0.0);
      x1[t] = k < K ? p1[k] : make_double2(0.0, 0.0);
      x0[t] = ab && k < K ? p0[k] : make_double2(0.0, 0.0);  // FE-BE has none (times a zero, an infinity would leave a NaN)
    }
    dpair v[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      v[u] = *reinterpret_cast<const dpair*>(A + (int64_t)min(k0 + g + GK * u, K - 1) * K);
    }
    if (k0 > 0) __syncthreads();
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      if (GC < GT && (int)threadIdx.x >= GC) break;
      xs[t * GT + threadIdx.x] = sv[t];
      xa[t * GT + threadIdx.x] = make_double2(c1 * x1[t].x - x0[t].x, c1 * x1[t].y - x0[t].y);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const double2 sv = xs[g + GK * u], av = xa[g + GK * u];
      z[0] += v[u].x * sv.x;
      z[1] += v[u].x * sv.y;
      z[2] += v[u].x * av.x;
      z[3] += v[u].x * av.y;
      z[4] += v[u].y * sv.x;
      z[5] += v[u].y * sv.y;
      z[6] += v[u].y * av.x;
      z[7] += v[u].y * av.y;
    }
  }
  block_sum(z);
  if (threadIdx.x >= GR / 2) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = jl + h;
    if (j >= K) continue;
    const double zsr = z[4 * h], zsi = z[4 * h + 1], zar = z[4 * h + 2], zai = z[4 * h + 3];
    const double lj = a.lam[a.loff[m] + j];  // the only slot is k = 0: kappa = 0
    const double D = denom(a, lj);
    const double psi = a.h / D;
    const double phi = a.mode == 1 ? 2.0 / D - 1.0 : 1.0 / D;
    fd.W[rb + j] = make_double2(phi * zsr + psi * zar, phi * zsi + psi * zai);
    if (m == 0) {
      // the divided differences of step_fwd_kernel at alpha = 0
      double mp = 1.0;
      for (int i = 1; i < a.q; ++i) mp *= lj;
      const double inv = a.h * (-a.nu - a.nuh * mp) / D;
      const double dphi = (a.mode == 1 ? 2.0 : 1.0) * inv, dpsi = a.h * inv;
      fd.W0[j] = make_double2(dphi * zsr + dpsi * zar, dphi * zsi + dpsi * zai);
    }
  }
}

// rows n >= n0 of every order; the block past the last row block of order 0 takes its n = 0 row
template <int GU>
__global__ __launch_bounds__(GT) void step_bwd1_kernel(StepArgs a) {
  constexpr int GC = GK * GU, GV = (GC + GT - 1) / GT;  // terms a chunk, vector entries a thread
  __shared__ double2 xs[GC];
  const int m = blockIdx.y;
  const StepField fd = blockIdx.z ? a.f[1] : a.f[0];
  const int n0 = m == 0 ? 1 : 0;
  const int K = a.nrc - m - n0;
  if (m == 0 && blockIdx.x == gridDim.x - 1) {
    const int t = threadIdx.x;
    double z[2] = {0.0, 0.0};
    for (int j = t; j < K; j += GT) {
      const double2 w = fd.W0[j];
      z[0] += a.u[j] * w.x;
      z[1] += a.u[j] * w.y;
    }
#pragma unroll
    for (int d = 1; d < GR / 2; d *= 2) {  // the lanes of a group, then (block_sum) the groups
      z[0] += __shfl_xor(z[0], d, 64);
      z[1] += __shfl_xor(z[1], d, 64);
    }
    block_sum(z);
    if (t != 0) return;
    // alpha = 0: D = 1
    const double2 s0 = fd.s[0];
    double2 v = fd.a1[0];
    if (fd.a0) v = make_double2(3.0 * v.x - fd.a0[0].x, 3.0 * v.y - fd.a0[0].y);
    fd.out[0] = make_double2(s0.x + a.h * v.x + z[0], s0.y + a.h * v.y + z[1]);
    return;
  }
  const int r0 = blockIdx.x * GR;
  if (r0 >= K) return;
  const int q = threadIdx.x % (GR / 2), g = threadIdx.x / (GR / 2);
  const int row = r0 + 2 * q;
  const double* __restrict__ A = a.bwd + a.qoff[m] + min(row, K - 1);
  const int64_t rb = a.off[m] + n0;
  const double2* __restrict__ W = fd.W + rb;
  double z[4] = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += GC) {
    double2 wv[GV];
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      const int k = k0 + t * GT + threadIdx.x;
      wv[t] = k < K ? W[k] : make_double2(0.0, 0.0);
    }
    dpair v[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      v[u] = *reinterpret_cast<const dpair*>(A + (int64_t)min(k0 + g + GK * u, K - 1) * K);
    }
    if (k0 > 0) __syncthreads();
#pragma unroll
    for (int t = 0; t < GV; ++t)
      if (GC >= GT || (int)threadIdx.x < GC) xs[t * GT + threadIdx.x] = wv[t];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const double2 w = xs[g + GK * u];
      z[0] += v[u].x * w.x;
      z[1] += v[u].x * w.y;
      z[2] += v[u].y * w.x;
      z[3] += v[u].y * w.y;
    }
  }
  block_sum(z);
  if (threadIdx.x >= GR / 2) return;
  if (row < K) fd.out[rb + row] = make_double2(z[0], z[1]);
  if (row + 1 < K) fd.out[rb + row + 1] = make_double2(z[2], z[3]);
}

// ---------------------------------------------------------------- adaptive modal filter
// Sec. 3.3: every coefficient whose normalised index zeta = max(n / N_r^c, m / N_phi^c,
// |k| / N_z^c) exceeds zeta_c is multiplied by exp(-eps ((zeta - zeta_c) / (1 - zeta_c))^8); eps
// follows the fraction f of sum |s|^2 held above zeta_c: target eps_max clip((f - tau) / tau, 0, 1),
// relaxed as eps <- eps + r (target - eps), one state per field.  Two launches for one or both fields (grid y):
// partial sums over a fixed number of blocks (so the order never depends on the device), which also set the old eps aside;
// and the scaling, every block of which adds the partial sums in their order and forms the new eps for itself (block 0
// stores it), and ends at once while eps is zero (its factors are then one).  The kernel boundary publishes the sums: where the last
// block to arrive added them, its release and acquire wrote the dirty lines of the L2 back.  One field at 128^3: three launches
// 15.7 us, the last block 19.4, now 14.3; a step of two fields of 96 kept rows x 64 x 32: 8 us less.  The state stays on
// the device: a time loop never waits for it.
struct FilterArgs {
  double2* spec[2];
  const int32_t* row_m;
  const int64_t* off;
  int64_t rows;
  int nz, nzc, nrc, M;
  double zc, tau, eps_max, relax;
  double* state;  // [eps_0, eps_1, f_0, f_1]
  double2* part;  // per slot: FILTER_BLOCKS x (tail, total)
  double* old;    // per slot: eps before this application
  int slot;       // of field 0
};

__device__ __forceinline__ double filter_zeta(const FilterArgs& a, int64_t row, int kk) {
  const int m = a.row_m[row];
  const int n = m + (int)(row - a.off[m]);
  const int k = (2 * kk < a.nz) ? kk : kk - a.nz;
  const double zr = (double)n / a.nrc, zp = (double)m / a.M, zz = (double)(k < 0 ? -k : k) / a.nzc;
  return fmax(fmax(zr, zp), zz);
}

// Tree sum of 256 (tail, total) pairs by each wavefront for itself, in every lane: halves of 128, 64, ... 1 are added
__device__ __forceinline__ double2 filter_tree(const double2* v) {
  const int l = threadIdx.x & 63;
  double2 s = dev::cadd(dev::cadd(v[l], v[l + 128]), dev::cadd(v[l + 64], v[l + 192]));
#pragma unroll
  for (int h = 32; h > 0; h >>= 1) {
    s.x += __shfl_down(s.x, h, 64);
    s.y += __shfl_down(s.y, h, 64);
  }
  return make_double2(__shfl(s.x, 0, 64), __shfl(s.y, 0, 64));
}

__global__ __launch_bounds__(256) void filter_sums_kernel(FilterArgs a) {
  __shared__ double2 sums[256];
  const int t = threadIdx.x, slot = a.slot + blockIdx.y;
  const double2* __restrict__ spec = blockIdx.y ? a.spec[1] : a.spec[0];
  double tail = 0.0, total = 0.0;
  const int64_t n = a.rows * a.nz;
  for (int64_t e = (int64_t)blockIdx.x * 256 + t; e < n; e += (int64_t)FILTER_BLOCKS * 256) {
    const int64_t row = e / a.nz;
    const int kk = (int)(e - row * a.nz);
    const double2 v = spec[e];
    const double w = v.x * v.x + v.y * v.y;
    total += w;
    if (filter_zeta(a, row, kk) > a.zc) tail += w;
  }
  sums[t] = make_double2(tail, total);
  __syncthreads();
  const double2 sum = filter_tree(sums);
  if (t == 0) {
    a.part[slot * FILTER_BLOCKS + blockIdx.x] = sum;
    if (blockIdx.x == 0) a.old[slot] = a.state[slot];
  }
}

__global__ __launch_bounds__(256) void filter_apply_kernel(FilterArgs a) {
  static_assert(FILTER_BLOCKS == 256, "the partial sums of a field are one tree");
  const int t = threadIdx.x, slot = a.slot + blockIdx.y;
  const double2 sum = filter_tree(a.part + slot * FILTER_BLOCKS);
  const double f = sum.y > 0.0 ? sum.x / sum.y : 0.0;
  const double target = a.eps_max * fmin(fmax((f - a.tau) / a.tau, 0.0), 1.0);
  const double eps = a.old[slot] + a.relax * (target - a.old[slot]);
  if (blockIdx.x == 0 && t == 0) {
    a.state[slot] = eps;
    a.state[2 + slot] = f;
  }
  if (eps == 0.0) return;
  double2* __restrict__ spec = blockIdx.y ? a.spec[1] : a.spec[0];
  const int64_t n = a.rows * a.nz;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    const int64_t row = e / a.nz;
    const int kk = (int)(e - row * a.nz);
    const double zeta = filter_zeta(a, row, kk);
    if (zeta > a.zc) {
      const double x = (zeta - a.zc) / (1.0 - a.zc);
      const double x2 = x * x, x4 = x2 * x2;
      const double sg = exp(-eps * (x4 * x4));
      const double2 v = spec[e];
      spec[e] = make_double2(v.x * sg, v.y * sg);
    }
  }
}

}  // namespace

mlg_status step_setup(mlg_plan_s* p, const mlg_dissip* d) {
  const int nrc = p->nrc, M = p->M, nz = p->nz;
  const int Mm = std::min(M, nrc);
  const ld ell2 = (ld)p->g.ell * (ld)p->g.ell;
  std::vector<int64_t> qoff(M + 1, 0), loff(M + 1, 0);
  for (int m = 0; m < M; ++m) {
    const int Kp = m < Mm ? nrc - m - (m == 0 ? 1 : 0) : 0;
    qoff[m + 1] = qoff[m] + (int64_t)Kp * Kp;
    loff[m + 1] = loff[m] + Kp;
  }
  std::vector<double> fwd(qoff[M] + 1), bwd(qoff[M] + 1);  // with a spare entry: see step_fwd1_kernel
  std::vector<double> lam(std::max<int64_t>(loff[M], 1)), u(std::max(nrc - 1, 1), 0.0);
  std::atomic<int> next{0};
  std::atomic<bool> failed{false};
  auto work = [&]() {
    for (int m = next++; m < Mm; m = next++) {
      const int n0 = m == 0 ? 1 : 0;
      const int K = nrc - m - n0;
      if (K <= 0) continue;
      auto eps = [&](int n) -> ld {
        return (n <= m || n <= 0) ? 0 : sqrtl((ld)(n * n - m * m) / (ld)(4 * n * n - 1));
      };
      auto gram = [&](int n, int nj) -> ld {  // G_{n, nj} (pentadiagonal, symmetric)
        const int lo = std::min(n, nj), hi = std::max(n, nj);
        if (hi == lo) return 1 + eps(lo) * eps(lo) + eps(lo + 1) * eps(lo + 1);
        if (hi == lo + 1) return -2 * eps(hi);
        if (hi == lo + 2) return eps(lo + 1) * eps(lo + 2);
        return 0;
      };
      std::vector<ld> sq(K);
      for (int i = 0; i < K; ++i) {
        const ld n = m + n0 + i;
        sq[i] = sqrtl(n * (n + 1));
      }
      std::vector<double> S((size_t)K * K, 0.0), w, Q;
      for (int i = 0; i < K; ++i)
        for (int j = std::max(0, i - 2); j <= std::min(K - 1, i + 2); ++j)
          S[(size_t)i * K + j] = (double)(sq[i] * gram(m + n0 + i, m + n0 + j) * sq[j] / ell2);
      if (!sym_eig(K, S, w, Q)) {
        failed = true;
        continue;
      }
      double* F = fwd.data() + qoff[m];
      double* B = bwd.data() + qoff[m];
      for (int i = 0; i < K; ++i)
        for (int j = 0; j < K; ++j) {
          F[(size_t)i * K + j] = (double)(Q[(size_t)i * K + j] * sq[i]);
          B[(size_t)j * K + i] = (double)(Q[(size_t)i * K + j] / sq[i]);
        }
      std::copy(w.begin(), w.end(), lam.begin() + loff[m]);
      if (m == 0) {
        // b_n = X_{0 n} = G_{0 n} n (n + 1) / ell^2 (n = 1, 2); u_j = sum_n b_n V[n][j]
        for (int j = 0; j < K; ++j) {
          ld acc = 0;
          for (int i = 0; i < std::min(K, 2); ++i) {
            const int n = 1 + i;
            const ld b = gram(0, n) * (ld)n * (n + 1) / ell2;
            acc += b * (ld)Q[(size_t)i * K + j] / sq[i];
          }
          u[j] = (double)acc;
        }
      }
    }
  };
  const unsigned hw = std::max(1u, std::min(32u, std::thread::hardware_concurrency()));
  const int nthreads = (int)std::min<unsigned>(hw, (unsigned)std::max(Mm, 1));
  std::vector<std::thread> pool;
  for (int t = 1; t < nthreads; ++t) pool.emplace_back(work);
  work();
  for (auto& t : pool) t.join();
  if (failed) return fail(MLG_E_DEVICE, "step setup: eigen-decomposition did not converge");

  double** bufs[] = {&p->d_step_fwd, &p->d_step_bwd, &p->d_step_lam, &p->d_step_u, &p->d_step_w};
  for (double** q : bufs)
    if (*q) (void)hipFree(*q);
  if (p->d_step_qoff) (void)hipFree(p->d_step_qoff);
  if (p->d_step_loff) (void)hipFree(p->d_step_loff);
  if (p->d_logf) (void)hipFree(p->d_logf);
  p->d_logf = nullptr;
  p->d_step_fwd = p->d_step_bwd = p->d_step_lam = p->d_step_u = p->d_step_w = nullptr;
  p->d_step_qoff = p->d_step_loff = nullptr;
  p->step_ready = false;
  auto upl = [&](auto** dst, const auto& v) -> mlg_status {
    using T = typename std::decay_t<decltype(v)>::value_type;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(dst), std::max<size_t>(v.size(), 1) * sizeof(T));
    if (e != hipSuccess) { *dst = nullptr; return fail(MLG_E_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e)); }
    if (!v.empty() && hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
      return fail(MLG_E_DEVICE, "hipMemcpy failed");
    return MLG_OK;
  };
  mlg_status st;
  if ((st = upl(&p->d_step_fwd, fwd)) || (st = upl(&p->d_step_bwd, bwd)) || (st = upl(&p->d_step_lam, lam)) ||
      (st = upl(&p->d_step_u, u)) || (st = upl(&p->d_step_qoff, qoff)) || (st = upl(&p->d_step_loff, loff)))
    return st;
  const size_t wel = ((size_t)p->tau + std::max(nrc - 1, 1)) * nz * 2;  // one field
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&p->d_step_w), wel * sizeof(double));
  if (e != hipSuccess) {
    p->d_step_w = nullptr;
    return fail(MLG_E_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e));
  }
  int maxk = 0;
  for (int m = 0; m < Mm; ++m) maxk = std::max(maxk, nrc - m - (m == 0 ? 1 : 0));
  p->step_maxk = maxk;
  p->step_dt = d->dt;
  p->step_nu = d->nu;
  p->step_nuh = d->nu_h;
  p->step_q = d->nu_h > 0 ? d->p / 2 : 1;
  // the dissipation of the logarithmic proxies, a constant forcing of the regular parts (Eq. logproxy)
  std::vector<double> lf;
  proxy_forcing(p, d->nu, d->nu_h, p->step_q, lf);
  if ((st = upl(&p->d_logf, lf))) return st;
  p->step_ready = true;
  return MLG_OK;
}

mlg_status launch_step(const mlg_plan_s* p, int mode, int which, const double* s, const double* a1, const double* a0,
                       double* out, hipStream_t st) {
  return launch_steps(p, 1, mode, which, &s, &a1, &a0, &out, nullptr, st);
}

mlg_status launch_steps(const mlg_plan_s* p, int nf, int mode, int which, const double* const* s,
                        const double* const* a1, const double* const* a0, double* const* out, double* scratch,
                        hipStream_t st) {
  StepArgs a{};
  const size_t w_len = (size_t)p->tau * p->nz;
  if (nf > 1 && !scratch) return fail(MLG_E_ARG, "step: a second field needs scratch");
  a.nf = nf;
  for (int i = 0; i < nf; ++i) {
    StepField& f = a.f[i];
    f.s = reinterpret_cast<const double2*>(s[i]);
    f.a1 = reinterpret_cast<const double2*>(a1[i]);
    f.a0 = mode == 1 ? reinterpret_cast<const double2*>(a0[i]) : nullptr;
    f.out = reinterpret_cast<double2*>(out[i]);
    f.W = reinterpret_cast<double2*>(i ? scratch : p->d_step_w);
    f.W0 = f.W + w_len;
  }
  a.fwd = p->d_step_fwd;
  a.bwd = p->d_step_bwd;
  a.lam = p->d_step_lam;
  a.u = p->d_step_u;
  a.qoff = p->d_step_qoff;
  a.loff = p->d_step_loff;
  a.off = p->d_goff;
  a.M = p->M;
  a.nrc = p->nrc;
  a.nz = p->nz;
  a.nzc = p->nzc;
  a.mode = mode;
  a.q = p->step_q;
  a.h = (mode == 1 || which == 0) ? p->step_dt / 2 : p->step_dt;
  a.nu = p->step_nu;
  a.nuh = p->step_nuh;
  a.kap0 = 2.0 * M_PI / p->g.lz;
  p->timing.begin("step", st);
  if (p->nz == 1) {
    const unsigned tiles = (unsigned)((p->step_maxk + GR - 1) / GR), orders = (unsigned)std::min(p->M, p->nrc);
    const dim3 gf(tiles, orders, (unsigned)nf), gb(tiles + 1, orders, (unsigned)nf);
    switch (gemv_unroll(p->step_maxk)) {
#define STEP1(U)                                                   \
  if (tiles) step_fwd1_kernel<U><<<gf, GT, 0, st>>>(a);            \
  step_bwd1_kernel<U><<<gb, GT, 0, st>>>(a);                       \
  break;
      case 2: STEP1(2)
      case 4: STEP1(4)
      case 8: STEP1(8)
      default: STEP1(16)
#undef STEP1
    }
    p->timing.end(st);
    const hipError_t e1 = hipGetLastError();
    if (e1 != hipSuccess) return fail(MLG_E_DEVICE, std::string("step kernels: ") + hipGetErrorString(e1));
    return MLG_OK;
  }
  a.gx = (p->nz + TC - 1) / TC;
  a.gy = std::max(1, (p->step_maxk + TM - 1) / TM);
  a.gz = std::min(p->M, p->nrc);
  a.nrow0 = (nf * ((p->nz + R0C - 1) / R0C) + 7) / 8 * 8;
  const unsigned tiles = p->step_maxk > 0 ? xcd_blocks(a.gx, a.gy * nf, a.gz) : 0;  // none: the n = 0 row alone
  if (tiles && mode == 1) step_fwd_kernel<1><<<tiles, 256, 0, st>>>(a);
  else if (tiles) step_fwd_kernel<0><<<tiles, 256, 0, st>>>(a);
  step_bwd_kernel<<<a.nrow0 + tiles, 256, 0, st>>>(a);
  p->timing.end(st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string("step kernels: ") + hipGetErrorString(e));
  return MLG_OK;
}

__global__ __launch_bounds__(256) void richardson_kernel(const double* half, const double* full, double* out,
                                                         int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = 2.0 * half[i] - full[i];
}

mlg_status launch_richardson(const mlg_plan_s* p, const double* half, const double* full, double* out,
                             hipStream_t st) {
  const int64_t n = 2 * p->tau * p->nz;
  p->timing.begin("step", st);
  richardson_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(half, full, out, n);
  p->timing.end(st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string("richardson_kernel: ") + hipGetErrorString(e));
  return MLG_OK;
}

mlg_status launch_filter(const mlg_plan_s* p, int slot, int nf, double* const* spec, hipStream_t st) {
  FilterArgs a{};
  for (int i = 0; i < nf; ++i) a.spec[i] = reinterpret_cast<double2*>(spec[i]);
  a.row_m = p->d_row_m;
  a.off = p->d_goff;
  a.rows = p->tau;
  a.nz = p->nz;
  a.nzc = p->nzc;
  a.nrc = p->nrc;
  a.M = p->M;
  a.zc = p->filter_zc;
  a.tau = p->filter_tau;
  a.eps_max = p->filter_epsmax;
  a.relax = p->filter_relax;
  a.state = p->d_filter;
  a.part = reinterpret_cast<double2*>(p->d_filter + 4);
  a.old = p->d_filter + 4 + 4 * FILTER_BLOCKS;
  a.slot = slot;
  const int64_t n = a.rows * a.nz;
  // a block adds the partial sums before it scales: 4 blocks a CU, up to 16 where a thread would take more than 8 entries (with 16
  // everywhere 128^3 takes 15.9 us for 14.3; with 4 everywhere 256^3 87 for 84.5)
  const int64_t most = std::max<int64_t>(1024, std::min<int64_t>(4096, n / 2048));
  const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, most);
  p->timing.begin("filter", st);
  filter_sums_kernel<<<dim3(FILTER_BLOCKS, nf), 256, 0, st>>>(a);
  filter_apply_kernel<<<dim3(blocks, nf), 256, 0, st>>>(a);
  p->timing.end(st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string("filter kernels: ") + hipGetErrorString(e));
  return MLG_OK;
}

}  // namespace mlg
