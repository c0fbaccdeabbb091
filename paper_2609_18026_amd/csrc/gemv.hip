// Radial products of 2D plans (N_z = 1): every azimuthal order multiplies its table by one complex column, so
// the MFMA tiles of gemm_fold.hip (64 real columns) would be nearly empty and their K loop, one LDS stage
// after the other, serial.  Here they are matrix-vector products (dev_common.h) on the lanes of a
// whole block, partial sums meeting in a fixed order, folded over the node symmetry as in gemm_fold.hip and
// for odd N_r too (the middle node is its own mirror).  The axial transform of N_z = 1 is the
// identity: these kernels read and write the spectrum itself.
// Bound by the latency of one launch and, from about N_r = 512, by the tables, half of which are read once.
// N_r = 768, 2 orders: backward 37 -> 5.1 us, forward 63 -> 4.4 us, and no z transforms (4.7 us each).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "dev_common.h"
#include "mlg_internal.h"

namespace mlg {
namespace {

using namespace ::mlg::dev;

struct Gemv2D {
  const double* A;     // backward: Pbar [m][n-m][i]; forward: w Pbar [m][i][n-m]
  const double2* x;    // backward: spectrum; forward: harmonics [m][i]
  double2* y;
  const int64_t* off;
  int nr, nrc, orders; // orders the two-thirds mask (or the plan) keeps
};

// f(i) = E + O, f(N-1-i) = E - O for the half nodes i (the middle node of an odd N_r once)
template <int GU>
__global__ __launch_bounds__(GT) void gemv_bwd_kernel(Gemv2D a) {
  constexpr int GC = GK * GU, GV = (GC + GT - 1) / GT;  // degrees a chunk, vector entries a thread
  __shared__ double2 xs[GC];
  const int m = blockIdx.y, nr = a.nr, half = (nr + 1) / 2;
  const int q = threadIdx.x % (GR / 2), g = threadIdx.x / (GR / 2);
  const int i = blockIdx.x * GR + 2 * q;
  const int K = a.nrc > m ? a.nrc - m : 0;
  const double* __restrict__ A = a.A + a.off[m] * nr + min(i, half - 1);  // entry i + 1 <= half lies in the row
  const double2* __restrict__ x = a.x + a.off[m];
  double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // E and O of node i, of node i + 1
  for (int c0 = 0; c0 < K; c0 += GC) {
    double2 xv[GV];
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      const int k = c0 + t * GT + threadIdx.x;
      xv[t] = k < K ? x[k] : make_double2(0.0, 0.0);
    }
    dpair e[GU / 2], o[GU / 2];
#pragma unroll
    for (int u = 0; u < GU / 2; ++u) {
      const int j = c0 + 2 * (g + GK * u);  // pairs of degrees
      e[u] = *reinterpret_cast<const dpair*>(A + (int64_t)min(j, K - 1) * nr);
      o[u] = *reinterpret_cast<const dpair*>(A + (int64_t)min(j + 1, K - 1) * nr);
    }
    if (c0 > 0) __syncthreads();  // the last chunk's reads of xs are done
#pragma unroll
    for (int t = 0; t < GV; ++t)
      if (GC >= GT || (int)threadIdx.x < GC) xs[t * GT + threadIdx.x] = xv[t];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GU / 2; ++u) {
      const double2 xe = xs[2 * (g + GK * u)], xo = xs[2 * (g + GK * u) + 1];
      acc[0] += e[u].x * xe.x;
      acc[1] += e[u].x * xe.y;
      acc[2] += o[u].x * xo.x;
      acc[3] += o[u].x * xo.y;
      acc[4] += e[u].y * xe.x;
      acc[5] += e[u].y * xe.y;
      acc[6] += o[u].y * xo.x;
      acc[7] += o[u].y * xo.y;
    }
  }
  block_sum(acc);
  if (threadIdx.x >= GR / 2) return;
  double2* __restrict__ y = a.y + (int64_t)m * nr;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int n = i + h;
    if (n >= half) continue;
    y[n] = make_double2(acc[4 * h] + acc[4 * h + 2], acc[4 * h + 1] + acc[4 * h + 3]);
    if (2 * n + 1 != nr) y[nr - 1 - n] = make_double2(acc[4 * h] - acc[4 * h + 2], acc[4 * h + 1] - acc[4 * h + 3]);
  }
}

// even n - m take the sums of a node and its mirror, odd ones the differences; a lane's two rows are the pair.
// Orders past the kept ones are written as zero.
template <int GU>
__global__ __launch_bounds__(GT) void gemv_fwd_kernel(Gemv2D a) {
  constexpr int GC = GK * GU, GV = (GC + GT - 1) / GT;  // terms a chunk, vector entries a thread
  __shared__ double2 xs[GC], xd[GC];
  const int m = blockIdx.y, nr = a.nr, half = (nr + 1) / 2;
  const int q = threadIdx.x % (GR / 2), g = threadIdx.x / (GR / 2);
  const int K = a.nrc > m ? a.nrc - m : 0;
  const int j0 = blockIdx.x * GR, j = j0 + 2 * q;
  if (j0 >= K) return;
  double2* __restrict__ y = a.y + a.off[m];
  if (m >= a.orders) {
    if ((int)threadIdx.x < GR && j0 + (int)threadIdx.x < K) y[j0 + threadIdx.x] = make_double2(0.0, 0.0);
    return;
  }
  // the pair (K - 1, K) of an odd K reads on into node i + 1, i < half: inside the table
  const double* __restrict__ A = a.A + a.off[m] * nr + min(j, (K - 1) / 2 * 2);
  const double2* __restrict__ x = a.x + (int64_t)m * nr;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c0 = 0; c0 < half; c0 += GC) {
    double2 xv[GV], xw[GV];
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      const int i = c0 + t * GT + threadIdx.x;
      xv[t] = i < half ? x[i] : make_double2(0.0, 0.0);
      xw[t] = i < half ? x[nr - 1 - i] : make_double2(0.0, 0.0);
    }
    dpair v[GU];
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      v[u] = *reinterpret_cast<const dpair*>(A + (int64_t)min(c0 + g + GK * u, half - 1) * K);
    }
    if (c0 > 0) __syncthreads();
#pragma unroll
    for (int t = 0; t < GV; ++t) {
      const int e = t * GT + threadIdx.x;
      if (GC < GT && e >= GC) break;
      const bool mid = 2 * (c0 + e) + 1 == nr;  // the middle node counts once in the sum and not in the difference
      xs[e] = mid ? xv[t] : cadd(xv[t], xw[t]);
      xd[e] = mid ? make_double2(0.0, 0.0) : csub(xv[t], xw[t]);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GU; ++u) {
      const double2 s = xs[g + GK * u], d = xd[g + GK * u];
      acc[0] += v[u].x * s.x;
      acc[1] += v[u].x * s.y;
      acc[2] += v[u].y * d.x;
      acc[3] += v[u].y * d.y;
    }
  }
  block_sum(acc);
  if (threadIdx.x >= GR / 2) return;
  if (j < K) y[j] = make_double2(acc[0], acc[1]);
  if (j + 1 < K) y[j + 1] = make_double2(acc[2], acc[3]);
}

mlg_status check(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
  return MLG_OK;
}

}  // namespace

bool gemv_ok(const mlg_plan_s* p) { return p->nz == 1 && p->prec == MLG_FP64 && p->use_fold; }

mlg_status launch_gemv(const mlg_plan_s* p, int dir, const double* x, double* y, int orders, hipStream_t s) {
  Gemv2D a{};
  a.A = dir > 0 ? p->d_Pb : p->d_Pf;
  a.x = reinterpret_cast<const double2*>(x);
  a.y = reinterpret_cast<double2*>(y);
  a.off = p->d_goff;
  a.nr = p->nr;
  a.nrc = p->nrc;
  a.orders = std::min(orders, p->M);
  const int half = (p->nr + 1) / 2;
  p->timing.begin("radial_gemm", s);
  if (dir > 0) {
    const dim3 grid((unsigned)((half + GR - 1) / GR), (unsigned)a.orders);
    switch (gemv_unroll(p->nrc)) {
      case 2: gemv_bwd_kernel<2><<<grid, GT, 0, s>>>(a); break;
      case 4: gemv_bwd_kernel<4><<<grid, GT, 0, s>>>(a); break;
      case 8: gemv_bwd_kernel<8><<<grid, GT, 0, s>>>(a); break;
      default: gemv_bwd_kernel<16><<<grid, GT, 0, s>>>(a);
    }
  } else {
    const dim3 grid((unsigned)((p->nrc + GR - 1) / GR), (unsigned)p->M);
    switch (gemv_unroll(half)) {
      case 2: gemv_fwd_kernel<2><<<grid, GT, 0, s>>>(a); break;
      case 4: gemv_fwd_kernel<4><<<grid, GT, 0, s>>>(a); break;
      case 8: gemv_fwd_kernel<8><<<grid, GT, 0, s>>>(a); break;
      default: gemv_fwd_kernel<16><<<grid, GT, 0, s>>>(a);
    }
  }
  p->timing.end(s);
  return check("gemv kernel");
}

}  // namespace mlg
