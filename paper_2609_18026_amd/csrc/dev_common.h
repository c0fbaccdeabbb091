// Device-side complex helpers shared by the kernel sources.
#pragma once

#include <hip/hip_runtime.h>

namespace mlg {
namespace dev {

typedef double double4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// multiply by -i (forward) or +i (inverse)
__device__ __forceinline__ double2 cmul_mi(double2 a, bool inv) {
  return inv ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// The chip dispatches the blocks of a launch to its 8 XCDs round-robin (block b to XCD b mod 8),
// and each XCD has its own L2.  For per-order products (tiles x, y of order z share the order's
// tables) xcd_tile deals whole orders to the XCDs in turn: XCD c runs the gx * gy tiles of order
// c, then those of c + 8, and so on, so that one L2 serves each order's tables and the triangular
// work (which shrinks with the order) is spread evenly.  The launch has xcd_blocks(gx, gy, gz)
// blocks; xcd_tile returns false for the padding blocks of the last round (b: the block's index, where the
// launch starts with blocks of another kind).
struct Tile3 {
  int x, y, z;
};
__device__ __forceinline__ bool xcd_tile(int gx, int gy, int gz, Tile3& t, int b) {
  const int per = gx * gy;
  const int c = b & 7, slot = b >> 3;
  const int tile = slot % per;
  t.z = c + 8 * (slot / per);
  t.x = tile % gx;
  t.y = tile / gx;
  return t.z < gz;
}
__device__ __forceinline__ bool xcd_tile(int gx, int gy, int gz, Tile3& t) {
  return xcd_tile(gx, gy, gz, t, blockIdx.x);
}
__host__ __device__ inline unsigned xcd_blocks(int gx, int gy, int gz) {
  return 8u * (unsigned)gx * (unsigned)gy * (unsigned)((gz + 7) / 8);
}

// Matrix-vector products of 2D plans (gemv.hip, step.hip).  A block takes GR rows of an order and the whole
// contraction: lane q of 8 owns two adjacent rows (one 16-byte table load a term), the GK groups of 8
// lanes every GK-th term.  The contraction goes in chunks of GK GU terms: the loads of the chunk's vector
// entries and then the GU table loads of every lane all go out together, with clamped indices and no branch,
// and the block shares the vector through LDS (zero past the end).  GU covers the whole contraction
// up to 1024 terms.  With the vector read from memory by every lane, its
// returned bytes, not the table's, bound the kernels (the first step product 11.6 us at N_r = 768).
constexpr int GR = 16;
constexpr int GK = 64;
constexpr int GT = GR / 2 * GK;  // threads
inline int gemv_unroll(int terms) { return terms <= 2 * GK ? 2 : (terms <= 4 * GK ? 4 : (terms <= 8 * GK ? 8 : 16)); }
typedef double dpair __attribute__((ext_vector_type(2), aligned(8)));  // two adjacent table entries

// acc[0 .. NA) summed over the GK groups; the totals of the lanes' rows end in threads 0 .. GR / 2 - 1
template <int NA>
__device__ __forceinline__ void block_sum(double (&acc)[NA]) {
  constexpr int GL = GR / 2;
  __shared__ double part[GT / 64][GL][NA];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = threadIdx.x % GL;
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    acc[i] += __shfl_xor(acc[i], 8, 64);
    acc[i] += __shfl_xor(acc[i], 16, 64);
    acc[i] += __shfl_xor(acc[i], 32, 64);
  }
  if (lane < GL) {
#pragma unroll
    for (int i = 0; i < NA; ++i) part[wave][q][i] = acc[i];
  }
  __syncthreads();
  if (threadIdx.x >= GL) return;
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    double s = part[0][q][i];
#pragma unroll
    for (int w = 1; w < GT / 64; ++w) s += part[w][q][i];
    acc[i] = s;
  }
}

// Logarithmic proxy (Eq. logproxy).  Potentials psi~ + c_psi Lambda, chi~ + c_chi Lambda with Lambda = ln(r^2 + ell^2):
// with q = (1 - x)^2 / ell^2 = grad_h^2 Lambda and r (1 - x) / ell^2 = 2 r / (r^2 + ell^2), the proxy parts add
// u_phi = -c_psi r sqrt(q) / ell, u_z = -c_chi q, w_phi = -2 c_chi r q^{3/2} / ell, w_z = -c_psi q to the
// m = 0, k = 0 harmonics (fields 1, 2, 4, 5 of u_r, u_phi, u_z, w_r, w_phi, w_z).
struct LogProxy {
  double cpsi, cchi, ell;
};
__device__ __forceinline__ double proxy_part(const LogProxy& p, int field, double rinv, double q) {
  const double r = 1.0 / rinv, sq = sqrt(q);
  if (field == 1) return -p.cpsi * r * sq / p.ell;
  if (field == 2) return -p.cchi * q;
  if (field == 4) return -2.0 * p.cchi * r * q * sq / p.ell;
  return field == 5 ? -p.cpsi * q : 0.0;
}

// Storage conversions: reduced-precision plans keep fields as float / float2 in memory while the
// kernels compute in double.
__device__ __forceinline__ double2 ld2(const double2* p) { return *p; }
__device__ __forceinline__ double2 ld2(const float2* p) {
  const float2 v = *p;
  return make_double2((double)v.x, (double)v.y);
}
__device__ __forceinline__ double2 to_d2(double2 a) { return a; }
__device__ __forceinline__ double2 to_d2(float2 a) { return make_double2((double)a.x, (double)a.y); }
__device__ __forceinline__ void st2(double2* p, double2 v) { *p = v; }
__device__ __forceinline__ void st2(float2* p, double2 v) { *p = make_float2((float)v.x, (float)v.y); }
__device__ __forceinline__ double ld1(const double* p) { return *p; }
__device__ __forceinline__ double ld1(const float* p) { return (double)*p; }
__device__ __forceinline__ void st1(double* p, double v) { *p = v; }
__device__ __forceinline__ void st1(float* p, double v) { *p = (float)v; }
template <typename S2>
__device__ __forceinline__ S2 czero();
template <>
__device__ __forceinline__ double2 czero<double2>() { return make_double2(0.0, 0.0); }
template <>
__device__ __forceinline__ float2 czero<float2>() { return make_float2(0.f, 0.f); }

}  // namespace dev
}  // namespace mlg
