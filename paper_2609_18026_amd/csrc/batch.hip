// Batched pseudospectral KPP term for many uneven 2D instances.
//
// For each instance b (N_z = 1): R_b = Mask(F(gamma u (1 - u))), u = B(Mask(u_hat_b)) (Sec. 3.3;
// Sec. 5.2, Eq. kpp; the two-thirds mask holds for the field entering the product too).  Three launches run
// the phases; the kernel boundaries order them (a grid-wide barrier inside one cooperative launch costs about 50 us on
// this part, against a few microseconds for a launch boundary).  The azimuthal phase, and the radial phases with tables, are
// persistent (a fixed number of blocks per CU, each walking its share of the phase's work list); with the
// recurrence the radial phases take a block per order:
//   1. backward radial transform per (instance, kept m): f_m(r_i) = sum_n Pbar_n^m(x_i) u_hat_n^m;
//      Pbar streamed from per-instance tables or regenerated in the kernel (phases 1 and 3) by the
//      normalised three-term recurrence (FP64) from states kept every 32 degrees;
//   2. per (instance, group of azimuthal lines): inverse real FFT in phi, gamma u (1 - u),
//      forward FFT, two-thirds mask;
//   3. forward radial projection per (instance, kept m): u_hat_n^m = sum_i w_i Pbar_n^m(x_i) g_m(r_i);
//      one item per instance writes the zeros of its masked orders.
// Both radial phases use Pbar_n^m(-x) = (-1)^(n-m) Pbar_n^m(x): the tables hold the nodes of one half, the even and
// odd degrees are summed apart (backward) or act on sums and differences of mirrored nodes (forward).
// Work lists of each phase are sorted by cost (largest first) and dealt round-robin to the
// blocks.  Data may be FP64 or FP32 (template T); recurrences and tables are built in FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "dft_reg.h"
#include "mlg_internal.h"

namespace mlg {

// radices of the azimuthal passes
#define BATCH_RADICES(X) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10)
constexpr int BT_PASSES = 4;

struct BatchInst {
  int nr, nphi, M, nrc;
  int mact;           // orders in the product: kept by the mask, with degrees, below the azimuthal Nyquist order
  int64_t spec_off;   // complex elements into the packed spectra
  int64_t mix_off;    // complex elements into the workspace (M x nr harmonics)
  int64_t tb_off;     // backward table Pbar [m][n-m][i]  (reals), i over the (N_r + 1) / 2 nodes of one half
  int64_t tf_off;     // forward table w Pbar [m][i][n-m] (reals), the same nodes
  int64_t rec_off;    // recurrence data: per m, (nrc - m) pairs (a_n, b_n)
  int64_t start_off;  // recurrence states [m][segment][2][i], the same nodes
  int64_t node_off;   // x_i, then w_i
  int64_t tw_off;     // exp(-2 pi i t / N_phi), complex
};

// One order of one instance in a radial phase, with every offset in it: a block reads it in one go where the
// chain item -> instance -> triangular offset -> data cost three more dependent loads.  nr == 0: K zeros at spec.
struct RadialItem {
  int64_t spec, mix, tab, rec, start, node;
  int nr, K;
};

// One group of lines in the azimuthal phase.
struct PhiItem {
  int64_t mix, tw;
  int nr, nphi, mact, q0;
  uint32_t rad;  // radices of the passes, a byte each
  int nrad;
};

struct BatchConfig {
  int recurrence;   // 1: regenerate Pbar in the kernels, 0: stream it from the tables
  int threads;      // 128 or 256
  int blocks_per_cu;
  int lines;        // azimuthal lines per phase-2 item (even)
  int blocks[3];    // blocks of each phase's launch (0: the kernel does not fit)
};

}  // namespace mlg

struct mlg_batch_s {
  int count = 0;
  int device = 0;
  mlg_precision prec = MLG_FP64;
  double gamma_default = 0.25;
  std::vector<mlg::BatchInst> inst;
  std::vector<int64_t> spec_offsets;  // count + 1
  int64_t spec_total = 0, mix_total = 0;
  double* d_tab = nullptr;     // FP64 tables (backward, forward, recurrence, start, nodes, twiddles)
  float* d_tab32 = nullptr;    // FP32 copies of the backward / forward tables (FP32 batches)
  mlg::RadialItem* d_radial[2] = {nullptr, nullptr};  // phases 1 and 3
  mlg::PhiItem* d_phi = nullptr;                      // phase 2
  int nitems[3] = {0, 0, 0};
  mlg::BatchConfig cfg{0, 256, 2, 8, {0, 0, 0}};
  int tuned = 0;
  int cus = 0;
  size_t ws_bytes = 0;
};

namespace mlg {
namespace {

template <typename T>
struct Cx {
  T x, y;
};
template <typename T>
__device__ __forceinline__ Cx<T> cx(T a, T b) {
  return Cx<T>{a, b};
}
template <typename T>
__device__ __forceinline__ Cx<T> operator+(Cx<T> a, Cx<T> b) { return cx(a.x + b.x, a.y + b.y); }
template <typename T>
__device__ __forceinline__ Cx<T> operator-(Cx<T> a, Cx<T> b) { return cx(a.x - b.x, a.y - b.y); }
template <typename T>
__device__ __forceinline__ Cx<T> scl(Cx<T> a, T s) { return cx(a.x * s, a.y * s); }

// Azimuthal transforms in place.  With n = R n', an outer stage of a line takes the butterflies x[n2 + n' n1] over n1 (inverse:
// transform, then w_n^(-k1 n2); forward: w_n^(k1 n2), then transform), which leaves R blocks of length n'; the
// innermost blocks, of length R, hold gridpoint values in registers, where the inverse transform, the product and the forward
// transform follow each other.  Every butterfly writes where it read, so there is one buffer, and on the way back the
// same stages in reverse end in natural order.  Registers are FP64 whatever the storage.
// Entry i of a line (and of the twiddle table) lies at i + i / 16: the strides of the radices would meet in a few banks.
// Quotients of small numbers by reciprocals: exact for idx < 4096 and divisors up to 256.
__host__ __device__ __forceinline__ int bgap(int i) { return i + (i >> 4); }
__host__ __device__ __forceinline__ int bpitch(int n) { return (bgap(n - 1) + 1) | 1; }
__device__ __forceinline__ int bquot(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// w = exp(-2 pi i / n) in tw, step = n / len; the inverse works on conjugates
template <typename T, int R>
__device__ __forceinline__ void outer_stage(Cx<T>* X, int n, int pitch, int len, int step, const double2* tw, int nl, bool inv) {
  const int nb = len / R, per = n / R;
  const float iper = 1.0f / (float)per, inb = 1.0f / (float)nb;
  const double sgn = inv ? -1.0 : 1.0;
  for (int idx = threadIdx.x; idx < nl * per; idx += blockDim.x) {
    const int line = bquot(idx, iper), j = idx - line * per;
    const int blk = bquot(j, inb), n2 = j - blk * nb;
    Cx<T>* x = X + line * pitch;
    const int base = blk * len + n2;
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const Cx<T> e = x[bgap(base + r * nb)];
      v[r] = make_double2((double)e.x, sgn * (double)e.y);
    }
    if (!inv) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = dev::cmul(v[r], tw[bgap(n2 * r * step)]);
    }
    dev::Dft<R, false>::run(v);
    if (inv) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = dev::cmul(v[r], tw[bgap(n2 * r * step)]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) x[bgap(base + r * nb)] = cx<T>((T)v[r].x, (T)(sgn * v[r].y));
  }
}

// both packed lines: gamma u (1 - u)
template <typename T, int R>
__device__ __forceinline__ void inner_stage(Cx<T>* X, int n, int pitch, int nl, double gamma) {
  const int per = n / R;
  const float iper = 1.0f / (float)per;
  for (int idx = threadIdx.x; idx < nl * per; idx += blockDim.x) {
    const int line = bquot(idx, iper), base = (idx - line * per) * R;
    Cx<T>* x = X + line * pitch;
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const Cx<T> e = x[bgap(base + r)];
      v[r] = make_double2((double)e.x, (double)e.y);
    }
    dev::Dft<R, true>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = make_double2(gamma * v[r].x * (1.0 - v[r].x), gamma * v[r].y * (1.0 - v[r].y));
    dev::Dft<R, false>::run(v);
#pragma unroll
    for (int r = 0; r < R; ++r) x[bgap(base + r)] = cx<T>((T)v[r].x, (T)v[r].y);
  }
}

// One loop over the stages there and back: the code of each is there once.
template <typename T>
__device__ __forceinline__ void kpp_lines(Cx<T>* X, const PhiItem& I, int pitch, const double2* tw, int nl, double gamma) {
  const int n = I.nphi, last = I.nrad - 1;
  for (int q = 0; q <= 2 * last; ++q) {
    const int p = q <= last ? q : 2 * last - q;
    int step = 1;
    for (int k = 0; k < p; ++k) step *= I.rad >> 8 * k & 255;
    const int R = I.rad >> 8 * p & 255;
#define BATCH_OUTER(N) \
  case N:              \
    outer_stage<T, N>(X, n, pitch, n / step, step, tw, nl, q < last); \
    break;
#define BATCH_INNER(N) \
  case N:              \
    inner_stage<T, N>(X, n, pitch, nl, gamma); \
    break;
    if (p < last) {
      switch (R) { BATCH_RADICES(BATCH_OUTER) }
    } else {
      switch (R) { BATCH_RADICES(BATCH_INNER) }
    }
#undef BATCH_OUTER
#undef BATCH_INNER
    __syncthreads();
  }
}

template <typename T>
struct BatchArgs {
  const double* tab;
  const T* tabT;         // tables in the data precision (backward / forward)
  const Cx<T>* spec_in;
  Cx<T>* spec_out;
  Cx<T>* mix;
  const RadialItem* radial[2];
  const PhiItem* phi;
  int nitems[3];
  int lines;
  T gamma;
};

// Radial phases from the tables.  The whole block shares the contraction: the lanes of a sub (a wavefront, or half of one
// where that covers the row) take two adjacent nodes (backward) or degrees (forward) with 16-byte loads, the subs every
// subs-th term, U terms of loads at a time with clamped rows (the vector in LDS is zero past its end); the
// partial sums of the subs meet in LDS.  Bound by the one read of the table: forward 42 us at 6.1 TB/s for 64 instances
// (N_r 48 .. 256, N_phi 32 .. 256), where one thread per output walking the whole contraction over both halves of the
// nodes took 110 us.
constexpr int BT_DEG = 256;                     // the largest number of degrees, and of nodes
constexpr int BT_PAD = 32;                      // zeros past the end of a vector: subs U terms at most
constexpr int BT_VEC = (BT_DEG + 2 * BT_PAD);   // complex entries of the vector in LDS

// two adjacent table entries, on the alignment of one; where the second lies past a row it is the next row's first or, at the
// end of a table, the entry of the array that follows, and its sum is not stored
template <typename T>
struct TPair {
  typedef T v __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};

// lanes of a sub take two nodes each; SUB subs a wavefront (2 where 64 nodes fit half of it)
template <typename T, int SUB>
__device__ __forceinline__ void backward_table(const T* __restrict__ P, Cx<T>* s, int K, int nh, int nr, Cx<T>* mix) {
  constexpr int LN = 64 / SUB, U = 4;
  const int sub = threadIdx.x / LN, subs = blockDim.x / LN, q = 2 * (threadIdx.x % LN), col = min(q, nh - 1);
  Cx<T> e[2], o[2];
  e[0] = e[1] = o[0] = o[1] = cx<T>(0, 0);
  for (int j0 = sub; 2 * j0 < K; j0 += subs * U) {
    typename TPair<T>::v p[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        p[u][h] = *reinterpret_cast<const typename TPair<T>::v*>(P + min(2 * (j0 + subs * u) + h, K - 1) * nh + col);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Cx<T> se = s[2 * (j0 + subs * u)], so = s[2 * (j0 + subs * u) + 1];
      e[0] = e[0] + scl(se, p[u][0].x);
      e[1] = e[1] + scl(se, p[u][0].y);
      o[0] = o[0] + scl(so, p[u][1].x);
      o[1] = o[1] + scl(so, p[u][1].y);
    }
  }
  __syncthreads();  // the vector has been read
  Cx<T>* part = s;  // [sub][parity][node]
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    part[2 * sub * 2 * LN + q + h] = e[h];
    part[(2 * sub + 1) * 2 * LN + q + h] = o[h];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nh; i += blockDim.x) {
    Cx<T> se = part[i], so = part[2 * LN + i];
    for (int w = 1; w < subs; ++w) {
      se = se + part[2 * w * 2 * LN + i];
      so = so + part[(2 * w + 1) * 2 * LN + i];
    }
    mix[i] = se + so;
    if (nr - 1 - i != i) mix[nr - 1 - i] = se - so;
  }
}

template <typename T>
__device__ void phase_backward(const BatchArgs<T>& A, const RadialItem I, char* smem) {
  const int K = I.K, nr = I.nr, nh = (nr + 1) / 2;
  Cx<T>* mix = A.mix + I.mix;
  Cx<T>* s = reinterpret_cast<Cx<T>*>(smem);
  for (int t = threadIdx.x; t < K + 2 * BT_PAD; t += blockDim.x) s[t] = t < K ? A.spec_in[I.spec + t] : cx<T>(0, 0);
  __syncthreads();
  if (nh <= 64) {
    backward_table<T, 2>(A.tabT + I.tab, s, K, nh, nr, mix);
  } else {
    backward_table<T, 1>(A.tabT + I.tab, s, K, nh, nr, mix);
  }
  __syncthreads();
}

// Azimuthal phase: np pairs of lines, each pair one complex line.  Bound by latency: load, stages and store of an item follow
// each other with a barrier between them, so what counts is few stages and every item resident at once.  Loads run over the
// lines of an order first (L adjacent nodes, 128 bytes for 8).  64 instances as above: radix-2 to 5 passes between two
// buffers 25 us, of which about 8 were a second turn of blocks and 4 the launch; now 18.4 at 8 lines in 128 threads, the shape that the
// autotuner takes (17.5 at 12 lines in 256, which it does not try).
template <typename T>
__device__ void phase_phi(const BatchArgs<T>& A, const PhiItem I, char* smem) {
  const int n = I.nphi, q0 = I.q0, L = A.lines, np = L / 2, nr = I.nr, mact = I.mact, pitch = bpitch(n);
  Cx<T>* X = reinterpret_cast<Cx<T>*>(smem);
  // the twiddle table follows the lines, at a multiple of 16 bytes
  double2* tw = reinterpret_cast<double2*>(smem + ((size_t)np * pitch * sizeof(Cx<T>) + 15) / 16 * 16);
  const double* twg = A.tab + I.tw;
  for (int e = threadIdx.x; e < n; e += blockDim.x) tw[bgap(e)] = make_double2(twg[2 * e], twg[2 * e + 1]);
  Cx<T>* mix = A.mix + I.mix;
  const float inp = 1.0f / (float)np, il = 1.0f / (float)L;
  for (int e = threadIdx.x; e < np * (n / 2 + 1); e += blockDim.x) {
    const int m = (int)(((float)e + 0.5f) * inp), p = e - m * np;
    const int qa = q0 + 2 * p, qb = qa + 1;
    const Cx<T>* h = mix + (int64_t)min(m, mact - 1) * nr;
    Cx<T> a = h[min(qa, nr - 1)], c = h[min(qb, nr - 1)];
    if (m >= mact || qa >= nr) a = cx<T>(0, 0);
    if (m >= mact || qb >= nr) c = cx<T>(0, 0);
    if (m == 0) {
      X[p * pitch] = cx(a.x, c.x);
    } else {
      X[p * pitch + bgap(m)] = cx(a.x - c.y, a.y + c.x);
      X[p * pitch + bgap(n - m)] = cx(a.x + c.y, -a.y + c.x);
    }
  }
  __syncthreads();
  kpp_lines<T>(X, I, pitch, tw, np, (double)A.gamma);
  const double sc = 0.5 / (double)n;
  for (int e = threadIdx.x; e < mact * L; e += blockDim.x) {
    const int m = (int)(((float)e + 0.5f) * il), ll = e - m * L, q = q0 + ll;
    if (q >= nr) continue;
    const Cx<T>* Zp = X + (ll >> 1) * pitch;
    const Cx<T> zm = Zp[bgap(m)], zc = Zp[bgap(m == 0 ? 0 : n - m)];
    const double ax = zm.x, ay = zm.y, bx = zc.x, by = -(double)zc.y;
    mix[(int64_t)m * nr + q] = (ll & 1) == 0 ? cx<T>((T)(sc * (ax + bx)), (T)(sc * (ay + by)))
                                             : cx<T>((T)(sc * (ay - by)), (T)(-sc * (ax - bx)));
  }
  __syncthreads();
}

// lanes of a sub take an even and the next odd degree, NG times
template <typename T, int SUB, int NG, int U>
__device__ __forceinline__ void forward_table(const T* __restrict__ P, Cx<T>* g, int K, int nh, Cx<T>* out) {
  constexpr int LN = 64 / SUB;
  const int sub = threadIdx.x / LN, subs = blockDim.x / LN, q = 2 * (threadIdx.x % LN);
  Cx<T> e[NG], o[NG];
  int col[NG];
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    e[c] = o[c] = cx<T>(0, 0);
    col[c] = min(q + 128 * c, K - 1);
  }
  for (int i0 = sub; i0 < nh; i0 += subs * U) {
    typename TPair<T>::v p[U][NG];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NG; ++c)
        p[u][c] = *reinterpret_cast<const typename TPair<T>::v*>(P + min(i0 + subs * u, nh - 1) * K + col[c]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Cx<T> sum = g[2 * (i0 + subs * u)], dif = g[2 * (i0 + subs * u) + 1];
#pragma unroll
      for (int c = 0; c < NG; ++c) {
        e[c] = e[c] + scl(sum, p[u][c].x);
        o[c] = o[c] + scl(dif, p[u][c].y);
      }
    }
  }
  __syncthreads();  // the vector has been read
  Cx<T>* part = g;  // [sub][degree]
  constexpr int ROW = 2 * LN * NG;
#pragma unroll
  for (int c = 0; c < NG; ++c) {
    part[sub * ROW + q + 128 * c] = e[c];
    part[sub * ROW + q + 128 * c + 1] = o[c];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < K; t += blockDim.x) {
    Cx<T> v = part[t];
    for (int w = 1; w < subs; ++w) v = v + part[w * ROW + t];
    out[t] = v;
  }
}

template <typename T>
__device__ void phase_forward(const BatchArgs<T>& A, const RadialItem I, char* smem) {
  const int K = I.K, nr = I.nr, nh = (nr + 1) / 2;
  Cx<T>* out = A.spec_out + I.spec;
  if (nr == 0) {
    for (int t = threadIdx.x; t < K; t += blockDim.x) out[t] = cx<T>(0, 0);
    return;
  }
  Cx<T>* g = reinterpret_cast<Cx<T>*>(smem);  // [half node][sum, difference]
  const Cx<T>* mix = A.mix + I.mix;
  for (int i = threadIdx.x; i < nh + BT_PAD; i += blockDim.x) {
    const int ic = min(i, nh - 1);
    const Cx<T> a = mix[ic], b = mix[nr - 1 - ic];
    const bool in = i < nh, mid = nr - 1 - i == i;  // the middle node of an odd N_r stands alone
    g[2 * i] = !in ? cx<T>(0, 0) : (mid ? a : a + b);
    g[2 * i + 1] = in && !mid ? a - b : cx<T>(0, 0);
  }
  __syncthreads();
  const T* P = A.tabT + I.tab;
  if (K <= 64) forward_table<T, 2, 1, 4>(P, g, K, nh, out);
  else if (K <= 128) forward_table<T, 1, 1, 8>(P, g, K, nh, out);
  else forward_table<T, 1, 2, 4>(P, g, K, nh, out);
  __syncthreads();
}

template <typename T, int PHASE>
__global__ __launch_bounds__(256, PHASE == 0 ? 6 : (PHASE == 1 ? 4 : 5)) void batch_kernel(BatchArgs<T> A) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  for (int it = blockIdx.x; it < A.nitems[PHASE]; it += gridDim.x) {
    if constexpr (PHASE == 0) phase_backward<T>(A, A.radial[0][it], smem);
    else if constexpr (PHASE == 1) phase_phi<T>(A, A.phi[it], smem);
    else phase_forward<T>(A, A.radial[1][it], smem);
  }
}

// Radial phases with the recurrence Pbar_n^m = a_n x Pbar_{n-1}^m - b_n Pbar_{n-2}^m in registers: a block takes an order, its
// wavefronts consecutive segments of RC_S degrees (the two values before each segment are kept per node), the
// lanes of a wavefront NPL nodes each of one half (NPL = 2 above 64 half nodes).  a_n, b_n and the coefficients are the
// same for the whole wavefront and come by scalar loads (pointers that do not alias, indices the compiler sees to be
// uniform).  The entries n = m (0, 1) and n = m + 1 (sqrt(2 m + 3), 0) start the first segment from (-Pbar_m^m, 0).
// A block per order whatever the launch shape asks: dealt to fewer blocks, an order waits for another's first loads.
// 64 instances (N_r 48 .. 256, N_phi 32 .. 256): backward 33 us (a thread a node over both halves, coefficients from
// LDS) -> 15; forward 42 us from the tables (256 MB at 6.1 TB/s) -> 23, of which the FP64 operations are about 5 and
// 12 (8 of them the sums over the lanes), launch and first loads 6, the scalar loads 4 and 2.
constexpr int RC_S = 32;  // degrees per segment
constexpr int RC_B = 8;   // degrees per scalar load, backward
constexpr int RC_F = 8;   // degrees per transposing sum, forward
// Wavefronts per order: RC_FEW up to RC_ITEMS orders in the launch (one a SIMD), where the chip has places to spare and the chain of
// an order bounds the phase, 2 above.  One instance of 256 x 16, all three phases: 24.9 -> 17.5 us (FP32 with forward tables, before: 21.2),
// 64 of 256 x 16 (384 orders) 43.1 -> 32.8, 12 of 256 x 256 (1032) 41.8 / 39.6; 64 of 128 x 128 (2752) 52.4 / 52.0 (FP32 47.3 / 48.4),
// 512 of 16 x 16 (3072) 18.4 / 20.4.
constexpr int RC_FEW = 4, RC_ITEMS = 1024;

// Touches the lines of a wavefront's recurrence or coefficients, so that the scalar loads of the backward phase find them in the
// L2: 18.8 -> 15.4 us (nothing forward, where a degree takes longer than its loads).
template <typename A>
__device__ __forceinline__ void touch(const A* p, int count) {
  const int line = 64 / (int)sizeof(A);
  for (int e = (threadIdx.x & 63) * line; e < count; e += 64 * line) {
    const int w = *reinterpret_cast<const volatile int*>(p + e);
    (void)w;
  }
}

template <int NPL>
struct Recurrence {
  double x[NPL], p0[NPL], p1[NPL];
  __device__ __forceinline__ void start(const double* __restrict__ tab, const RadialItem& I, int lane, int nh, int seg) {
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      const int i = min(lane + 64 * j, nh - 1);
      x[j] = tab[I.node + i];
      p0[j] = tab[I.start + (2 * seg) * nh + i];
      p1[j] = tab[I.start + (2 * seg + 1) * nh + i];
    }
  }
  __device__ __forceinline__ void step(double a, double b) {
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      const double p2 = (a * x[j]) * p1[j] - b * p0[j];
      p0[j] = p1[j];
      p1[j] = p2;
    }
  }
};

template <typename T, int NPL, int W>
__device__ __forceinline__ void recur_backward(const double* __restrict__ tab, const Cx<T>* __restrict__ spec,
                                               Cx<T>* __restrict__ mix, const RadialItem& I, int wave) {
  __shared__ Cx<double> part[(W - 1) * 2 * 64 * NPL];  // [wave][parity][node] of the wavefronts after the first
  const int lane = threadIdx.x & 63, K = I.K, nr = I.nr, nh = (nr + 1) / 2;
  const int segs = (K + RC_S - 1) / RC_S, seg = wave * segs / W;
  const int end = min((wave + 1) * segs / W * RC_S, K);
  const double* __restrict__ rec = tab + I.rec;
  const Cx<T>* __restrict__ s = spec + I.spec;
  int t = seg * RC_S;
  touch(rec + 2 * t, 2 * (end - t));
  touch(s + t, end - t);
  Recurrence<NPL> r;
  r.start(tab, I, lane, nh, min(seg, segs - 1));
  double re[2][NPL], im[2][NPL];
#pragma unroll
  for (int j = 0; j < NPL; ++j) re[0][j] = re[1][j] = im[0][j] = im[1][j] = 0.0;
  auto term = [&](int par, double a, double b, double sx, double sy) {
    r.step(a, b);
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
      re[par][j] += sx * r.p1[j];
      im[par][j] += sy * r.p1[j];
    }
  };
  for (; t + RC_B <= end; t += RC_B) {
    double ab[2 * RC_B];
    Cx<T> v[RC_B];
#pragma unroll
    for (int u = 0; u < RC_B; ++u) {
      ab[2 * u] = rec[2 * (t + u)];
      ab[2 * u + 1] = rec[2 * (t + u) + 1];
      v[u] = s[t + u];
    }
#pragma unroll
    for (int u = 0; u < RC_B; ++u) term(u & 1, ab[2 * u], ab[2 * u + 1], (double)v[u].x, (double)v[u].y);
  }
  for (; t < end; t += 2) {
    term(0, rec[2 * t], rec[2 * t + 1], (double)s[t].x, (double)s[t].y);
    if (t + 1 < end) term(1, rec[2 * t + 2], rec[2 * t + 3], (double)s[t + 1].x, (double)s[t + 1].y);
  }
  if (wave > 0) {
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
      for (int j = 0; j < NPL; ++j)
        part[((wave - 1) * 2 + par) * 64 * NPL + lane + 64 * j] = Cx<double>{re[par][j], im[par][j]};
  }
  __syncthreads();
  if (wave > 0) return;
  Cx<T>* out = mix + I.mix;
#pragma unroll
  for (int j = 0; j < NPL; ++j) {
    const int i = lane + 64 * j;
    Cx<double> e{re[0][j], im[0][j]}, o{re[1][j], im[1][j]};
#pragma unroll
    for (int w = 0; w < W - 1; ++w) {
      e = e + part[2 * w * 64 * NPL + i];
      o = o + part[(2 * w + 1) * 64 * NPL + i];
    }
    if (i >= nh) continue;
    out[i] = cx<T>((T)(e.x + o.x), (T)(e.y + o.y));
    if (nr - 1 - i != i) out[nr - 1 - i] = cx<T>((T)(e.x - o.x), (T)(e.y - o.y));
  }
}

// One step of the transposing sum over the lanes: of two values a lane keeps the one its bit names, summed with the
// partner's (lane ^ 32, lane ^ 16: one swap instruction a register).
template <int MASK>
__device__ __forceinline__ double swap_sum(double a, double b) {
  const int2 ua = __builtin_bit_cast(int2, a), ub = __builtin_bit_cast(int2, b);
  if constexpr (MASK == 32) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ua.x, (unsigned)ub.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)ua.y, (unsigned)ub.y, false, false);
    return __builtin_bit_cast(double, make_int2((int)lo[0], (int)hi[0])) +
           __builtin_bit_cast(double, make_int2((int)lo[1], (int)hi[1]));
  } else {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)ua.x, (unsigned)ub.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)ua.y, (unsigned)ub.y, false, false);
    return __builtin_bit_cast(double, make_int2((int)lo[0], (int)hi[0])) +
           __builtin_bit_cast(double, make_int2((int)lo[1], (int)hi[1]));
  }
}
// value of the lane's partner: row mirror (lane ^ 15), half-row mirror (^ 7), quad reversal (^ 3), quad pairs (^ 1)
template <int CTRL>
__device__ __forceinline__ double dpp_partner(double a) {
  const int2 u = __builtin_bit_cast(int2, a);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, u.x, CTRL, 0xf, 0xf, false),
                                              __builtin_amdgcn_update_dpp(0, u.y, CTRL, 0xf, 0xf, false)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_sum(double a, double b, bool bit) {
  return (bit ? b : a) + dpp_partner<CTRL>(bit ? a : b);
}

template <typename T, int NPL, int W>
__device__ __forceinline__ void recur_forward(const double* __restrict__ tab, const Cx<T>* __restrict__ mix,
                                              Cx<T>* __restrict__ spec, const RadialItem& I, int wave) {
  const int lane = threadIdx.x & 63, K = I.K, nr = I.nr, nh = (nr + 1) / 2;
  const int segs = (K + RC_S - 1) / RC_S, seg = wave * segs / W;
  const int end = min((wave + 1) * segs / W * RC_S, K);
  if (seg * RC_S >= end) return;
  const double* __restrict__ rec = tab + I.rec;
  const Cx<T>* __restrict__ g = mix + I.mix;
  Recurrence<NPL> r;
  r.start(tab, I, lane, nh, seg);
  double gx[2][NPL], gy[2][NPL];  // weighted sums and differences of mirrored nodes, 0 past the last node
#pragma unroll
  for (int j = 0; j < NPL; ++j) {
    const int i = lane + 64 * j, ic = min(i, nh - 1);
    const double w = i < nh ? tab[I.node + nh + ic] : 0.0;
    const bool mid = nr - 1 - ic == ic;  // the middle node of an odd N_r stands alone
    const Cx<T> a = g[ic], b = g[nr - 1 - ic];
    const double bx = mid ? 0.0 : (double)b.x, by = mid ? 0.0 : (double)b.y;
    gx[0][j] = w * ((double)a.x + bx);
    gy[0][j] = w * ((double)a.y + by);
    gx[1][j] = mid ? 0.0 : w * ((double)a.x - bx);
    gy[1][j] = mid ? 0.0 : w * ((double)a.y - by);
  }
  const bool b3 = lane & 8, b2 = lane & 4;
  T* out = reinterpret_cast<T*>(spec + I.spec);
  for (int t0 = seg * RC_S; t0 < end; t0 += RC_F) {
    // the terms past the column take the entries that follow in the table: their sums are not stored
    double v[2 * RC_F];  // 2 d + (0 re, 1 im) of degree t0 + d
#pragma unroll
    for (int d = 0; d < RC_F; ++d) {
      r.step(rec[2 * (t0 + d)], rec[2 * (t0 + d) + 1]);
      v[2 * d] = r.p1[0] * gx[d & 1][0];
      v[2 * d + 1] = r.p1[0] * gy[d & 1][0];
#pragma unroll
      for (int j = 1; j < NPL; ++j) {
        v[2 * d] += r.p1[j] * gx[d & 1][j];
        v[2 * d + 1] += r.p1[j] * gy[d & 1][j];
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = swap_sum<32>(v[q], v[q + 8]);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = swap_sum<16>(v[q], v[q + 4]);
#pragma unroll
    for (int q = 0; q < 2; ++q) v[q] = dpp_sum<0x140>(v[q], v[q + 2], b3);
    v[0] = dpp_sum<0x141>(v[0], v[1], b2);
    v[0] += dpp_partner<0x1b>(v[0]);
    v[0] += dpp_partner<0xb1>(v[0]);
    if (!(lane & 3) && (lane >> 3) < end - t0) out[2 * t0 + (lane >> 2)] = (T)v[0];
  }
}

template <typename T, bool FWD, int W>
__global__ __launch_bounds__(64 * W) void batch_recur_kernel(const RadialItem* __restrict__ items,
                                                                const double* __restrict__ tab,
                                                                const Cx<T>* __restrict__ in, Cx<T>* __restrict__ out) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RadialItem I = items[blockIdx.x];
  if constexpr (FWD) {
    if (I.nr == 0) {
      for (int t = threadIdx.x; t < I.K; t += 64 * W) out[I.spec + t] = cx<T>(0, 0);
    } else if (I.nr <= 128) {
      recur_forward<T, 1, W>(tab, in, out, I, wave);
    } else {
      recur_forward<T, 2, W>(tab, in, out, I, wave);
    }
  } else {
    if (I.nr <= 128) recur_backward<T, 1, W>(tab, in, out, I, wave);
    else recur_backward<T, 2, W>(tab, in, out, I, wave);
  }
}

// LDS of a launch: the table phases hold the vector, then the partial sums of the subs; phase 2 lines / 2 complex lines, then the
// twiddle table (nphi complex FP64).
size_t radial_smem(const mlg_batch_s* bt, int threads) {
  const size_t cs = bt->prec == MLG_FP32 ? sizeof(Cx<float>) : sizeof(Cx<double>);
  return std::max((size_t)BT_VEC, (size_t)threads / 64 * BT_DEG) * cs;
}
size_t phi_smem(const mlg_batch_s* bt, int lines) {
  size_t mx = 0;
  const size_t cs = bt->prec == MLG_FP32 ? sizeof(Cx<float>) : sizeof(Cx<double>);
  for (const auto& I : bt->inst)
    mx = std::max(mx, ((size_t)(lines / 2) * bpitch(I.nphi) * cs + 15) / 16 * 16 + (size_t)bpitch(I.nphi) * sizeof(Cx<double>));
  return mx;
}

// blocks of each phase: the configured count per CU, capped by what the kernel's registers and LDS allow
template <typename T>
void set_blocks(const mlg_batch_s* bt, BatchConfig& c) {
  const void* k[3] = {reinterpret_cast<const void*>(batch_kernel<T, 0>), reinterpret_cast<const void*>(batch_kernel<T, 1>),
                      reinterpret_cast<const void*>(batch_kernel<T, 2>)};
  for (int p = 0; p < 3; ++p) {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, k[p], c.threads, p == 1 ? phi_smem(bt, c.lines) : radial_smem(bt, c.threads));
    c.blocks[p] = e == hipSuccess && n > 0 ? std::min(n, c.blocks_per_cu) * bt->cus : 0;
  }
}
void set_blocks(const mlg_batch_s* bt, BatchConfig& c) {
  if (bt->prec == MLG_FP32) set_blocks<float>(bt, c);
  else set_blocks<double>(bt, c);
}

template <typename T>
mlg_status run_batch(const mlg_batch_s* bt, double gamma, const void* in, void* out, void* ws, hipStream_t s,
                     const BatchConfig& c) {
  BatchArgs<T> A{};
  A.tab = bt->d_tab;
  if constexpr (sizeof(T) == 8)
    A.tabT = reinterpret_cast<const T*>(bt->d_tab);
  else
    A.tabT = reinterpret_cast<const T*>(bt->d_tab32);
  A.spec_in = reinterpret_cast<const Cx<T>*>(in);
  A.spec_out = reinterpret_cast<Cx<T>*>(out);
  A.mix = reinterpret_cast<Cx<T>*>(ws);
  for (int p = 0; p < 2; ++p) A.radial[p] = bt->d_radial[p];
  A.phi = bt->d_phi;
  for (int p = 0; p < 3; ++p) {
    A.nitems[p] = bt->nitems[p];
    if (c.blocks[p] <= 0) return fail(MLG_E_DEVICE, "batch kernel does not fit on a CU");
  }
  A.lines = c.lines;
  A.gamma = (T)gamma;
  const size_t rad = radial_smem(bt, c.threads);
  const unsigned th = (unsigned)c.threads;
  if (!c.recurrence) batch_kernel<T, 0><<<c.blocks[0], th, rad, s>>>(A);
  else if (A.nitems[0] > RC_ITEMS) batch_recur_kernel<T, false, 2><<<A.nitems[0], 128, 0, s>>>(A.radial[0], A.tab, A.spec_in, A.mix);
  else batch_recur_kernel<T, false, RC_FEW><<<A.nitems[0], 64 * RC_FEW, 0, s>>>(A.radial[0], A.tab, A.spec_in, A.mix);
  batch_kernel<T, 1><<<c.blocks[1], th, phi_smem(bt, c.lines), s>>>(A);
  if (!c.recurrence) batch_kernel<T, 2><<<c.blocks[2], th, rad, s>>>(A);
  else if (A.nitems[0] > RC_ITEMS) batch_recur_kernel<T, true, 2><<<A.nitems[2], 128, 0, s>>>(A.radial[1], A.tab, A.mix, A.spec_out);
  else batch_recur_kernel<T, true, RC_FEW><<<A.nitems[2], 64 * RC_FEW, 0, s>>>(A.radial[1], A.tab, A.mix, A.spec_out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string("batch kernel launch: ") + hipGetErrorString(e));
  return MLG_OK;
}

using ld = long double;

}  // namespace

mlg_status batch_run(const mlg_batch_s* bt, double gamma, const void* in, void* out, void* ws, hipStream_t s,
                     const BatchConfig& c) {
  if (bt->prec == MLG_FP32) return run_batch<float>(bt, gamma, in, out, ws, s, c);
  return run_batch<double>(bt, gamma, in, out, ws, s, c);
}

// what a launch shape is accepted by: two buffers of the lines and the twiddle table within 64 KB
size_t batch_smem(const mlg_batch_s* bt, int lines) {
  size_t mx = 0;
  const size_t cs = bt->prec == MLG_FP32 ? sizeof(Cx<float>) : sizeof(Cx<double>);
  for (const auto& I : bt->inst) mx = std::max(mx, (size_t)I.nphi * ((lines / 2) * 2 * cs + sizeof(Cx<double>)));
  return mx;
}

}  // namespace mlg

// ------------------------------------------------------------------------------------ host side
namespace mlg {
namespace {

template <typename V>
mlg_status up(V** dst, const std::vector<typename std::remove_pointer<V*>::type>& src) {
  using E = typename std::remove_pointer<V*>::type;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(dst), std::max<size_t>(src.size(), 1) * sizeof(E));
  if (e != hipSuccess) { *dst = nullptr; return fail(MLG_E_ALLOC, std::string("hipMalloc: ") + hipGetErrorString(e)); }
  if (!src.empty()) {
    e = hipMemcpy(*dst, src.data(), src.size() * sizeof(E), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(MLG_E_DEVICE, std::string("hipMemcpy: ") + hipGetErrorString(e));
  }
  return MLG_OK;
}

void free_batch(mlg_batch_s* b) {
  if (!b) return;
  void* ptrs[] = {b->d_tab, b->d_tab32, b->d_radial[0], b->d_radial[1], b->d_phi};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  delete b;
}

// the fewest passes of the radices (at most BT_PASSES for n = 2^a 3^b 5^c <= 256), the largest as small as possible
int batch_radices(int n, int* rad) {
#define BATCH_LIST(R) R,
  const int list[] = {BATCH_RADICES(BATCH_LIST)};
#undef BATCH_LIST
  for (int passes = 1; passes <= BT_PASSES; ++passes) {
    // the radices as digits, none above the one before it
    for (int top : list) {
      int left = n, k = 0, cap = top;
      if (left % top) continue;
      for (rad[k++] = top, left /= top; left > 1 && k < passes; ++k) {
        int best = 0;
        for (int r : list)
          if (r <= cap && left % r == 0) best = r;
        if (!best) break;
        rad[k] = cap = best;
        left /= best;
      }
      if (left == 1) return k;
    }
  }
  return -1;
}

// values per node of the recurrence states of a column of K degrees
int64_t rec_states(int K) { return 2 * ((std::max(K, 0) + RC_S - 1) / RC_S); }

// Work lists sorted by estimated cost, largest first.
mlg_status build_radial(mlg_batch_s* bt, const std::vector<int64_t>& tri) {
  std::vector<RadialItem> w[2];
  const int64_t* off = tri.data();
  for (int b = 0; b < bt->count; ++b) {
    const BatchInst& I = bt->inst[b];
    const int nh = (I.nr + 1) / 2;
    int64_t start = I.start_off;
    for (int m = 0; m < I.mact; start += rec_states(I.nrc - m) * nh, ++m) {
      RadialItem it{I.spec_off + off[m], I.mix_off + (int64_t)m * I.nr, I.tb_off + off[m] * nh, I.rec_off + 2 * off[m],
                    start, I.node_off, I.nr, I.nrc - m};
      w[0].push_back(it);
      it.tab = I.tf_off + off[m] * nh;
      w[1].push_back(it);
    }
    if (off[I.M] > off[I.mact])
      w[1].push_back(RadialItem{I.spec_off + off[I.mact], 0, 0, 0, 0, 0, 0, (int)(off[I.M] - off[I.mact])});
    off += I.M + 1;
  }
  for (int p = 0; p < 2; ++p) {
    std::stable_sort(w[p].begin(), w[p].end(), [](const RadialItem& a, const RadialItem& c) {
      return (int64_t)a.K * a.nr > (int64_t)c.K * c.nr;
    });
    if (mlg_status st = up(&bt->d_radial[p], w[p])) return st;
    bt->nitems[2 * p] = (int)w[p].size();
  }
  return MLG_OK;
}

mlg_status build_phi(mlg_batch_s* bt, int lines) {
  struct W { double cost; PhiItem item; };
  std::vector<W> w;
  for (int b = 0; b < bt->count; ++b) {
    const BatchInst& I = bt->inst[b];
    int rad[BT_PASSES];
    const int nrad = batch_radices(I.nphi, rad);
    uint32_t packed = 0;
    for (int p = 0; p < nrad; ++p) packed |= (uint32_t)rad[p] << 8 * p;
    for (int q = 0; q < I.nr; q += lines)
      w.push_back({(double)lines * I.nphi * std::log2((double)I.nphi + 1.0),
                   PhiItem{I.mix_off, I.tw_off, I.nr, I.nphi, I.mact, q, packed, nrad}});
  }
  std::stable_sort(w.begin(), w.end(), [](const W& a, const W& c) { return a.cost > c.cost; });
  std::vector<PhiItem> codes(w.size());
  for (size_t i = 0; i < w.size(); ++i) codes[i] = w[i].item;
  if (bt->d_phi) (void)hipFree(bt->d_phi);
  bt->d_phi = nullptr;
  if (mlg_status st = up(&bt->d_phi, codes)) return st;
  bt->nitems[1] = (int)codes.size();
  return MLG_OK;
}

}  // namespace
}  // namespace mlg

using namespace mlg;

extern "C" {

mlg_status mlg_batch_create(int count, const mlg_grid* grids, mlg_precision prec, int device, mlg_batch* out) {
  if (!out) return fail(MLG_E_ARG, "out is NULL");
  *out = nullptr;
  if (count <= 0 || count > 16384 || !grids) return fail(MLG_E_ARG, "count must be in [1, 16384] and grids non-NULL");
  if (prec != MLG_FP64 && prec != MLG_FP32) return fail(MLG_E_UNSUPPORTED, "batches support MLG_FP64 and MLG_FP32");
  for (int b = 0; b < count; ++b) {
    const mlg_grid& g = grids[b];
    if (!std::isfinite(g.ell) || !(g.ell > 0)) return fail(MLG_E_ARG, "ell must be positive and finite");
    if (g.nz != 1) return fail(MLG_E_UNSUPPORTED, "batched instances are 2D (N_z = 1)");
    if (g.nr < 2 || g.nr > 256) return fail(MLG_E_UNSUPPORTED, "batched instances need 2 <= N_r <= 256");
    if (g.nphi < 2 || g.nphi > 256) return fail(MLG_E_UNSUPPORTED, "batched instances need 2 <= N_phi <= 256");
    int r[16];
    if (factor_radices(g.nphi, r) < 0) return fail(MLG_E_UNSUPPORTED, "N_phi must have prime factors 2, 3, 5 only");
    if (g.nrc < 0 || g.nrc > g.nr) return fail(MLG_E_ARG, "N_r^c out of range");
    if (g.nphic < 0 || g.nphic > g.nphi / 2 + 1) return fail(MLG_E_ARG, "N_phi^c out of range");
    if (g.dealias != 0 && g.dealias != 1) return fail(MLG_E_ARG, "dealias must be 0 or 1");
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev)
    return fail(MLG_E_ARG, "device index out of range or no HIP device");
  int prev = -1;
  (void)hipGetDevice(&prev);
  if (hipSetDevice(device) != hipSuccess) return fail(MLG_E_DEVICE, "hipSetDevice failed");
  mlg_batch_s* bt = new (std::nothrow) mlg_batch_s();
  if (!bt) return fail(MLG_E_ALLOC, "host allocation failed");
  bt->count = count;
  bt->device = device;
  bt->prec = prec;
  hipDeviceProp_t prop;
  (void)hipGetDeviceProperties(&prop, device);
  bt->cus = prop.multiProcessorCount;
  std::vector<double> tab;
  std::vector<int64_t> tri;
  bt->spec_offsets.assign(count + 1, 0);
  int64_t mix = 0;
  for (int b = 0; b < count; ++b) {
    const mlg_grid& g = grids[b];
    BatchInst I{};
    I.nr = g.nr;
    I.nphi = g.nphi;
    I.nrc = g.nrc ? g.nrc : g.nr;
    I.M = g.nphic ? g.nphic : g.nphi / 2;
    const int nr = I.nr, nrc = I.nrc, M = I.M, nh = (nr + 1) / 2;
    I.mact = std::min({M, nrc, (g.nphi + 1) / 2, g.dealias ? (g.nphi - 1) / 3 + 1 : M});
    const size_t tri0 = tri.size();
    int64_t t = 0;
    for (int m = 0; m < M; ++m) {
      tri.push_back(t);
      t += std::max(nrc - m, 0);
    }
    tri.push_back(t);
    const int64_t tau = t;
    I.spec_off = bt->spec_offsets[b];
    bt->spec_offsets[b + 1] = I.spec_off + tau;
    I.mix_off = mix;
    mix += (int64_t)M * nr;
    std::vector<long double> th, wl;
    gl_theta(nr, th, wl);
    I.tb_off = (int64_t)tab.size();
    tab.resize(tab.size() + tau * nh);
    I.tf_off = (int64_t)tab.size();
    tab.resize(tab.size() + tau * nh);
    I.rec_off = (int64_t)tab.size();
    tab.resize(tab.size() + 2 * tau);
    I.start_off = (int64_t)tab.size();
    int64_t states = 0;
    for (int m = 0; m < M; ++m) states += rec_states(nrc - m);
    tab.resize(tab.size() + states * nh);
    I.node_off = (int64_t)tab.size();
    tab.resize(tab.size() + 2 * nh);
    I.tw_off = (int64_t)tab.size();
    tab.resize(tab.size() + 2 * g.nphi);
    std::vector<long double> col(nrc + 2);
    int64_t start = I.start_off;
    for (int i = 0; i < nh; ++i) {
      tab[I.node_off + i] = (double)cosl(th[i]);
      tab[I.node_off + nh + i] = (double)wl[i];
    }
    for (int m = 0; m < M; ++m) {
      const int K = std::max(nrc - m, 0);
      if (K == 0) continue;
      const int64_t tr = tri[tri0 + m];
      for (int i = 0; i < nh; ++i) {
        pbar_col(m, nrc, th[i], col.data());
        for (int t = 0; t < K; t += RC_S) {
          double* p = &tab[start + 2 * (t / RC_S) * nh + i];
          p[0] = t ? (double)col[t - 2] : -(double)col[0];
          p[nh] = t ? (double)col[t - 1] : 0.0;
        }
        for (int n = m; n < nrc; ++n) {
          tab[I.tb_off + (tr + n - m) * nh + i] = (double)col[n - m];
          tab[I.tf_off + tr * nh + (int64_t)i * K + (n - m)] = (double)(wl[i] * col[n - m]);
        }
      }
      start += rec_states(K) * nh;
      for (int n = m; n < nrc; ++n) {
        ld a = 0, c = n == m ? 1 : 0;
        if (n > m) a = sqrtl((ld)(4 * n * n - 1) / (ld)(n * n - m * m));
        if (n >= m + 2) {
          c = sqrtl((ld)((2 * n + 1) * (n - 1 - m) * (n - 1 + m)) / (ld)((2 * n - 3) * (n * n - m * m)));
        }
        tab[I.rec_off + 2 * (tr + n - m)] = (double)a;
        tab[I.rec_off + 2 * (tr + n - m) + 1] = (double)c;
      }
    }
    const ld pi = acosl(-1.0L);
    for (int q = 0; q < g.nphi; ++q) {
      tab[I.tw_off + 2 * q] = (double)cosl(-2 * pi * q / g.nphi);
      tab[I.tw_off + 2 * q + 1] = (double)sinl(-2 * pi * q / g.nphi);
    }
    bt->inst.push_back(I);
  }
  tab.resize(tab.size() + 2 * RC_F);  // read past the last column's recurrence
  bt->spec_total = bt->spec_offsets[count];
  bt->mix_total = mix;
  bt->ws_bytes = (size_t)mix * (prec == MLG_FP32 ? 8 : 16) + 256;
  mlg_status st;
  if ((st = up(&bt->d_tab, tab)) || (st = build_radial(bt, tri))) {
    free_batch(bt);
    if (prev >= 0) (void)hipSetDevice(prev);
    return st;
  }
  if (prec == MLG_FP32) {
    std::vector<float> t32(tab.begin(), tab.end());
    if ((st = up(&bt->d_tab32, t32))) {
      free_batch(bt);
      if (prev >= 0) (void)hipSetDevice(prev);
      return st;
    }
  }
  if ((st = build_phi(bt, bt->cfg.lines))) {
    free_batch(bt);
    if (prev >= 0) (void)hipSetDevice(prev);
    return st;
  }
  set_blocks(bt, bt->cfg);
  if (prev >= 0) (void)hipSetDevice(prev);
  *out = bt;
  return MLG_OK;
}

mlg_status mlg_batch_destroy(mlg_batch b) {
  free_batch(b);
  return MLG_OK;
}

mlg_status mlg_batch_query(mlg_batch b, int64_t* spec_offsets, int64_t* workspace_bytes) {
  if (!b) return fail(MLG_E_ARG, "batch is NULL");
  if (spec_offsets)
    for (int i = 0; i <= b->count; ++i) spec_offsets[i] = b->spec_offsets[i];
  if (workspace_bytes) *workspace_bytes = (int64_t)b->ws_bytes;
  return MLG_OK;
}

mlg_status mlg_batch_rhs_scalar(mlg_batch b, double gamma, const void* spec_in, void* spec_out, void* ws,
                                void* stream) {
  if (!b) return fail(MLG_E_ARG, "batch is NULL");
  if (!spec_in || !spec_out || !ws) return fail(MLG_E_ARG, "null buffer");
  if (spec_in == spec_out) return fail(MLG_E_ARG, "spec_in and spec_out must not alias");
  if (!std::isfinite(gamma)) return fail(MLG_E_ARG, "gamma must be finite");
  int prev = -1;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(b->device);
  mlg_status st = batch_run(b, gamma, spec_in, spec_out, ws, static_cast<hipStream_t>(stream), b->cfg);
  if (prev >= 0) (void)hipSetDevice(prev);
  return st;
}

mlg_status mlg_batch_set_config(mlg_batch b, const mlg_batch_config* c) {
  if (!b || !c) return fail(MLG_E_ARG, "null argument");
  if ((c->recurrence != 0 && c->recurrence != 1) || (c->threads != 64 && c->threads != 128 && c->threads != 256) ||
      c->blocks_per_cu < 1 || c->blocks_per_cu > 8 || c->lines < 2 || c->lines > 32 || (c->lines & 1))
    return fail(MLG_E_ARG, "invalid batch configuration");
  const size_t shm = batch_smem(b, c->lines);
  if (shm > 65536) return fail(MLG_E_ARG, "configuration needs more than 64 KiB of LDS");
  BatchConfig nc{c->recurrence, c->threads, c->blocks_per_cu, c->lines, {0, 0, 0}};
  int prev = -1;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(b->device);
  const mlg_status st = nc.lines != b->cfg.lines ? build_phi(b, nc.lines) : MLG_OK;
  set_blocks(b, nc);
  if (prev >= 0) (void)hipSetDevice(prev);
  if (st) return st;
  b->cfg = nc;
  return MLG_OK;
}

mlg_status mlg_batch_get_config(mlg_batch b, mlg_batch_config* c) {
  if (!b || !c) return fail(MLG_E_ARG, "null argument");
  c->recurrence = b->cfg.recurrence;
  c->threads = b->cfg.threads;
  c->blocks_per_cu = b->cfg.blocks_per_cu;
  c->lines = b->cfg.lines;
  return MLG_OK;
}

mlg_status mlg_batch_autotune(mlg_batch b, double gamma, const void* spec_in, void* spec_out, void* ws, void* stream,
                              mlg_batch_config* chosen, double* best_ms) {
  if (!b) return fail(MLG_E_ARG, "batch is NULL");
  if (!spec_in || !spec_out || !ws) return fail(MLG_E_ARG, "null buffer");
  int prev = -1;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(b->device);
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
    return fail(MLG_E_DEVICE, "hipEventCreate failed");
  const int lines_c[] = {4, 8, 16};
  const int thr_c[] = {128, 256};
  const int bpc_c[] = {1, 2, 4, 8};
  BatchConfig best = b->cfg;
  float best_t = 1e30f;
  mlg_status st = MLG_OK;
  for (int lines : lines_c) {
    if (batch_smem(b, lines) > 65536) continue;
    if ((st = build_phi(b, lines))) break;
    for (int rec = 0; rec < 2; ++rec)
      for (int thr : thr_c)
        for (int bpc : bpc_c) {
          BatchConfig c{rec, thr, bpc, lines, {0, 0, 0}};
          set_blocks(b, c);
          if ((st = batch_run(b, gamma, spec_in, spec_out, ws, s, c))) break;  // warm-up
          (void)hipEventRecord(e0, s);
          for (int r = 0; r < 3; ++r)
            if ((st = batch_run(b, gamma, spec_in, spec_out, ws, s, c))) break;
          (void)hipEventRecord(e1, s);
          if (st) break;
          (void)hipEventSynchronize(e1);
          float ms = 0;
          (void)hipEventElapsedTime(&ms, e0, e1);
          ms /= 3;
          if (ms < best_t) {
            best_t = ms;
            best = c;
          }
        }
    if (st) break;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st == MLG_OK) st = build_phi(b, best.lines);
  if (st == MLG_OK) {
    b->cfg = best;
    b->tuned = 1;
    if (chosen) {
      chosen->recurrence = best.recurrence;
      chosen->threads = best.threads;
      chosen->blocks_per_cu = best.blocks_per_cu;
      chosen->lines = best.lines;
    }
    if (best_ms) *best_ms = best_t;
  }
  if (prev >= 0) (void)hipSetDevice(prev);
  return st;
}

}  // extern "C"
