// In-register DFTs of the lengths 2, 3, 4, 5, 6, 8, 9, 10, 12, 15 and 16, shared by the FFTs of fft_mix.hip and batch.hip.
#pragma once

#include "dev_common.h"

namespace mlg {
namespace dev {

// cos and sin of 2 pi j / R
template <int R>
struct Root;
template <>
struct Root<6> {
  static constexpr double c[6] = {1.0, 0.5, -0.5, -1.0, -0.5, 0.5};
  static constexpr double s[6] = {0.0, 0.8660254037844386, 0.8660254037844386, 0.0, -0.8660254037844386,
                                  -0.8660254037844386};
};
template <>
struct Root<8> {
  static constexpr double c[8] = {1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0, -0.7071067811865476, 0.0,
                                  0.7071067811865476};
  static constexpr double s[8] = {0.0, 0.7071067811865476, 1.0, 0.7071067811865476, 0.0, -0.7071067811865476, -1.0,
                                  -0.7071067811865476};
};
template <>
struct Root<9> {
  static constexpr double c[9] = {1.0, 0.766044443118978, 0.17364817766693036, -0.5, -0.9396926207859084,
                                  -0.9396926207859084, -0.5, 0.17364817766693036, 0.766044443118978};
  static constexpr double s[9] = {0.0, 0.6427876096865394, 0.984807753012208, 0.8660254037844386,
                                  0.3420201433256687, -0.3420201433256687, -0.8660254037844386, -0.984807753012208,
                                  -0.6427876096865394};
};
template <>
struct Root<10> {
  static constexpr double c[10] = {1.0, 0.8090169943749475, 0.30901699437494745, -0.30901699437494745,
                                   -0.8090169943749475, -1.0, -0.8090169943749475, -0.30901699437494745,
                                   0.30901699437494745, 0.8090169943749475};
  static constexpr double s[10] = {0.0, 0.5877852522924731, 0.9510565162951535, 0.9510565162951535,
                                   0.5877852522924731, 0.0, -0.5877852522924731, -0.9510565162951535,
                                   -0.9510565162951535, -0.5877852522924731};
};
template <>
struct Root<12> {
  static constexpr double c[12] = {1.0, 0.8660254037844386, 0.5, 0.0, -0.5, -0.8660254037844386, -1.0,
                                   -0.8660254037844386, -0.5, 0.0, 0.5, 0.8660254037844386};
  static constexpr double s[12] = {0.0, 0.5, 0.8660254037844386, 1.0, 0.8660254037844386, 0.5, 0.0, -0.5,
                                   -0.8660254037844386, -1.0, -0.8660254037844386, -0.5};
};
template <>
struct Root<15> {
  static constexpr double c[15] = {1.0, 0.9135454576426009, 0.6691306063588582, 0.30901699437494745,
                                   -0.10452846326765347, -0.5, -0.8090169943749475, -0.9781476007338057,
                                   -0.9781476007338057, -0.8090169943749475, -0.5, -0.10452846326765347,
                                   0.30901699437494745, 0.6691306063588582, 0.9135454576426009};
  static constexpr double s[15] = {0.0, 0.4067366430758002, 0.7431448254773942, 0.9510565162951535,
                                   0.9945218953682733, 0.8660254037844386, 0.5877852522924731, 0.20791169081775934,
                                   -0.20791169081775934, -0.5877852522924731, -0.8660254037844386,
                                   -0.9945218953682733, -0.9510565162951535, -0.7431448254773942,
                                   -0.4067366430758002};
};
template <>
struct Root<16> {
  static constexpr double c[16] = {1.0, 0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0,
                                   -0.3826834323650898, -0.7071067811865476, -0.9238795325112867, -1.0,
                                   -0.9238795325112867, -0.7071067811865476, -0.3826834323650898, 0.0,
                                   0.3826834323650898, 0.7071067811865476, 0.9238795325112867};
  static constexpr double s[16] = {0.0, 0.3826834323650898, 0.7071067811865476, 0.9238795325112867, 1.0,
                                   0.9238795325112867, 0.7071067811865476, 0.3826834323650898, 0.0,
                                   -0.3826834323650898, -0.7071067811865476, -0.9238795325112867, -1.0,
                                   -0.9238795325112867, -0.7071067811865476, -0.3826834323650898};
};

// multiply by exp(-+ 2 pi i J / R) (forward: minus); J and R are compile-time constants after unrolling
template <int R, bool INV>
__device__ __forceinline__ double2 rot(double2 a, int J) {
  if (J == 0) return a;
  if (4 * J == R) return cmul_mi(a, INV);
  if (2 * J == R) return make_double2(-a.x, -a.y);
  if (4 * J == 3 * R) return cmul_mi(a, !INV);
  return cmul(a, make_double2(Root<R>::c[J], INV ? Root<R>::s[J] : -Root<R>::s[J]));
}

// In-register DFT of length R: v[n] -> V[k] = sum_n v[n] exp(-+ 2 pi i n k / R)
template <int R, bool INV>
struct Dft;
template <bool INV>
struct Dft<2, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[2]) {
    const double2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};
template <bool INV>
struct Dft<3, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[3]) {
    constexpr double h = 0.86602540378443864676;  // sqrt(3) / 2
    const double2 t1 = cadd(v[1], v[2]), t3 = cmul_mi(cscale(csub(v[1], v[2]), h), INV);
    const double2 t2 = make_double2(v[0].x - 0.5 * t1.x, v[0].y - 0.5 * t1.y);
    v[0] = cadd(v[0], t1);
    v[1] = cadd(t2, t3);
    v[2] = csub(t2, t3);
  }
};
template <bool INV>
struct Dft<4, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[4]) {
    const double2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const double2 t2 = cadd(v[1], v[3]), t3 = cmul_mi(csub(v[1], v[3]), INV);
    v[0] = cadd(t0, t2);
    v[1] = cadd(t1, t3);
    v[2] = csub(t0, t2);
    v[3] = csub(t1, t3);
  }
};
template <bool INV>
struct Dft<5, INV> {
  static __device__ __forceinline__ void run(double2 (&v)[5]) {
    constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;  // cos 2 pi / 5, cos 4 pi / 5
    constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;   // sin 2 pi / 5, sin 4 pi / 5
    const double2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]), t3 = csub(v[1], v[4]), t4 = csub(v[2], v[3]);
    const double2 r1 = make_double2(v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y);
    const double2 r2 = make_double2(v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y);
    const double2 i1 = cmul_mi(make_double2(s1 * t3.x + s2 * t4.x, s1 * t3.y + s2 * t4.y), INV);
    const double2 i2 = cmul_mi(make_double2(s2 * t3.x - s1 * t4.x, s2 * t3.y - s1 * t4.y), INV);
    v[0] = cadd(v[0], cadd(t1, t2));
    v[1] = cadd(r1, i1);
    v[4] = csub(r1, i1);
    v[2] = cadd(r2, i2);
    v[3] = csub(r2, i2);
  }
};
// R = A B: n = B n1 + n2, k = k1 + A k2
template <int A, int B, bool INV>
struct DftAB {
  static __device__ __forceinline__ void run(double2 (&v)[A * B]) {
    double2 y[A][B];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
      double2 t[A];
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) t[n1] = v[B * n1 + n2];
      Dft<A, INV>::run(t);
#pragma unroll
      for (int k1 = 0; k1 < A; ++k1) y[k1][n2] = rot<A * B, INV>(t[k1], n2 * k1);
    }
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
      Dft<B, INV>::run(y[k1]);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = y[k1][k2];
    }
  }
};
template <bool INV> struct Dft<6, INV> : DftAB<2, 3, INV> {};
template <bool INV> struct Dft<8, INV> : DftAB<2, 4, INV> {};
template <bool INV> struct Dft<9, INV> : DftAB<3, 3, INV> {};
template <bool INV> struct Dft<10, INV> : DftAB<2, 5, INV> {};
template <bool INV> struct Dft<12, INV> : DftAB<3, 4, INV> {};
template <bool INV> struct Dft<15, INV> : DftAB<3, 5, INV> {};
template <bool INV> struct Dft<16, INV> : DftAB<4, 4, INV> {};

}  // namespace dev
}  // namespace mlg
