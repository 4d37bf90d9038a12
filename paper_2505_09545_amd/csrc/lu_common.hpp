// Device helpers shared by the LU's kernels (lu.hip, tiles.hip, solve_step.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <utility>

#include "gdm_common.hpp"

namespace gdm {

// 16 x 16 x 4 products; rows of the result in register q of lane group lk: 4 lk + q
// (FP32), lk + 4 q (FP64)
template <typename T> struct acc_of;
template <> struct acc_of<double> { using type = v4d; };
template <> struct acc_of<float> { using type = v4f; };
__device__ inline v4d mfma16(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline v4f mfma16(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <typename CT> __device__ inline CT cmul_t(CT a, CT b) {
  CT r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  return r;
}
// t - l u: one entry of a rank-1 update
template <typename CT> __device__ inline CT r1_upd(CT t, const CT& l, const CT& u) {
  // four fused multiply-adds
  t.x = fma(l.y, u.y, fma(-l.x, u.x, t.x));
  t.y = fma(-l.y, u.x, fma(-l.x, u.y, t.y));
  return t;
}
template <typename CT> __device__ inline CT cinv_t(CT a) {
  // 1/a = conj(a) / |a|^2, with a scaled by the power of two 2^-e of its larger
  // component (exact) so that |a|^2 can neither overflow nor underflow; one
  // division (a = 0 gives NaN, as the quotient form did)
  const auto s = fabs(a.x) > fabs(a.y) ? fabs(a.x) : fabs(a.y);
  int e;
  (void)frexp(s, &e);
  const auto ar = ldexp(a.x, -e), ai = ldexp(a.y, -e);
  const auto id = 1 / (ar * ar + ai * ai);
  CT r;
  r.x = ldexp(ar * id, -e);
  r.y = ldexp(-ai * id, -e);
  return r;
}
// |re| + |im| as partial pivoting compares it
template <typename CT> __device__ inline float cabs1_f(const CT& v) { return (float)(fabs(v.x) + fabs(v.y)); }

// f(0), f(1), ..., f(N - 1) with compile-time indices (expanded whatever the
// unroller decides, so register arrays indexed by them stay in registers)
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace gdm
