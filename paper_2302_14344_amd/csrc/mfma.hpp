// Small dense tiles on the matrix cores, shared by the factorisations: 16 x 16 tile products and
// the factorisation and inversion of a 16 x 16 diagonal tile by one wave.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <type_traits>
#include <utility>

namespace subadmm {

// 16 x 16 tile products on the matrix cores, FP64 (v_mfma_f64_16x16x4f64) and FP32
// (v_mfma_f32_16x16x4f32).  A 16-deep product is four instructions s = 0..3; in each, lane l
// supplies A[l % 16][k] and B[k][l % 16] for one k of the four, and the result lane l,
// register r holds D[row][l % 16].  With g = l / 16:
//   FP64: row = 4 r + g;   FP32: row = 4 g + r.
// The products below take k = row(s, g) (Mfma<F>::k), so that a result serves as the B
// operand of a following product as it stands; any other one-to-one choice of k only
// reorders the sum of a tile product.
typedef double v4f64 __attribute__((ext_vector_type(4)));
typedef float v4f32 __attribute__((ext_vector_type(4)));

template <typename F>
struct Mfma;

template <>
struct Mfma<double> {
  typedef v4f64 V;
  static __device__ inline int k(int s, int g) { return 4 * s + g; }
  static __device__ inline V mul(const double* a, const double* b, V c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
    return c;
  }
};

template <>
struct Mfma<float> {
  typedef v4f32 V;
  static __device__ inline int k(int s, int g) { return 4 * g + s; }
  static __device__ inline V mul(const float* a, const float* b, V c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], c, 0, 0, 0);
    return c;
  }
};

// Explicit fused multiply-add: the same rounding wherever the code is inlined.
__device__ inline float tfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double tfma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <int... Is, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, Is...>, F&& f) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

// Value of lane kLane of each row of 16 lanes, in all lanes of the row (DPP row_newbcast).
template <int kLane>
__device__ inline float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + kLane, 0xf, 0xf, true));
}
template <int kLane>
__device__ inline double row_bcast(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), 0x150 + kLane, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x150 + kLane, 0xf, 0xf, true);
  return __longlong_as_double(((long long)(unsigned)hi << 32) | (long long)(unsigned)lo);
}

// 1 / sqrt(d), d positive and normal: the hardware estimate refined by Newton steps, two in FP64
// (the estimate is good to ~2^-24 there).
__device__ inline double rsqrt_refined(double d) {
  double y = __builtin_amdgcn_rsq(d);
#pragma unroll
  for (int k = 0; k < 2; ++k) y = __builtin_fma(0.5 * y, __builtin_fma(-(d * y), y, 1.0), y);
  return y;
}
__device__ inline float rsqrt_refined(float d) {
  const float y = __builtin_amdgcn_rsqf(d);
  return __builtin_fmaf(0.5f * y, __builtin_fmaf(-(d * y), y, 1.0f), y);
}

// Cholesky factor L of the jb x jb (jb <= 16) tile at D (lower triangle, leading dimension ld)
// and, in its place, L^-1 (lower; the strict upper triangle is not touched).  One wave, its four
// rows of 16 lanes doing the same: lane r (mod 16) holds row r of the tile and column r of the
// inverse in registers; step j broadcasts column j of L within the lane rows, which serves the
// tile's update and the forward substitution of the identity alike.  Every index is a constant
// (a run-time one would cost a select per register).  A pivot that is not positive is
// taken as one; returns whether all were positive and finite.  Out of line: its 64 registers of tile entries
// would otherwise weigh on every caller (inlined, the multi-step kernel's iteration spilled).
// Bound by the chain of a column (broadcast, reciprocal square root, scale, broadcast, update:
// ~300 cycles) and 120 updates: ~6,400 cycles for a full tile.
// keep (leading dimension ldk), where the caller gives one, receives L itself.
template <typename C, typename P, typename Q = std::nullptr_t>
__device__ __attribute__((noinline)) bool diag_tile(P D, int ld, int jb, Q keep = nullptr, int ldk = 0) {
  const int lane = threadIdx.x & 63, r = lane & 15;
  C row[16], x[16];
  static_for<16>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    const bool in = r < jb && c <= r;
    const C v = D[in ? (long)r * ld + c : 0];
    row[c] = in ? v : (C)0;
    x[c] = c == r ? (C)1 : (C)0;
  });
  bool ok = true;
  static_for<16>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    if (j < jb) {
      C d = row_bcast<j>(row[j]);
      const bool good = d > (C)0;
      ok = ok && good && __builtin_isfinite(d);
      d = good ? d : (C)1;
      const C iv = rsqrt_refined(d);
      const C lj = row[j] * iv;  // L[r][j]
      if constexpr (!std::is_same<Q, std::nullptr_t>::value)
        if (lane < jb && r >= j) keep[(long)r * ldk + j] = r == j ? d * iv : lj;
      x[j] *= iv;
      static_for<15 - j>([&](auto qc) {
        constexpr int c = j + 1 + decltype(qc)::value;
        const C lc = row_bcast<c>(lj);  // L[c][j]; zero beyond the tile
        row[c] = tfma(-lj, lc, row[c]);
        x[c] = tfma(-lc, x[j], x[c]);
      });
    }
  });
  static_for<16>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    if (lane < 16 && q >= r && q < jb) D[(long)q * ld + r] = x[q];
  });
  return ok;
}

}  // namespace subadmm
