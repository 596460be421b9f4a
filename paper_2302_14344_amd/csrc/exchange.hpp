// Values passed between workgroups of one launch through the device's point of coherence.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"

namespace subadmm {

// A value and the number of the exchange it belongs to, in one 64-bit word (FP32) or two
// (FP64, half of the value in each): written and read with agent-scope atomics, so a reader that
// finds the tag it waits for has the value, and nothing has to be ordered or reset.
template <typename T>
struct Tagged;
template <>
struct Tagged<float> {
  static constexpr int N = kClusterWordsF32;
  __device__ static void put(unsigned long long* p, float v, uint32_t tag) {
    const unsigned long long x = ((unsigned long long)__float_as_uint(v) << 32) | tag;
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ static bool get(const unsigned long long* p, float* v, uint32_t tag) {
    const unsigned long long x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *v = __uint_as_float((uint32_t)(x >> 32));
    return (uint32_t)x == tag;
  }
};
template <>
struct Tagged<double> {
  static constexpr int N = kClusterWordsF64;
  __device__ static void put(unsigned long long* p, double v, uint32_t tag) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    __hip_atomic_store(p, (b & 0xffffffff00000000ull) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, (b << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ static bool get(const unsigned long long* p, double* v, uint32_t tag) {
    const unsigned long long h = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long l = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *v = __longlong_as_double((long long)((h & 0xffffffff00000000ull) | (l >> 32)));
    return (uint32_t)h == tag && (uint32_t)l == tag;
  }
};

}  // namespace subadmm
