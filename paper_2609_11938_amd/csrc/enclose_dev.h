// Device code of the enclosure shared by its own kernel and the compact
// path's last pass.
#pragma once
#include <type_traits>

#include "common.h"
#include "impl.h"

namespace opa {

// first index in [lo, hi) with a[idx] > x (or hi); called by a whole wave
__device__ inline int64_t wave_upper_bound(const uint64_t *a, int64_t lo, int64_t hi, uint64_t x) {
  const int l = lane_id();
  while (hi - lo > OPA_WAVE) {
    const int64_t step = (hi - lo + OPA_WAVE - 1) / OPA_WAVE;
    int64_t p = lo + (int64_t)(l + 1) * step - 1;
    if (p > hi - 1) p = hi - 1;
    const uint64_t m = __ballot(a[p] > x);
    if (m == 0) return hi;
    const int f = __ffsll((unsigned long long)m) - 1;
    const int64_t nlo = f == 0 ? lo : lo + (int64_t)f * step;
    int64_t pf = lo + (int64_t)(f + 1) * step - 1;
    if (pf > hi - 1) pf = hi - 1;
    lo = nlo;
    hi = pf + 1;
  }
  const int64_t p = lo + l;
  const uint64_t m = __ballot(p < hi && a[p] > x);
  return m ? lo + __ffsll((unsigned long long)m) - 1 : hi;
}

__device__ __forceinline__ int64_t thread_upper_bound(const uint64_t *a, int64_t lo, int64_t hi,
                                                      uint64_t x) {
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// the widest vector that kBytes bytes are a multiple of
template <int kBytes> struct VecBytes {
  static_assert(kBytes % 4 == 0, "whole words");
  using type = typename std::conditional<kBytes % 16 == 0, uint4,
               typename std::conditional<kBytes % 8 == 0, uint2, uint32_t>::type>::type;
};

// kPer consecutive elements from p[i..), vector loads when aligned
template <int kPer, typename T>
__device__ __forceinline__ void load_run(const T *p, int64_t i, int nv, T (&o)[kPer]) {
  using V = typename VecBytes<sizeof(T) * kPer>::type;
  constexpr int kB = (int)sizeof(V);
  if (nv == kPer && (reinterpret_cast<uintptr_t>(p + i) & (kB - 1)) == 0) {
    const V *v = reinterpret_cast<const V *>(p + i);
#pragma unroll
    for (int q = 0; q < (int)(sizeof(T) * kPer) / kB; ++q) {
      const V t = v[q];
      memcpy(reinterpret_cast<char *>(o) + kB * q, &t, kB);
    }
  } else {
#pragma unroll
    for (int k = 0; k < kPer; ++k) o[k] = k < nv ? p[i + k] : T(0);
  }
}

template <int kPer, typename T>
__device__ __forceinline__ void store_run(T *p, int64_t i, int nv, const T (&o)[kPer]) {
  using V = typename VecBytes<sizeof(T) * kPer>::type;
  constexpr int kB = (int)sizeof(V);
  if (nv == kPer && (reinterpret_cast<uintptr_t>(p + i) & (kB - 1)) == 0) {
    V *v = reinterpret_cast<V *>(p + i);
#pragma unroll
    for (int q = 0; q < (int)(sizeof(T) * kPer) / kB; ++q) {
      V t;
      memcpy(&t, reinterpret_cast<const char *>(o) + kB * q, kB);
      v[q] = t;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (k < nv) p[i + k] = o[k];
  }
}

}  // namespace opa
