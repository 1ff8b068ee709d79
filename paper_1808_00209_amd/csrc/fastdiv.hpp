// Division of unsigned 32-bit integers by a divisor that is fixed per launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bnn {

// Unsigned division by a run-time invariant divisor d >= 1 with a multiply
// and shifts (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994): exact for every 32-bit n.
struct FastDiv {
  uint32_t d, m;
  int s1, s2;
};

inline FastDiv make_fastdiv(uint32_t d) {
  int l = 0;
  while ((uint64_t{1} << l) < d) ++l;  // l = ceil(log2 d)
  FastDiv f;
  f.d = d;
  f.m = static_cast<uint32_t>(((uint64_t{1} << 32) * ((uint64_t{1} << l) - d)) / d + 1);
  f.s1 = l < 1 ? l : 1;
  f.s2 = l > 1 ? l - 1 : 0;
  return f;
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) {
  const uint32_t t = __umulhi(f.m, n);
  return (t + ((n - t) >> f.s1)) >> f.s2;
}

// The same for n < 2^31 with two shifts and one multiply: m = ceil(2^(31 + s)
// / d), s = ceil(log2 d), so m d - 2^(31 + s) < d <= 2^s and the error of
// 2 n m / 2^(32 + s) against n / d stays below 1 / d.
struct FastDiv31 {
  uint32_t d, m;
  int s;
};

inline FastDiv31 make_fastdiv31(uint32_t d) {
  FastDiv31 f;
  f.d = d;
  f.s = 0;
  while ((uint64_t{1} << f.s) < d) ++f.s;
  f.m = static_cast<uint32_t>(((uint64_t{1} << (31 + f.s)) + d - 1) / d);
  return f;
}

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv31& f) {
  return __umulhi(n << 1, f.m) >> f.s;
}

}  // namespace bnn
