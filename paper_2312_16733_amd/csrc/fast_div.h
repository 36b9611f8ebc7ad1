// Division by a number that the host knows, as a multiplication and a shift (Granlund and Montgomery, "Division by Invariant
// Integers using Multiplication", 1994).
#pragma once

#if defined(__HIPCC__)
#define SNA_HD __host__ __device__ __forceinline__
#else
#define SNA_HD inline
#endif

namespace sna {

// x / d for 0 <= x < 2^31 and 1 <= d < 2^31.  With l = ceil(log2 d) the multiplier m is floor(2^(31 + l) / d) + 1, below 2^32.
// m d exceeds 2^(31 + l) by e, 0 < e <= d <= 2^l, so that x m / 2^(31 + l) exceeds x / d by x e / (d 2^(31 + l)) < 1 / d: no
// integer lies between the two.
struct FastDiv {
  unsigned m; int shift;            // shift < 0: d == 1
  static FastDiv by(int d) {
    if (d <= 1) return {0u, -1};
    int l = 1;
    while ((1ll << l) < d) ++l;
    return {(unsigned)(((1ull << (31 + l)) / (unsigned)d) + 1), l - 1};
  }
  SNA_HD int div(int x) const {
    return shift < 0 ? x : (int)((unsigned)(((unsigned long long)(unsigned)x * m) >> 32) >> shift);
  }
};

}  // namespace sna
