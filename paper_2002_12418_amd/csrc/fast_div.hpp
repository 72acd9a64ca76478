// Division by constants the host knows.
#pragma once
#include <hip/hip_runtime.h>

namespace mnnconv {

// Division of a value below 2^31 by a constant the host knows: q = mulhi(n, m) >> sh with m = ceil(2^(31+L) / d),
// L = ceil(log2 d), sh = L - 1 (exact for every n < 2^31).  A run-time division costs some thirty vector instructions,
// and the instruction count of the kernels that use this is part of their time.
struct FastDiv { unsigned m, sh, d; };
inline FastDiv make_fastdiv(unsigned d)
{
    FastDiv f{0u, 0u, d};
    if (d <= 1) return f;
    unsigned L = 0;
    while ((1u << L) < d) ++L;
    f.m = (unsigned)((((unsigned long long)1 << (31 + L)) + d - 1) / d);
    f.sh = L - 1;
    return f;
}
__device__ __forceinline__ unsigned fast_div(unsigned n, const FastDiv& f) { return f.d <= 1 ? n : (__umulhi(n, f.m) >> f.sh); }

// The same, for the same n < 2^31 (n + n has to fit), without a branch for d = 1: q = n * m >> (31 + L) with m = ceil(2^(31+L) / d), from 2^31 to 2^32 - 1.  For kernels whose time before the first load
// counts (sliding window on staged patches: places worked out in 0.8 us instead of 1.1; whole calls 5 x 5 128 -> 128 on 8 x 28 x 28 44.0 -> 41.1 us, 3 x 3 48 -> 96 on
// 24 x 40 x 40 28.1 -> 27.1, stride 2 64 -> 128 on 32 x 56 x 56 31.4 both).  Not everywhere: it takes registers, of which gemm_split.hip's gather and some transforms have none to spare (a wavefront per SIMD).
struct ConstDiv { unsigned m, L, d; };
inline ConstDiv make_constdiv(unsigned d)
{
    ConstDiv f{0u, 0u, d < 1 ? 1 : d};
    while ((1ull << f.L) < f.d) ++f.L;
    f.m = (unsigned)((((unsigned long long)1 << (31 + f.L)) + f.d - 1) / f.d);
    return f;
}
__device__ __forceinline__ unsigned const_div(unsigned n, const ConstDiv& f) { return __umulhi(n + n, f.m) >> f.L; }

}  // namespace mnnconv
