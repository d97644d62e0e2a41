// Division by a number that a launch fixes: the compiler's takes some 25 dependent scalar and vector instructions (64-bit ones several
// times that), and a workgroup's start has several in a row.  Plain integer rules, apart from the kernels so that they can be
// compiled and enumerated on the host.
#pragma once

#include <stdint.h>

namespace pkv {

struct FastDiv { uint32_t d, mul; };                      // mul = floor(2^32 / d), of 1 one less
inline FastDiv fast_div(long long d) { return {(uint32_t)d, d <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (unsigned long long)d)}; }

struct DivMod { int q, r; };
// n / d and n % d for 0 <= n < 2^31: n * mul / 2^32 is less than one below n / d.
__host__ __device__ __forceinline__ DivMod div_mod(int n, FastDiv f) {
    uint32_t q = (uint32_t)(((uint64_t)(uint32_t)n * f.mul) >> 32), r = (uint32_t)n - q * f.d;
    const bool one = r >= f.d;
    return {(int)(q + (one ? 1u : 0u)), (int)(one ? r - f.d : r)};
}

#ifdef __HIP__
// The same of a value that is uniform in the wavefront: the compiler would select by vector instructions.
__device__ __forceinline__ DivMod uniform_div_mod(int n, FastDiv f) {
    const DivMod x = div_mod(n, f);
    return {__builtin_amdgcn_readfirstlane(x.q), __builtin_amdgcn_readfirstlane(x.r)};
}
#endif

}  // namespace pkv
