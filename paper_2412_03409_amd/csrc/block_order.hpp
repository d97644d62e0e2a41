// Order of the blocks of a launch whose blocks differ in length.  Plain integer rules, apart from the kernels so that they
// can be compiled and enumerated on the host.
#pragma once

#include "fast_div.hpp"

namespace pkv {

struct HeadBlock { int head, rank; };     // head of the XCD, rank of the block in it: 0 is the longest

// Block j of an XCD that works on `heads` heads of nblk blocks each: head by head, the last `tail` heads longest block
// first.  With an even number of blocks every head starts at another rank, one further for each head and each 32
// workgroups: the hardware deals workgroups out in turn, and with ranks that repeat every 4, 6, 8, 12 or 16 of them some of
// an XCD's 32 compute units got the long blocks time and again (importance without a given log-sum-exp, B4 L32 H32/8 D128,
// us, ranks repeating / moving on: N900 1637 / 1343, N1500 3154 / 3014, N2048 5646 / 5052, N3000 11316 / 10655, N4096 20233
// / 18751; an odd number does that by itself, and moving on costs it 2 % at N2300).
__host__ __device__ __forceinline__ HeadBlock head_block(int j, int heads, FastDiv nblk, FastDiv tail) {
    const int n = (int)nblk.d, lead = heads - (int)tail.d;
    if (j < lead * n) {
        const DivMod x = div_mod(j, nblk);
        return {x.q, (n & 1) == 0 ? div_mod(x.r + x.q + x.q * n / 32, nblk).r : x.r};
    }
    const DivMod x = div_mod(j - lead * n, tail);
    return {lead + x.r, x.q};
}
__host__ __device__ __forceinline__ HeadBlock head_block(int j, int heads, int nblk, int tail) {
    return head_block(j, heads, fast_div(nblk), fast_div(tail));
}

// Whether the heads (B*L*H) fit a one-dimensional grid of whole heads per XCD, as many to each of the `xcds`, in which the bf16 kernels
// count them in 32 bits.  (The fp32 kernels have a two-dimensional one.)
inline bool heads_fit(long long heads, int xcds) { return (heads + xcds - 1) / xcds * xcds <= 0x7fffffffll; }

}  // namespace pkv
