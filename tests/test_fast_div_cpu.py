"""csrc/fast_div.hpp, compiled for the host: quotient and remainder by a precomputed multiplier, at the edges of the
quotients up to 400 and of a geometric sample of those beyond.  (That the quotient is at most one short for all of them follows from
the bound in the header.)"""
import ctypes as C
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_03409_amd", "csrc")
SHIM = """
#define __device__
#define __host__
#define __forceinline__ inline
#include "fast_div.hpp"
extern "C" int check(int d, int step) {     // the first n at which it is wrong, -1 if none
    const pkv::FastDiv f = pkv::fast_div(d);
    const long long top = 0x7fffffffll;
    for (long long q = 0; q * d <= top; q += 1 + q / step)
        for (long long n = q * d - 1; n <= q * d + 1; ++n) {
            if (n < 0 || n > top) continue;
            const pkv::DivMod x = pkv::div_mod((int)n, f);
            if (x.q != n / d || x.r != n % d) return (int)n;
        }
    const pkv::DivMod x = pkv::div_mod((int)top, f);
    return x.q == top / d && x.r == top % d ? -1 : (int)top;
}
"""


def test_quotients_and_remainders(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(tmp_path / "shim.cpp"), "-o", str(tmp_path / "shim.so")])
    lib = C.CDLL(str(tmp_path / "shim.so"))
    for d in [*range(1, 300), 511, 512, 513, 1000, 2047, 2048, 8191, 65535, 65536, 65537, 1 << 20, (1 << 30) - 1, 1 << 30, (1 << 31) - 1]:
        assert lib.check(d, 400) == -1, d
