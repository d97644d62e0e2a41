"""csrc/decode_rows.hpp, compiled for the host: the shape of a ranked launch on a compute unit that holds more than 16 wavefronts,
and the LDS it asks for."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_03409_amd", "csrc")
SHIM = """
#define __device__
#define __host__
#define __forceinline__ inline
#include "decode_rows.hpp"
extern "C" void shape(int gsz, long long units, long long cus, int N, int row_bytes, int resident, int* out) {
    pkv::RankedShape s = {gsz, -1, -1, false};
    pkv::ranked_shape(s, units, cus, N, row_bytes, resident);
    const long long segs = (units + 31) / 32, waves = 4ll * pkv::ranked_blocks(s, 32) * ((segs + gsz - 1) / gsz);
    out[0] = s.n4; out[1] = s.n2; out[2] = s.by_length; out[3] = pkv::ranked_lds(s, waves, cus); out[4] = (int)waves;
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("resident")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                           str(d / "shim.so")])
    return C.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("resident", [16, 20])
@pytest.mark.parametrize("N,row_bytes", [(128, 256), (384, 256), (385, 256), (4096, 256), (8192, 256)])
def test_shape_and_lds(shim, resident, N, row_bytes):
    cus, out = 256, (C.c_int * 5)()
    for segs in range(33, 1025):                          # of 32 units each
        groups = (segs + 511) // 512
        gsz = (segs + groups - 1) // groups
        shim.shape(gsz, segs * 32, cus, N, row_bytes, resident, out)
        n4, n2, by_length, lds, waves = out
        assert 0 <= n4 and 0 <= n2 and n4 + n2 <= gsz
        assert by_length or n4 == n2 == 0
        assert by_length or segs * 32 >= 16 * cus
        assert lds in (0, 31 << 10) and lds + 4 * 130 * 4 <= 64 << 10
        if lds:
            assert by_length and waves > 20 * cus
        if 20 * cus >= segs * 32 > 2.5 * 16 * cus and N <= 4096 and resident == 20:
            assert waves <= 1.03 * 20 * cus              # one round
