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
extern "C" int blocks(int gsz, int n4, int n2, int HU) { return pkv::ranked_blocks(pkv::RankedShape{gsz, n4, n2, true}, HU); }
extern "C" void unit(int block, int wv, int gsz, int n4, int n2, int HU, int n_seg, int* out) {
    const pkv::RankedUnit x = pkv::ranked_unit(block, wv, pkv::RankedShape{gsz, n4, n2, true}, HU, n_seg);
    out[0] = x.live; out[1] = x.UW; out[2] = x.first; out[3] = x.rank; out[4] = x.hu;
    out[5] = pkv::counted_units(wv / x.UW, 4 / x.UW, x.hu, HU);
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
    cus, out, one_round = 256, (C.c_int * 5)(), 0
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
        if segs * 32 <= resident * cus and N <= 4096:
            # several wavefronts per unit only where one round has room for them, or for a sixteenth each of the segments
            assert waves <= 1.03 * max(resident * cus, 1.25 * 32 * segs)
            one_round += 1
    assert one_round == (resident * cus // 32 - 32 if N <= 4096 else 0)


# Every workgroup of a ranked launch counts its units in once for each segment that it has units of, and a segment's counts add up
# to its units; no unit is counted in by a workgroup other than its own.
@pytest.mark.parametrize("HU", [1, 2, 3, 12, 25, 32, 40])
def test_counts_of_a_segment(shim, HU):
    out = (C.c_int * 6)()
    for n_seg, gsz, n4, n2 in ((1, 1, 0, 0), (7, 7, 2, 3), (50, 50, 12, 38), (130, 65, 8, 8), (97, 33, 33, 0), (640, 320, 60, 60)):
        total, units = [0] * n_seg, set()
        for block in range(shim.blocks(gsz, n4, n2, HU) * -(-n_seg // gsz)):
            mine = {}
            for wv in range(4):
                shim.unit(block, wv, gsz, n4, n2, HU, n_seg, out)
                live, UW, first, rank, hu, count = out
                if not live or wv % UW:
                    continue
                assert (first + rank, hu) not in units
                units.add((first + rank, hu))
                in_block, counts = mine.setdefault(first + rank, [0, 0])
                mine[first + rank] = [in_block + 1, counts + count]
            for seg, (in_block, counts) in mine.items():
                assert counts == in_block
                total[seg] += counts
        assert total == [HU] * n_seg and len(units) == n_seg * HU


def test_shapes_by_length_of_the_prompt(shim):
    """Where a shape made for few rows would lose on the many rows that a long prompt keeps, and back: bf16 rows of D 128."""
    out = (C.c_int * 5)()

    def shape(L, H, N):
        shim.shape(L, L * H, 256, N, 256, 20, out)
        return out[0] / L, out[1] / L

    for L, H in ((34, 32), (35, 32), (30, 40)):                    # up to 4.9 units per compute unit
        assert shape(L, H, 1000)[0] >= 0.23 and sum(shape(L, H, 1000)) == 1
        assert sum(shape(L, H, 400)) < 0.45
    assert sum(shape(40, 32, 1000)) == 0.5 and sum(shape(40, 32, 5000)) == 1
    assert sum(shape(64, 32, 5000)) == 0.25                        # what just fits a round of 20 does not do
    for L, H in ((80, 32), (96, 32), (100, 32)):
        assert sum(shape(L, H, 5000)) == 1
    assert shape(75, 32, 400) == (0, 19 / 75) and shape(80, 32, 818) == (0, 0.25)
