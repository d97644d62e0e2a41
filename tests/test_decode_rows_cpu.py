"""csrc/decode_rows.hpp, compiled for the host.  Where the rows of a decode step come from: every row that takes part has
its own source, and no row, taking part or not, is read from a slot that the step writes or that holds nothing.  Ranked
launches: every unit of every segment has its wavefronts exactly once."""
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
extern "C" int row(int ev, int r, int r0, int len, int len_old, int app, int shift, int r_new, int r_mask) {
    const pkv::RingMap ring = {shift, r_new, r_mask};
    const pkv::RowSource s = ev ? pkv::row_source<true>(r, r0, len, len_old, app, ring)
                                : pkv::row_source<false>(r, r0, len, len_old, app, ring);
    return s.slot * 4 + s.from_new * 2 + s.valid;
}
extern "C" void unit(int block, int wv, int gsz, int n4, int n2, int HU, int n_seg, int* out) {
    const pkv::RankedShape s = {gsz, n4, n2, true};
    const pkv::RankedUnit x = pkv::ranked_unit(block, wv, s, HU, n_seg);
    const int v[7] = {x.live, x.UW, x.first, x.n, x.rank, x.hu, pkv::ranked_blocks(s, HU)};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
extern "C" void shape(int gsz, long long units, long long cus, int N, int row_bytes, int* out) {
    pkv::RankedShape s = {gsz, -1, -1, false};
    pkv::ranked_shape(s, units, cus, N, row_bytes);
    out[0] = s.n4; out[1] = s.n2; out[2] = s.by_length;
}
extern "C" int length_class(int cap, int longest) { return pkv::length_class(cap, longest); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                           str(d / "shim.so")])
    return C.CDLL(str(d / "shim.so"))


@pytest.fixture(scope="module")
def row(shim):
    f = shim.row

    def call(*a):
        x = f(*map(int, a))
        return bool(x & 1), bool(x & 2), x >> 2
    return call


@pytest.mark.parametrize("block", [8, 16, 32])
def test_plain_step(row, block):
    for len_old in range(0, 70):
        for app in (False, True):
            ln = len_old + app
            for r0 in range(0, ln, block):
                for r in range(r0, r0 + block):
                    valid, new, slot = row(0, r, r0, ln, len_old, app, 0, -1, -1)
                    assert valid == (r < ln)
                    if valid:
                        assert new == (r == len_old) and (new or slot == r)
                    assert new or 0 <= slot < len_old, (len_old, app, r0, r)
                    assert not new or app


@pytest.mark.parametrize("block", [8, 16, 32])
@pytest.mark.parametrize("d", [1, 2, 7, 16])
def test_pruning_step(row, block, d):
    for base in (1, 2, 15, 16, 17, 31, 32, 40):
        for t in range(1, 3 * d + 4):
            for grown in (0, 1, 2, 9):
                if grown > max(0, t - 1 - d):
                    continue
                perm = base + grown                       # permanent entries before the step
                for grad in ((False, True) if t > d else (False,)):
                    ring0 = perm + 3                      # first ring slot
                    held = min(t, d + 1)                  # ring slots in use, this step's token among them
                    new_slot, decided = (t - 1) % (d + 1), t % (d + 1)
                    ln, r_new = perm + held, perm + new_slot
                    r_mask = perm + decided if t > d and not grad else -1
                    written = {ring0 + new_slot} | ({perm} if grad else set())
                    for r0 in range(0, ln, block):
                        for r in range(r0, r0 + block):
                            valid, new, slot = row(1, r, r0, ln, perm, True, ring0 - perm, r_new, r_mask)
                            assert valid == (r < ln and r != r_mask)
                            if valid:
                                assert new == (r == r_new)
                                assert new or slot == (r if r < perm else ring0 + r - perm)
                            if not new:
                                assert 0 <= slot < perm or ring0 <= slot < ring0 + held
                                assert slot not in written, (base, t, perm, grad, r0, r)


@pytest.mark.parametrize("HU", [1, 2, 3, 4, 5, 6, 7, 32, 41])
@pytest.mark.parametrize("n_seg,gsz,n4,n2", [
    (33, 33, 4, 4), (7, 7, 0, 0), (9, 9, 1, 8), (64, 64, 64, 0), (65, 65, 0, 65), (70, 35, 5, 3), (71, 36, 1, 1),
    (540, 270, 33, 33), (1037, 346, 43, 43), (13, 4, 2, 1), (5, 2, 0, 1), (1030, 344, 0, 0),
])
def test_ranked_units(shim, HU, n_seg, gsz, n4, n2):
    out = (C.c_int * 7)()
    groups = (n_seg + gsz - 1) // gsz
    shim.unit(0, 0, gsz, n4, n2, HU, n_seg, out)
    seen, without = {}, 0
    for block in range(out[6] * groups):
        uws, lives = set(), []
        for wv in range(4):
            shim.unit(block, wv, gsz, n4, n2, HU, n_seg, out)
            live, UW, first, n, rank, hu, _ = out
            uws.add(UW)
            lives.append(bool(live))
            without += not live and block < out[6] and n_seg >= gsz
            if live:
                assert 0 <= hu < HU and 0 <= rank < n <= gsz and first + n <= n_seg and first % gsz == 0
                assert UW == (4 if rank < n4 else 2 if rank < n4 + n2 else 1)
                seen.setdefault((first, rank, hu), []).append((block, wv))
        assert len(uws) == 1
        UW = uws.pop()      # the wavefronts of a unit agree, so a workgroup of one unit may leave as a whole
        assert all(len(set(lives[i:i + UW])) == 1 for i in range(0, 4, UW))
    assert len(seen) == n_seg * HU
    assert without <= 2 + 3      # wavefronts of a full group without a unit: at most the last workgroups of two classes
    for (first, rank, hu), who in seen.items():
        UW = 4 if rank < n4 else 2 if rank < n4 + n2 else 1
        assert len(who) == UW and len({b for b, _ in who}) == 1
        assert sorted(w & (UW - 1) for _, w in who) == list(range(UW))
        assert len({w & ~(UW - 1) for _, w in who}) == 1


def test_ranked_shapes(shim):
    out = (C.c_int * 3)()
    for cus in (32, 256, 304):
        for gsz in (1, 5, 8, 33, 64, 65, 512):
            for units in [4 * cus + 1, *(int(4 * cus * 1.07 ** i) for i in range(1, 60))]:
                for N, row_bytes in ((1, 128), (384, 256), (385, 256), (192, 512), (4096, 256), (4097, 128), (8192, 512)):
                    shim.shape(gsz, units, cus, N, row_bytes, out)
                    n4, n2, by_length = out
                    assert 0 <= n4 and 0 <= n2 and n4 + n2 <= gsz
                    assert by_length or n4 == n2 == 0
                    waves = 4 * n4 + 2 * n2 + (gsz - n4 - n2)
                    if N <= 4096 and gsz >= 64 and units <= 3 * 4 * cus:      # one round as long as that is possible
                        assert waves * units <= 1.03 * 16 * cus * gsz, (cus, gsz, units, N, n4, n2)


def test_length_classes(shim):
    for longest in (1, 2, 3, 100, 8192, (1 << 20) - 1):
        last = 15
        for cap in range(0, longest + 1, max(1, longest // 3000)):
            c = shim.length_class(cap, longest)
            assert 0 <= c <= last
            last = c
        assert shim.length_class(longest, longest) == 0
