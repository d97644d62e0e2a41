"""Where the rows of a decode step come from (csrc/decode_rows.hpp, compiled for the host): every row that takes part has
its own source, and no row, taking part or not, is read from a slot that the step writes or that holds nothing."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_03409_amd", "csrc")
SHIM = """
#define __device__
#define __forceinline__ inline
#include "decode_rows.hpp"
extern "C" int row(int ev, int r, int r0, int len, int len_old, int app, int shift, int r_new, int r_mask) {
    const pkv::RingMap ring = {shift, r_new, r_mask};
    const pkv::RowSource s = ev ? pkv::row_source<true>(r, r0, len, len_old, app, ring)
                                : pkv::row_source<false>(r, r0, len, len_old, app, ring);
    return s.slot * 4 + s.from_new * 2 + s.valid;
}
"""


@pytest.fixture(scope="module")
def row(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                           str(d / "shim.so")])
    f = C.CDLL(str(d / "shim.so")).row

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
