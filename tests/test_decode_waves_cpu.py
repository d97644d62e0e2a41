"""csrc/decode_rows.hpp, compiled for the host: the slot that a wavefront reads for each row of a block whose new row comes from
k_new, the target test of a pruning step, how many wavefronts a unit of a grouped launch has, and which units its workgroups take."""
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
extern "C" int slot(int ev, int r, int r0, int len, int len_old, int r_new, int shift, int r_mask) {
    const pkv::RingMap ring = {shift, r_new, r_mask};
    return ev ? pkv::row_slot<true>(r, r0, len, len_old, r_new, ring) : pkv::row_slot<false>(r, r0, len, len_old, r_new, ring);
}
extern "C" int within(int entries, int base, int N, int t) { return pkv::within_target(entries, base, N, t); }
extern "C" int waves(int blocks, int HU, int W) { return pkv::active_waves(blocks, HU, W); }
extern "C" int blocks(int HU, int waves, int W) { return pkv::grouped_blocks(HU, waves, W); }
extern "C" int unit(int block, int wv, int waves, int W, int HU) { const pkv::GroupedUnit x = pkv::grouped_unit(block, wv, waves, W, HU); return x.live ? x.hu : -1 - x.hu; }
extern "C" int counted(int at, int units, int hu, int HU) { return pkv::counted_units(at, units, hu, HU); }
extern "C" int segment(int x, int y, int n_seg) { return pkv::grouped_segment(x, y, pkv::grouped_turn(n_seg), pkv::fast_div(n_seg)); }
extern "C" int grouped(int n_seg, int HU, int nl, int L, int N, int row_bytes) { return pkv::units_grouped(n_seg, HU, nl, L, 256, N, row_bytes); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("waves")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return C.CDLL(str(d / "shim.so"))


@pytest.mark.parametrize("block", [8, 16, 32])
def test_slots_of_a_plain_step(lib, block):
    for len_old in range(0, 70):
        for app in (0, 1):
            ln = len_old + app
            if app and ln == 1:
                continue                                  # k_new stands in for the whole segment
            for r0 in range(0, ln, block):
                for r in range(r0, r0 + block):
                    s = lib.slot(0, r, r0, ln, len_old, len_old if app else -1, 0, -1)
                    assert 0 <= s < len_old, (len_old, app, r0, r)   # stored before, not written in this step
                    if r < len_old:
                        assert s == r


@pytest.mark.parametrize("block", [8, 16, 32])
@pytest.mark.parametrize("d", [1, 2, 7, 16, 40])
def test_slots_of_a_pruning_step(lib, block, d):
    for perm in (0, 1, 2, 15, 16, 17, 31, 32, 40):
        cap = perm + 3 + d + 1
        ring0 = cap - (d + 1)
        for t in range(1, 3 * d + 4):
            ln = perm + min(t, d + 1)
            if ln == 1:
                continue
            r_new = perm + (t - 1) % (d + 1)
            for grad in ((0, 1) if t > d else (1,)):
                r_mask = -1 if grad else perm + t % (d + 1)
                stored = {j % (d + 1) for j in range(max(0, t - 1 - d), t - 1)}      # ring slots of the tokens before this one
                for r0 in range(0, ln, block):
                    for r in range(r0, r0 + block):
                        s = lib.slot(1, r, r0, ln, perm, r_new, ring0 - perm, r_mask)
                        assert 0 <= s < cap and s != ring0 + (t - 1) % (d + 1)       # not the slot that the step writes
                        assert s < perm or s - ring0 in stored, (perm, t, r0, r)     # nor one that holds nothing
                        if r < ln and r not in (r_new, r_mask):
                            assert s == (r if r < perm else r + ring0 - perm)


def test_target_without_a_division(lib):
    for N in (1, 2, 7, 680, 8192):
        for base in {0, 1, N // 3, N}:
            for t in (1, 2, 5, 63, 64, 1000, 1 << 30):
                target = max(1, (2 * base * (N + t) + N) // (2 * N))
                for entries in {2, 3, target - 1, target, target + 1, 1 << 20}:
                    if entries >= 2:
                        assert lib.within(entries, base, N, t) == (entries <= target), (N, base, t, entries)


def test_active_waves(lib):
    for W in (4, 8):
        for HU in (1, 2, 3, 5, 9, 32):
            last = 1
            for blocks in range(0, 600):
                n = lib.waves(blocks, HU, W)
                assert n in (1, 2, 4, 8) and last <= n <= W
                assert n == W or (blocks <= n * 4 and n * HU >= W)       # no wavefront idle that a unit could have
                assert n == 1 or blocks > n // 2 * 4 or n // 2 * HU < W
                last = n


@pytest.mark.parametrize("HU", [1, 2, 3, 9, 10, 12, 14, 32, 40])
@pytest.mark.parametrize("W", [4, 8])
@pytest.mark.parametrize("n_seg", [1, 2, 7, 13, 16, 24, 40, 63, 64, 65])
def test_units_of_a_grouped_launch(lib, HU, W, n_seg):
    """A grid of n_seg x HU: every unit once with all its wavefronts, counts that add up to HU in each segment, and no index beyond the
    segments or HU, in wavefronts to spare too; the workgroups of a segment on all XCDs."""
    widths = [w for w in (1, 2, 4, 8) if w <= W]
    waves = [widths[s % len(widths)] for s in range(n_seg)]              # as the capacities have it
    seen, counts, xcds = [[] for _ in waves], [0] * n_seg, [[0] * 8 for _ in waves]
    for y in range(HU):
        for x in range(n_seg):
            seg = lib.segment(x, y, n_seg)
            assert 0 <= seg < n_seg
            xcds[seg][(y * n_seg + x) % 8] += 1
            if y >= lib.blocks(HU, waves[seg], W):
                continue
            for wv in range(W):
                u = lib.unit(y, wv, waves[seg], W, HU)
                hu = u if u >= 0 else -1 - u
                assert 0 <= hu < HU, (seg, y, wv)
                if u >= 0:
                    seen[seg].append(hu)
                    if wv % waves[seg] == 0:
                        counts[seg] += max(0, lib.counted(wv // waves[seg], W // waves[seg], hu, HU))
    for s, w in enumerate(waves):
        assert seen[s] == [u for u in range(HU) for _ in range(w)]
        assert counts[s] == HU
        assert max(xcds[s]) <= 2 * -(-HU // 8)


def test_which_launches_are_grouped(lib):
    """Only where many units are counted in one cache line of lens, the more the longer the prompt, and never beyond four units per
    compute unit."""
    assert lib.grouped(40, 24, 40, 40, 100, 256) and lib.grouped(32, 32, 1, 1, 200, 256) and lib.grouped(32, 32, 32, 32, 800, 128) and not lib.grouped(32, 32, 32, 32, 801, 128)
    assert not lib.grouped(1024, 1, 32, 32, 60, 256)              # segments of one unit
    assert not lib.grouped(32, 32, 4, 32, 60, 256)                # eight sequences, 4 of 32 layers
    assert not lib.grouped(16, 40, 1, 40, 60, 256)                # a layer a call
    for N in (60, 104, 105, 200):                                    # 256 of 1024 units in a line, 288 of 288
        assert lib.grouped(128, 8, 32, 32, N, 256) == lib.grouped(24, 12, 24, 24, N, 256) == (N <= 104)
    assert lib.grouped(64, 16, 32, 32, 200, 256) and not lib.grouped(64, 16, 32, 32, 201, 256)   # half of the units in a line
    for n_seg in range(1, 34):                                       # a sequence of 32 heads
        for N in (60, 104, 105, 200, 201, 304, 305, 400, 401):
            least = 6 if N <= 104 else 8 if N <= 200 else 17 if N <= 304 else 23 if N <= 400 else 99
            assert lib.grouped(n_seg, 32, n_seg, n_seg, N, 256) == (least <= n_seg <= 32), (n_seg, N)
