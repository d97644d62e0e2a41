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
extern "C" int waves(int blocks, int spread, int W) { return pkv::active_waves(blocks, spread, W); }
extern "C" int blocks(int HU, int waves, int W) { return pkv::grouped_blocks(HU, waves, W); }
extern "C" int unit(int block, int wv, int waves, int W, int HU) { const pkv::GroupedUnit x = pkv::grouped_unit(block, wv, waves, W, HU); return x.live ? x.hu : -1 - x.hu; }
extern "C" int counted(int at, int units, int hu, int HU) { return pkv::counted_units(at, units, hu, HU); }
extern "C" int spread(long long units, int cus, int N) { return pkv::spread_blocks(units, cus, N); }
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
    for units in (65, 256, 512, 513, 1024):
        for W, N in ((w, n) for w in (4, 8) for n in (1, 39, 40, 79, 80, 200, 319, 320, 400)):
            s = lib.spread(units, 256, N)
            assert 1 <= s <= 8
            last = 1
            for blocks in range(0, 600):
                n = lib.waves(blocks, s, W)
                assert n in (1, 2, 4, 8) and last <= n <= W
                assert n == W or blocks <= n * s
                assert n == 1 or blocks > n // 2 * s
                last = n


@pytest.mark.parametrize("HU", [1, 2, 3, 9, 10, 12, 14, 32, 40])
@pytest.mark.parametrize("W", [4, 8])
def test_units_of_a_grouped_launch(lib, HU, W):
    """Every unit once with all its wavefronts, counts that add up to HU, and no index beyond HU, in wavefronts to spare too."""
    for waves in [w for w in (1, 2, 4, 8) if w <= W]:
        n = lib.blocks(HU, waves, W)
        assert 1 <= n <= HU                               # a workgroup per unit is enough
        seen, counts = [], 0
        for block in range(n):
            for wv in range(W):
                x = lib.unit(block, wv, waves, W, HU)
                hu = x if x >= 0 else -1 - x
                assert 0 <= hu < HU, (block, wv, waves)
                if x >= 0:
                    seen.append(hu)
                    if wv % waves == 0:
                        counts += max(0, lib.counted(wv // waves, W // waves, hu, HU))
        assert seen == [u for u in range(HU) for _ in range(waves)]
        assert counts == HU
