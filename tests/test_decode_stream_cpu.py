"""The block stream of the grouped-query decode: gqa_share of csrc/decode_rows.hpp, compiled for the host, and the index rules
of decode_gqa_kernel and decode_gqa_merge_kernel around it.  Every block of every unit is worked on exactly once; every
shared unit's pieces lie in slots of their own, which the merge finds, inside the workspace that the size query returns."""
import ctypes as C
import os
import random
import subprocess

import pytest

import paper_2412_03409_amd as P

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_03409_amd", "csrc")
SHIM = """
#define __device__
#define __host__
#define __forceinline__ inline
#include "decode_rows.hpp"
extern "C" int share(int all, int waves) { return pkv::gqa_share(all, waves); }
extern "C" int least(int all, int waves, int units, int width) { return pkv::gqa_least(all, waves, units, width); }
extern "C" int share_of(int all, int waves, int least) { return pkv::gqa_share(all, waves, least); }
extern "C" int rows(int ev, int len, int cap, int base, int append, int t, int d, int block, int* blocks) {
    const pkv::StepRows r = ev ? pkv::step_rows<true>(len, cap, base, append, t, d) : pkv::step_rows<false>(len, cap, base, append, t, d);
    *blocks = pkv::row_blocks(r.rows, block);
    return r.rows * 2 + r.app;
}
// the blocks [w * share, ...) of a launch as the attention kernel walks them from segment `seg` on: seg, hu, blk, slot of each, -1
// for the slot of one that ends no piece in the workspace
extern "C" int kernel_walk(int w, int share, int all, int seg, const int* nb, const int* first, int HU, int* out) {
    const int x0 = w * share, x1 = x0 + share < all ? x0 + share : all;
    if (x0 >= all) return 0;
    const pkv::GqaPlace at = pkv::gqa_place(x0, first[seg], nb[seg], HU);
    int hu = at.hu, blk = at.blk, begun = x0 - blk;
    for (int x = x0;; ++x, out += 4) {
        const bool ends = blk + 1 == nb[seg], more = x + 1 < x1, shared = !(ends && begun >= x0);
        out[0] = seg; out[1] = hu; out[2] = blk; out[3] = (ends || !more) && shared ? pkv::gqa_slot(w, seg, hu, HU) : -1;
        if (!more) return x1 - x0;
        if (pkv::gqa_next(blk, hu, seg, nb[seg], HU) != pkv::GqaNext::block) begun = x + 1;
    }
}
extern "C" void merge_slots(int first, int nb, int seg, int hu, int HU, int share, int* out) {
    const pkv::GqaPieces p = pkv::gqa_pieces(first, nb, hu, HU, share);
    out[0] = p.n; out[1] = pkv::gqa_slot(p.wave, seg, hu, HU);
}
extern "C" unsigned long long base(unsigned long long at) { return pkv::gqa_ws_base(at); }
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("stream")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")])
    return C.CDLL(str(d / "shim.so"))


@pytest.fixture(scope="module")
def share(shim):
    return shim.share


def walk(share, lens, HU, BR, waves):
    """Highest slot used; asserts the rest."""
    nb = [max(1, -(-n // BR)) for n in lens]
    first = [0]
    for x in nb:
        first.append(first[-1] + x)
    everything = first[-1] * HU
    S = share(everything, waves)
    owner, slots = {}, {}
    for w in range(waves):
        x0, x1 = w * S, min(w * S + S, everything)
        if x0 >= everything:
            continue
        y0 = x0 // HU
        seg = max(i for i in range(len(nb)) if first[i] <= y0)
        hu, blk = divmod(x0 - first[seg] * HU, nb[seg])
        assert hu < HU
        begun = x0 - blk
        for x in range(x0, x1):
            assert (seg, hu, blk) not in owner
            owner[seg, hu, blk] = w
            ends, more = blk + 1 == nb[seg], x + 1 < x1
            if (ends or not more) and not (ends and begun >= x0):
                slot = w + seg * HU + hu
                assert slot not in slots
                slots[slot] = seg, hu
            if ends:
                seg, hu, blk, begun = (seg, hu + 1, 0, x + 1) if hu + 1 < HU else (seg + 1, 0, 0, x + 1)
            else:
                blk += 1
    assert len(owner) == everything
    top = max(slots, default=-1)
    for seg in range(len(nb)):
        for hu in range(HU):
            b0 = first[seg] * HU + hu * nb[seg]
            w0, pieces = b0 // S, (b0 + nb[seg] - 1) // S - b0 // S + 1
            assert {owner[seg, hu, b] for b in range(nb[seg])} == set(range(w0, w0 + pieces))
            for k in range(pieces if pieces > 1 else 0):
                assert slots.pop(w0 + k + seg * HU + hu) == (seg, hu)
    assert not slots
    return top


def test_every_block_once(share):
    rng = random.Random(0)
    for _ in range(1500):
        n, HU, waves = rng.randint(1, 40), rng.choice([1, 2, 3, 8]), rng.choice([1, 2, 7, 64, 300])
        lens = [rng.choice([0, 1, rng.randint(0, 40), rng.randint(0, 900)]) for _ in range(n)]
        assert walk(share, lens, HU, rng.choice([16, 32]), waves) < waves + n * HU


@pytest.mark.parametrize("G,HU", [(2, 1), (4, 8), (8, 3)])
@pytest.mark.parametrize("D", [64, 128])
def test_slots_fit_the_workspace(G, HU, D):
    for n_seg, N in [(1, 1), (1, 8192), (5, 300), (64, 511), (64, 512), (640, 100)]:
        B, L = (n_seg // 64, 64) if n_seg % 64 == 0 else (1, n_seg)
        words = P.prefixkv_workspace_bytes(3, B, L, G * HU, HU, N, D, P.PKV_BF16) // 4
        units = n_seg * HU
        slots = (words - (16 + n_seg + 1 + 15) // 16 * 16) // (G * (D + 2))
        assert slots - units >= 1                     # at least one wavefront


# Also with a single block for each wavefront, which short launches take: never more of them than half the wavefronts.
def test_every_block_once_in_short_launches(shim):
    rng = random.Random(2)
    for _ in range(300):
        n, HU = rng.randint(1, 40), rng.choice([1, 2, 3, 8])
        lens = [rng.choice([0, 1, rng.randint(0, 40), rng.randint(0, 900)]) for _ in range(n)]
        assert walk(lambda all, waves: shim.share_of(all, waves, 1), lens, HU, rng.choice([16, 32]), 2048) < 2048 + n * HU
    for width in (128, 256, 512, 1024):
        for units in (1, 8, 100, 1000):
            one = [all for all in range(1, 3000) if shim.least(all, 2048, units, width) == 1]
            assert one == list(range(1, min(1024, 32768 * units // width) + 1))
            assert all(shim.share_of(x, 2048, 1) == 1 for x in one)


# The same with the rules that the kernels compile: the walk of a wavefront, the slots it leaves pieces in and those the merge reads.
def test_rules_of_the_kernels(shim):
    rng, out = random.Random(3), (C.c_int * 40000)()
    for _ in range(300):
        n, HU, BR, waves = rng.randint(1, 40), rng.choice([1, 2, 3, 8]), rng.choice([16, 32]), rng.choice([1, 2, 7, 64, 2048])
        lens = [rng.choice([0, 1, rng.randint(0, 40), rng.randint(0, 900)]) for _ in range(n)]
        nb = [max(1, -(-x // BR)) for x in lens]
        first = [sum(nb[:i]) for i in range(n)]
        everything = sum(nb) * HU
        share = shim.share_of(everything, waves, rng.choice([1, 2]))
        c_nb, c_first = (C.c_int * n)(*nb), (C.c_int * n)(*first)
        blocks, slots = [], {}
        for w in range(-(-everything // share)):
            seg = max(i for i in range(n) if first[i] <= w * share // HU)
            for i in range(shim.kernel_walk(w, share, everything, seg, c_nb, c_first, HU, out)):
                blocks.append(tuple(out[4 * i:4 * i + 3]))
                if out[4 * i + 3] >= 0:
                    assert out[4 * i + 3] not in slots
                    slots[out[4 * i + 3]] = blocks[-1][:2]
        assert blocks == [(s, hu, b) for s in range(n) for hu in range(HU) for b in range(nb[s])]
        assert max(slots, default=-1) < waves + n * HU
        for s in range(n):
            for hu in range(HU):
                shim.merge_slots(first[s], nb[s], s, hu, HU, share, out)
                for k in range(out[0] if out[0] > 1 else 0):
                    assert slots.pop(out[1] + k) == (s, hu)
        assert not slots


# Whatever the prompt's length and the number of segments there is a slot for each unit and for each of the 2048 wavefronts of a
# launch on 256 compute units.
@pytest.mark.parametrize("G,HU,D", [(2, 1, 64), (4, 8, 128), (8, 3, 128), (8, 4, 64)])
@pytest.mark.parametrize("B,L,N", [(1, 1, 1), (1, 1, 500), (1, 1, 8192), (1, 32, 500), (10, 64, 100)])
def test_workspace_never_bounds_a_launch(B, L, N, G, HU, D):
    words = P.prefixkv_workspace_bytes(3, B, L, G * HU, HU, N, D, P.PKV_BF16) // 4
    slots = (words - (16 + B * L + 1 + 15) // 16 * 16) // (G * (D + 2))
    assert slots >= 2048 + B * L * HU


# Partial results go by 16 bytes; the caller's workspace may start anywhere.
def test_workspace_of_any_alignment(shim):
    shim.base.restype, shim.base.argtypes = C.c_ulonglong, [C.c_ulonglong]
    G, HU, D = 4, 8, 128
    slots = 2048 + 5 * HU
    size = P.prefixkv_workspace_bytes(3, 1, 5, G * HU, HU, 300, D, P.PKV_BF16)
    for at in range(1 << 40, (1 << 40) + 33):
        base = shim.base(at)
        assert base % 16 == 0 and base >= at
        assert base + 4 * ((16 + 5 + 1 + 15) // 16 * 16 + slots * G * (D + 2)) <= at + size


# The rows of a step, which a wavefront's share and its walk both go by.
def test_rows_of_a_step(shim):
    rng, nb = random.Random(1), C.c_int()
    for _ in range(3000):
        cap, t, d = rng.randint(1, 80), rng.choice([1, 2, 15, 16, 17, 1 << 30]), rng.choice([1, 15, 65535])
        n, base, append = rng.randint(0, cap), rng.randint(-1, cap), rng.random() < 0.5
        stores = append and n < cap
        assert shim.rows(0, n, cap, base, append, t, d, 16, C.byref(nb)) == 2 * (n + stores) + stores
        assert nb.value == max(1, -(-(n + stores) // 16))
        fits = base >= 0 and base <= cap - d - 1 and n <= cap - d - 1
        want = n + min(t, d + 1) if fits else 0
        assert shim.rows(1, n, cap, base, append, t, d, 32, C.byref(nb)) == 2 * want + fits
        assert nb.value == max(1, -(-want // 32))
