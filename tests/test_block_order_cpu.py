"""csrc/block_order.hpp, compiled for the host: every block of every head once, each head's blocks next to each other up
to the tail, whose blocks go longest first; with an even number of blocks the long ones are dealt out evenly."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_03409_amd", "csrc")
SHIM = """
#define __device__
#define __host__
#define __forceinline__ inline
#include "block_order.hpp"
extern "C" void block(int j, int heads, int nblk, int tail, int* out) {
    const pkv::HeadBlock x = pkv::head_block(j, heads, nblk, tail);
    out[0] = x.head;
    out[1] = x.rank;
}
extern "C" int fit(long long heads, int xcds) { return pkv::heads_fit(heads, xcds); }
"""


@pytest.fixture(scope="module")
def block(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o",
                           str(d / "shim.so")])
    lib = C.CDLL(str(d / "shim.so"))
    f = lib.block
    out = (C.c_int * 2)()

    def call(*a):
        f(*a, out)
        return out[0], out[1]
    call.fit = lambda heads: lib.fit(C.c_longlong(heads), 8)
    return call


@pytest.mark.parametrize("heads", [1, 2, 5, 40, 200])
@pytest.mark.parametrize("nblk", [1, 2, 3, 6, 8, 9, 12, 16, 64])
@pytest.mark.parametrize("tail", [1, 3, 32, 1000])
def test_every_block_once(block, heads, nblk, tail):
    tail = min(tail, heads)
    lead = heads - tail
    got = [block(j, heads, nblk, tail) for j in range(heads * nblk)]
    assert sorted(got) == [(h, r) for h in range(heads) for r in range(nblk)]
    assert [h for h, _ in got[:lead * nblk]] == [j // nblk for j in range(lead * nblk)]
    assert [r for _, r in got[lead * nblk:]] == [i // tail for i in range(tail * nblk)]


@pytest.mark.parametrize("nblk", [2, 3, 5, 6, 8, 9, 12, 16])
def test_blocks_are_dealt_out_evenly(block, nblk):
    """Workgroups dealt to 32 compute units in turn: none gets much more than its share of the work."""
    heads = 32 * nblk
    work = [0] * 32
    for j in range(heads * nblk):
        work[j % 32] += nblk - block(j, heads, nblk, 0)[1]
    assert max(work) <= 1.1 * sum(work) / 32, work


def test_heads_of_a_launch(block):
    """What eight equal shares of heads leave below 2^31, to the last one."""
    for heads in (1, 7, 8, 9, (1 << 31) - 16, (1 << 31) - 9, (1 << 31) - 8):
        assert block.fit(heads), heads
    for heads in ((1 << 31) - 7, (1 << 31) - 1, 1 << 31, 1 << 32, 1 << 40):
        assert not block.fit(heads), heads
