"""Decode steps of launches around what a compute unit holds of the ranked bf16 kernel (20 wavefronts, 5120 units on 256 compute
units): one full round, just over it, several rounds, and long prompts with four workgroups per compute unit; against the CPU
oracle with the bars of the other GPU tests."""
import pytest
import torch

import paper_2412_03409_amd as P
from test_gpu_parity import DEV, run_decode_case, run_evict_case

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


@pytest.mark.parametrize("B,L,H,N,D,frac", [
    (4, 32, 32, 390, 128, 0.06),     # 4096 units
    (5, 32, 32, 390, 128, 0.06),     # 5120: one round of single wavefronts
    (5, 33, 31, 770, 64, 0.04),      # 5115, an odd number of heads
    (7, 31, 24, 390, 128, 0.06),     # 5208: more than one round
    (6, 33, 32, 390, 128, 0.06),     # 6336
    (5, 31, 31, 775, 128, 0.03),     # 4805 of long prompts, four, two and one wavefront each: 31 KB of LDS
    (3, 21, 24, 770, 128, 0.03),     # 1512 of long prompts: four wavefronts or two
    (3, 21, 25, 300, 64, 0.2),       # 1575 of short ones, an odd number of heads: workgroups with units of two segments
    (8, 33, 33, 200, 64, 0.1),       # 8712 of short prompts, index order
])
def test_rounds(B, L, H, N, D, frac):
    run_decode_case(B, L, H, H, N, D, BF16, frac, 2, seed=B * L + H)


@pytest.mark.parametrize("B,L,H,N,D,frac,d,steps", [
    (5, 32, 32, 390, 128, 0.05, 2, 4),
    (6, 33, 33, 770, 64, 0.03, 3, 5),
])
def test_rounds_with_pruning(B, L, H, N, D, frac, d, steps):
    run_evict_case(B, L, H, H, N, D, BF16, frac, d, steps, seed=B * L + H)


# Two ranges of layers stepped on two streams at once: their words of lens share cache lines, are read through the caches and
# counted on by both launches; bit for bit what one stream gives.
@pytest.mark.parametrize("L,N", [(60, 64), (14, 200)])       # ranked launches; one unit per workgroup
def test_two_streams_of_one_cache(L, N):
    B, H, D, T = 2, 32, 128, 8
    g = torch.Generator().manual_seed(L)
    rnd = lambda *s: torch.randn(s, generator=g).to(BF16).to(DEV)
    k, v = rnd(B, L, H, N, D), rnd(B, L, H, N, D)
    q, kn, vn = rnd(T, B, L, H, D), rnd(T, B, L, H, D), rnd(T, B, L, H, D)
    order = torch.argsort(torch.rand((B, L, N), generator=g), dim=-1).int().to(DEV)
    lengths = torch.randint(1, N // 2, (B, L), generator=g, dtype=torch.int32).to(DEV)
    scale = torch.full((L,), 0.1, device=DEV)
    outs, caches = [], []
    for streams in (1, 2):
        cache = P.prefixkv_compact(k, v, order, lengths, T, int(lengths.sum()) + B * L * T)
        out = torch.zeros_like(q)
        torch.cuda.synchronize()
        st = [torch.cuda.Stream() for _ in range(streams)]
        for t in range(T):
            for i, (l0, l1) in enumerate(((0, L // 2), (L // 2, L))):
                with torch.cuda.stream(st[i % streams]):
                    P.prefixkv_decode_attn(cache, q[t], kn[t], vn[t], scale, N, l0, l1, out=out[t])
        torch.cuda.synchronize()
        outs.append(out)
        caches.append(cache)
    assert torch.equal(caches[1].lens.cpu(), lengths.cpu() + T)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(caches[0].lens, caches[1].lens) and torch.equal(caches[0].kc, caches[1].kc) and torch.equal(caches[0].vc, caches[1].vc)
