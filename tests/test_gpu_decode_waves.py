"""Decode launches whose units have one, two, four or all of a workgroup's wavefronts, the new row in any of their blocks, against the CPU oracle with the bars of the other GPU tests."""
import pytest
import torch

from test_gpu_parity import run_decode_case, run_evict_case

pytestmark = pytest.mark.gpu
BF16, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("B,L,H,Hkv,N,D,dt,frac", [
    (1, 32, 32, 32, 400, 128, BF16, 0.3),    # 1024 units, grouped: four to a workgroup up to 8 blocks, two up to 16
    (1, 32, 32, 32, 401, 128, BF16, 0.3),    # one to a workgroup
    (2, 17, 20, 20, 130, 128, BF16, 0.5),    # 680 of short prompts
    (6, 1, 32, 32, 100, 128, BF16, 0.6),     # 192
    (70, 1, 2, 2, 64, 64, BF16, 0.7),        # 140 of 70 segments
    (3, 30, 9, 3, 190, 128, F32, 0.4),       # 810, three to a KV head, one of which stores the new row; an odd number of heads
    (3, 24, 12, 12, 1003, 64, BF16, 0.2),    # 864, one to a workgroup, 32-row blocks
    (1, 40, 12, 12, 610, 128, BF16, 0.3),    # 480
    (2, 14, 12, 12, 1200, 128, BF16, 0.1),   # 336: eight wavefronts, a block each
    (2, 16, 16, 8, 300, 64, F32, 0.3),       # 256 units of two query heads
])
def test_spread(B, L, H, Hkv, N, D, dt, frac):
    run_decode_case(B, L, H, Hkv, N, D, dt, frac, 3, seed=N)


@pytest.mark.parametrize("B,L,H,Hkv,N,D,dt,frac,d,steps", [
    (1, 32, 32, 32, 340, 128, BF16, 0.2, 40, 44),
    (1, 24, 20, 20, 200, 64, BF16, 0.1, 1, 5),
    (2, 15, 9, 3, 190, 128, F32, 0.3, 5, 9),
])
def test_spread_with_pruning(B, L, H, Hkv, N, D, dt, frac, d, steps):
    run_evict_case(B, L, H, Hkv, N, D, dt, frac, d, steps, seed=N)
