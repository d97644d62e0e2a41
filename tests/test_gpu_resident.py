"""Decode steps of launches around what a compute unit holds of the ranked bf16 kernel (20 wavefronts, 5120 units on 256 compute
units): one full round, just over it, several rounds, and long prompts with four workgroups per compute unit; against the CPU
oracle with the bars of the other GPU tests."""
import pytest
import torch

from test_gpu_parity import run_decode_case, run_evict_case

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
