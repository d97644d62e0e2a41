"""Parity at the sizes where a launch rule changes its form (edges of its ranges, remainders, the smallest and
largest counts), against the CPU oracle and with the bars of the other GPU tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_03409_amd as P
from test_gpu_parity import DEV, check_importance, np32, rand_qk, run_decode_case, run_evict_case

pytestmark = pytest.mark.gpu


# decode_attn_kernel: 8 wavefronts per unit up to 512 units, 4 up to 1024, ranked launches beyond (one to four units
# per workgroup), one capacity register per lane up to 64 segments of a launch, groups of segments beyond 512
@pytest.mark.parametrize("B,L,H,Hkv,N,D,dtype,frac,steps,layers", [
    (1, 16, 32, 32, 150, 64, torch.bfloat16, 0.4, 2, None),     # 512 units
    (1, 19, 27, 27, 60, 64, torch.bfloat16, 0.4, 2, None),      # 513
    (1, 25, 41, 41, 300, 64, torch.bfloat16, 0.3, 2, None),     # 1025: ranked, 41 heads leave a remainder of 1
    (2, 32, 18, 18, 90, 128, torch.bfloat16, 0.5, 2, None),     # ranked, 64 segments
    (1, 64, 20, 20, 40, 64, torch.bfloat16, 0.5, 1, (1, 64)),   # ranked over a layer range of 63 segments
    (5, 13, 18, 18, 70, 64, torch.float32, 0.3, 2, None),       # 65 segments, fp32
    (3, 30, 14, 14, 50, 64, torch.bfloat16, 0.4, 2, (3, 29)),   # layer range, more than 64 segments
    (9, 60, 2, 2, 33, 64, torch.bfloat16, 0.6, 2, None),        # 540 segments: two groups
    (17, 61, 3, 1, 20, 64, torch.float32, 0.5, 1, None),        # 1037 segments: three groups, one KV head
    (8, 33, 32, 32, 24, 64, torch.bfloat16, 0.3, 1, None),      # 8448 units: one wavefront each
])
def test_decode_launch_shapes(B, L, H, Hkv, N, D, dtype, frac, steps, layers):
    run_decode_case(B, L, H, Hkv, N, D, dtype, frac, steps, seed=B * L + H, layer_range=layers)


@pytest.mark.parametrize("B,L,H,Hkv,N,D,dtype,frac,d,steps", [
    (1, 19, 27, 27, 60, 64, torch.bfloat16, 0.4, 2, 5),
    (2, 33, 18, 18, 40, 64, torch.bfloat16, 0.5, 3, 6),         # ranked
    (5, 13, 18, 18, 30, 128, torch.float32, 0.3, 20, 24),       # ranked, ring longer than the kept part
])
def test_decode_evict_launch_shapes(B, L, H, Hkv, N, D, dtype, frac, d, steps):
    run_evict_case(B, L, H, Hkv, N, D, dtype, frac, d, steps, seed=B * L + H)


def run_importance_case(B, L, H, Hkv, N, D, dtype, negative=False):
    """Importance with and without the caller's log-sum-exp; rows at twice their length apart."""
    q, k, scale = rand_qk(N + D + H, B, L, H, Hkv, N, D, dtype)
    scale = -scale if negative else scale
    want, lse = oracle.importance(np32(q), np32(k), scale.numpy(), want_lse=True)
    qd = torch.cat([q, q], dim=-1).to(DEV)[..., :D]
    kd = torch.cat([k, k], dim=-1).to(DEV)[..., D:]
    check_importance(np32(P.prefixkv_importance(qd, kd, scale.to(DEV))), want)
    lse_d = torch.from_numpy(lse.astype(np.float32)).to(DEV)
    check_importance(np32(P.prefixkv_importance(qd, kd, scale.to(DEV), lse=lse_d)), want)


# importance_f32_kernel: 16-row tiles dealt to four wavefronts
@pytest.mark.parametrize("N", [1, 15, 16, 17, 64, 65, 129, 300])
@pytest.mark.parametrize("H,Hkv,D,negative", [(2, 2, 64, False), (4, 1, 128, True)])
def test_importance_f32_tiles(N, H, Hkv, D, negative):
    run_importance_case(2, 2, H, Hkv, N, D, torch.float32, negative)
