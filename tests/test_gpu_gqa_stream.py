"""Grouped-query decode steps at the edges of their block stream: lengths around a block, units shared by many wavefronts,
more wavefronts than blocks, more segments than a wavefront holds the block counts of, empty segments, keys at -inf; against
the CPU oracle or fp64, with the bars of the other GPU tests."""
import pytest
import torch

import paper_2412_03409_amd as P
from test_gpu_parity import DEV, OUT_ATOL, run_decode_case, run_evict_case

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


@pytest.mark.parametrize("B,L,H,Hkv,N,D,frac,steps,layers", [
    (1, 1, 2, 1, 14, 128, 1.0, 4, None),        # blocks of 16 rows: 14 ... 18
    (1, 1, 8, 1, 30, 64, 1.0, 4, None),         # blocks of 32 rows: 30 ... 34
    (2, 3, 16, 2, 65, 128, 0.6, 2, (1, 3)),     # groups of 8, a layer range
    (1, 2, 32, 8, 8192, 128, 0.5, 1, None),     # 2048 wavefronts share 16 units
    (3, 9, 12, 3, 700, 64, 0.5, 2, None),       # a wavefront ends in the middle of units
    (11, 24, 4, 2, 40, 128, 0.5, 2, None),      # 264 segments
    (9, 61, 8, 1, 24, 64, 0.5, 1, (0, 60)),     # 540 segments of a block or two
    # several head groups per KV head (6: three of 2, 12: three of 4, 16: two of 8): the first one stores the appended row
    (2, 3, 12, 2, 300, 128, 0.5, 2, None),
    (1, 2, 12, 2, 700, 64, 0.6, 2, None),
    (1, 2, 12, 1, 500, 128, 0.9, 2, None),
    (3, 4, 24, 2, 90, 64, 0.5, 3, (1, 4)),
    (1, 2, 16, 1, 700, 128, 0.7, 2, None),
    (2, 3, 32, 2, 200, 64, 0.6, 2, None),
    (1, 1, 16, 1, 8192, 128, 0.9, 1, None),     # a unit in over 200 wavefronts
    (1, 9, 12, 2, 4100, 64, 0.9, 1, None),      # three or four blocks a wavefront
])
def test_stream(B, L, H, Hkv, N, D, frac, steps, layers):
    run_decode_case(B, L, H, Hkv, N, D, BF16, frac, steps, seed=B * L + H, layer_range=layers)


@pytest.mark.parametrize("D", [64, 128])
def test_empty_segments(D):
    run_decode_case(3, 4, 8, 2, 100, D, BF16, 0.5, 2, seed=D, zero_seq=True)


@pytest.mark.parametrize("B,L,H,Hkv,N,D,frac,d,steps", [
    (1, 2, 2, 1, 16, 128, 0.5, 1, 6),
    (2, 3, 8, 2, 90, 64, 0.4, 15, 34),          # ring and survivors cross block borders
    (1, 5, 32, 4, 400, 128, 0.5, 7, 20),
    (11, 24, 4, 2, 33, 64, 0.5, 3, 7),          # 264 segments
    (2, 3, 12, 2, 90, 128, 0.4, 7, 18),         # several head groups per KV head: the first one moves the survivor
    (1, 3, 12, 1, 200, 64, 0.5, 5, 14),
    (2, 2, 16, 1, 120, 64, 0.5, 15, 34),
    (1, 2, 32, 2, 400, 128, 0.5, 3, 9),
])
def test_stream_with_pruning(B, L, H, Hkv, N, D, frac, d, steps):
    run_evict_case(B, L, H, Hkv, N, D, BF16, frac, d, steps, seed=B * L + H)


@pytest.mark.parametrize("H,D", [(4, 128), (8, 64)])
def test_keys_at_minus_infinity(H, D):
    B, L, Hkv, N, inf_rows = 1, 2, 2, 90, [*range(0, 33), *range(48, 64)]
    g = torch.Generator().manual_seed(H * D)
    k = torch.randn((B, L, Hkv, N, D), generator=g).abs()
    k[:, :, :, inf_rows] = -float("inf")
    v = torch.randn((B, L, Hkv, N, D), generator=g).to(BF16)
    q = (torch.randn((B, L, H, D), generator=g).abs() + 0.1).to(BF16)
    k, scale = k.to(BF16), torch.full((L,), D ** -0.5)
    order = torch.arange(N, dtype=torch.int32).expand(B, L, N).contiguous().to(DEV)
    lengths = torch.full((B, L), N, dtype=torch.int32, device=DEV)
    cache = P.prefixkv_compact(k.to(DEV), v.to(DEV), order, lengths, 1, B * L * (N + 1))
    out = P.prefixkv_decode_attn(cache, q.to(DEV), None, None, scale.to(DEV), N)
    rep = lambda x: x.repeat_interleave(H // Hkv, 2).double()
    s = (rep(k) * q.double().unsqueeze(3)).sum(-1) * D ** -0.5
    want = (torch.softmax(s, -1).unsqueeze(-1) * rep(v)).sum(3)
    assert (out.cpu().double() - want).abs().max() <= OUT_ATOL


# Whatever the workspace holds beforehand, and whatever its alignment, must not matter; nothing is written past its end.
@pytest.mark.parametrize("shift", [0, 1, 4, 12])
def test_dirty_workspace(shift):
    B, L, H, Hkv, N, D = 1, 3, 4, 1, 600, 128
    g = torch.Generator().manual_seed(1)
    rnd = lambda *s: torch.randn(s, generator=g).to(BF16).to(DEV)
    k, v, q = rnd(B, L, Hkv, N, D), rnd(B, L, Hkv, N, D), rnd(B, L, H, D)
    order = torch.arange(N, dtype=torch.int32, device=DEV).expand(B, L, N).contiguous()
    lengths = torch.tensor([[600, 3, 170]], dtype=torch.int32, device=DEV)
    scale = torch.full((L,), 0.1, device=DEV)
    n = P.prefixkv_workspace_bytes(3, B, L, H, Hkv, N, D, P.PKV_BF16)
    outs = []
    for fill in (0, 255, 127):
        cache = P.prefixkv_compact(k, v, order, lengths, 0, B * L * N)
        buf = torch.full((shift + n + 64,), fill, dtype=torch.uint8, device=DEV)
        outs.append(P.prefixkv_decode_attn(cache, q, None, None, scale, N, ws=buf[shift:shift + n]))
        assert (buf[:shift] == fill).all() and (buf[shift + n:] == fill).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
