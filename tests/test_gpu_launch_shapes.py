"""Parity at the sizes where a launch rule changes its form (edges of its ranges, remainders, the smallest and
largest counts), against the CPU oracle and with the bars of the other GPU tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_03409_amd as P
from test_gpu_parity import DEV, OUT_ATOL, check_importance, check_select, np32, rand_qk, run_decode_case, run_evict_case
from pkv_workloads import synthetic_importance
from tolerances import LSE_ATOL, LSE_RTOL

pytestmark = pytest.mark.gpu


# decode_attn_kernel on 256 compute units: 8 wavefronts per unit up to 512 units, 4 up to 1024, ranked launches beyond (one,
# two or four units per workgroup), one capacity register per lane up to 64 segments of a launch, groups of segments
# beyond 512
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


# head_mean_parts_kernel: four quarters of the heads, eight at a time, remainders and empty quarters
@pytest.mark.parametrize("H", [1, 3, 5, 31, 33, 41, 67])
def test_importance_head_remainders(H):
    run_importance_case(2, 1, H, H, 70, 64, torch.bfloat16)


# importance_f32_kernel: 16-row tiles dealt to four wavefronts
@pytest.mark.parametrize("N", [1, 15, 16, 17, 64, 65, 129, 300])
@pytest.mark.parametrize("H,Hkv,D,negative", [(2, 2, 64, False), (4, 1, 128, True)])
def test_importance_f32_tiles(N, H, Hkv, D, negative):
    run_importance_case(2, 2, H, Hkv, N, D, torch.float32, negative)


# prefill_attn_kernel: 128-query blocks, 64-key stages, plain stages below the diagonal; the last heads of an XCD run
# longest block first
@pytest.mark.parametrize("B,L,H,Hkv,N,D,negative", [
    (1, 1, 1, 1, 1, 128, False), (1, 1, 3, 1, 63, 64, False), (1, 1, 2, 2, 64, 128, True), (1, 2, 4, 2, 65, 128, False),
    (1, 1, 2, 1, 127, 64, True), (1, 1, 9, 3, 129, 128, False), (2, 1, 5, 5, 192, 64, False),
    (1, 1, 2, 2, 193, 128, False), (1, 1, 3, 3, 321, 128, True), (1, 3, 4, 4, 257, 64, False),
    (2, 5, 30, 30, 257, 64, False),      # 300 heads of 3 blocks: heads in order, then the longest-first tail
])
def test_prefill_stages(B, L, H, Hkv, N, D, negative):
    q, k, scale = rand_qk(N + D + H, B, L, H, Hkv, N, D, torch.bfloat16)
    scale = -scale if negative else scale
    v = torch.randn(k.shape, generator=torch.Generator().manual_seed(N)).to(torch.bfloat16)
    out, lse = P.prefixkv_prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), scale.to(DEV))
    want, want_lse = oracle.prefill_attn(np32(q), np32(k), np32(v), scale.numpy(), out_bf16=True)
    assert np.abs(np32(out) - want).max() <= OUT_ATOL
    np.testing.assert_allclose(lse.cpu().numpy(), want_lse, rtol=LSE_RTOL, atol=LSE_ATOL)


def test_prefill_moving_reference_and_infinite_keys():
    """Scores that grow along the keys, a scale of zero, and keys
    that score -inf for a whole stage (the rows of the oracle are fp64)."""
    N, D = 300, 64
    g = torch.Generator().manual_seed(5)
    q = torch.randn((1, 3, 1, N, D), generator=g).abs()
    k = torch.randn((1, 3, 1, N, D), generator=g).abs() * torch.linspace(0, 1, N).view(1, 1, 1, N, 1) ** 2
    k[:, 2, :, 64:128] = -float("inf")
    v = torch.randn((1, 3, 1, N, D), generator=g)
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    scale = torch.tensor([1.0, 0.0, 0.3])
    out, lse = P.prefixkv_prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), scale.to(DEV))
    s = torch.einsum("blhmd,blhnd->blhmn", q.double(), k.double()) * scale.double().view(1, 3, 1, 1, 1)
    s = s.masked_fill(torch.ones(N, N).triu(1).bool(), -float("inf"))
    want = torch.softmax(s, -1) @ v.double()
    assert (out.cpu().double() - want).abs().max() <= OUT_ATOL
    np.testing.assert_allclose(lse.cpu().numpy(), torch.logsumexp(s, -1).numpy(), rtol=LSE_RTOL, atol=LSE_ATOL)


# importance: fused kernel (up to 768 positions, heads near a multiple of the CUs) or stream kernels, the latter with 32
# or 64 stationary rows per wavefront and with one or two groups of wavefronts; and the fused kernel again when the
# workspace holds the column sums alone
@pytest.mark.parametrize("B,L,H,Hkv,N,D,negative", [
    (1, 1, 1, 1, 1, 64, False), (1, 1, 2, 1, 127, 128, False), (1, 1, 3, 3, 128, 64, True), (1, 2, 4, 2, 129, 128, False),
    (1, 1, 2, 2, 257, 128, True), (1, 2, 3, 1, 449, 64, False), (1, 1, 2, 2, 768, 128, False), (1, 1, 2, 1, 769, 64, False),
    (1, 8, 40, 8, 65, 64, False),        # 320 heads: streams, more than one workgroup per CU
    (4, 8, 32, 32, 130, 64, False),      # 1024 heads of 2 blocks: 64 rows per wavefront with a given log-sum-exp
    (4, 8, 32, 32, 100, 64, False),      # ... 1 block: 32 rows
    (2, 7, 20, 4, 300, 64, False),       # 280 heads, longest-first tail
])
def test_importance_launch_shapes(B, L, H, Hkv, N, D, negative):
    run_importance_case(B, L, H, Hkv, N, D, torch.bfloat16, negative)


@pytest.mark.parametrize("N", [300, 768])
def test_importance_workspace_limits(N):
    B, L, H, D = 1, 1, 4, 64
    q, k, scale = rand_qk(N, B, L, H, H, N, D, torch.bfloat16)
    want = oracle.importance(np32(q), np32(k), scale.numpy())
    rows = B * L * H * N * 4
    assert P.prefixkv_workspace_bytes(0, B, L, H, H, N, D, P.PKV_BF16) >= 2 * rows
    small = torch.empty((rows + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    lib = P.load()
    from paper_2412_03409_amd import binding as bind
    qd, kd, sd, out = q.to(DEV), k.to(DEV), scale.to(DEV), torch.empty((B, L, N), device=DEV)
    s = bind._shape(B, L, H, H, N, D, P.PKV_BF16)

    def call(nbytes):
        return lib.prefixkv_importance(s, bind._ptr(qd), bind._strides5(qd), bind._ptr(kd), bind._strides5(kd),
                                       bind._ptr(sd), None, bind._ptr(out), bind._ptr(small), nbytes, bind._stream())
    assert call(small.numel()) == 0
    check_importance(np32(out), want)
    assert call(small.numel() - 256) == 5


# sort_prefix_kernel: runs of 64 (one key per lane), 128, 256 and 512 keys; no, one and several merges; padding in the last
# run and in whole runs; ties across runs
@pytest.mark.parametrize("N", [63, 64, 65, 128, 129, 257, 640, 1025, 2048, 2049, 4097, 8191])
def test_sort_merges(N):
    check_select(synthetic_importance(1, 3, N, seed=N, ties=True), max(4, N))
    check_select(synthetic_importance(1, 2, N, seed=N + 1), max(3, N // 2))


# The probabilities of a 32-key tile are rounded to bf16 against the maximum over the keys up to the end of that tile.  Here
# key 0 scores 0, key 32 of the same 64-key stage scores d > 0 and every other key e^-60 less: a query that sees both weighs
# key 0 with exp(-d), in fp32, while its probability is exactly 1.  Values 1 and -bf16(exp(-d)) cancel but for the rounding
# of exp(-d) to 8 bits, which a reference taken over both tiles would put into the probability: the result would be 0.
def test_prefill_reference_per_tile():
    N, D = 192, 64
    d = torch.tensor([0.53125, 0.578125, 0.59375, 0.6875, 0.9375, 1.359375])      # exact in bf16
    H = d.numel()
    w = torch.exp(-d.double())
    wb = w.to(torch.bfloat16).double()
    want = (w - wb) / (1 + w)
    assert (want.abs() > 6e-4).all()
    q, k, v = (torch.zeros((1, 1, H, N, D), dtype=torch.float32) for _ in range(3))
    q[..., 0] = 1
    k[..., 0] = -60
    k[0, 0, :, 0, 0] = 0
    k[0, 0, :, 32, 0] = d
    v[0, 0, :, 0, :] = 1
    v[0, 0, :, 32, :] = -wb.float().view(H, 1)
    out, _ = P.prefixkv_prefill_attn(*(x.to(torch.bfloat16).to(DEV) for x in (q, k, v)), torch.ones(1, device=DEV))
    got = out[0, 0, :, 32:].cpu().double()
    # one bf16 rounding of the result, and a few fp32 roundings of the two terms of order one
    assert ((got - want.view(H, 1, 1)).abs() <= 2.0 ** -8 * want.abs().view(H, 1, 1) + 1e-6).all()


# Values in the future of a query do not reach it, whatever they are, unless they lie in its own 32-key tile (there they
# meet a probability of zero).
@pytest.mark.parametrize("N,D,rows", [(192, 128, (40, 97)), (192, 64, (32, 159)), (161, 128, (64, 160)), (300, 64, (224, 299))])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_prefill_non_finite_values(N, D, rows, bad):
    q, k, scale = rand_qk(N, 1, 2, 3, 3, N, D, torch.bfloat16)
    v = torch.randn(k.shape, generator=torch.Generator().manual_seed(N)).to(torch.bfloat16)
    clean, _ = P.prefixkv_prefill_attn(q.to(DEV), k.to(DEV), v.to(DEV), scale.to(DEV))
    for row in rows:
        vb = v.clone()
        vb[..., row, :] = bad
        out, _ = P.prefixkv_prefill_attn(q.to(DEV), k.to(DEV), vb.to(DEV), scale.to(DEV))
        first = row // 32 * 32
        assert torch.equal(out[..., :first, :], clean[..., :first, :])
        assert not torch.isfinite(out[..., row:, :]).any()


# A layer whose logit scale is NaN has no result; its neighbours do.
@pytest.mark.parametrize("D", [64, 128])
def test_prefill_nan_scale(D):
    q, k, scale = rand_qk(D, 1, 3, 2, 1, 200, D, torch.bfloat16)
    scale[1] = float("nan")
    out, lse = P.prefixkv_prefill_attn(q.to(DEV), k.to(DEV), k.to(DEV), scale.to(DEV))
    assert out[:, 1].isnan().all() and lse[:, 1].isnan().all()
    assert out[:, ::2].isfinite().all() and lse[:, ::2].isfinite().all()


# prefixkv_importance takes every workspace that holds what its kernels use, through the Python entry point as well: one
# sized for more layers, one sized for a given log-sum-exp (bf16, up to 768 positions), two rows for a long prompt.
@pytest.mark.parametrize("N,dtype,sized_for", [
    (680, torch.bfloat16, (32, False)), (680, torch.bfloat16, (2, True)), (300, torch.bfloat16, (2, False)),
    (801, torch.bfloat16, (2, False)), (1537, torch.bfloat16, (2, False)), (120, torch.float32, (2, False)),
])
def test_importance_workspace_of_other_calls(N, dtype, sized_for):
    B, L, H, D = 1, 2, 2, 64
    q, k, scale = rand_qk(N, B, L, H, H, N, D, dtype)
    want = oracle.importance(np32(q), np32(k), scale.numpy())
    code = P.PKV_BF16 if dtype == torch.bfloat16 else P.PKV_F32
    nbytes = P.prefixkv_workspace_bytes(0, B, sized_for[0], H, H, N, D, code, sized_for[1])
    row, rows = ((r * 4 * B * L * H * N + 255) // 256 * 256 for r in (1, 2))
    nbytes = min(nbytes, 2 * row)
    guarded = torch.full((nbytes + 4096,), 0x5a, dtype=torch.uint8, device=DEV)
    args = q.to(DEV), k.to(DEV), scale.to(DEV)
    check_importance(np32(P.prefixkv_importance(*args, ws=guarded[:nbytes])), want)
    assert (guarded[nbytes:] == 0x5a).all()
    least = 2 * row if dtype == torch.float32 else row if N <= 768 else rows
    check_importance(np32(P.prefixkv_importance(*args, ws=guarded[:least])), want)
    assert (guarded[nbytes:] == 0x5a).all()
    with pytest.raises(ValueError):
        P.prefixkv_importance(*args, ws=guarded[:least - 256])
    with pytest.raises(ValueError):
        P.prefixkv_importance(*args, ws=guarded[:0])


# Keys that score -inf weigh nothing, also where they fill the blocks a wavefront starts with (16 rows at D = 128 in bf16,
# 8 in fp32): with 8 and 4 wavefronts per unit and in the ranked launches.
@pytest.mark.parametrize("B,L,H,D,dtype,distance", [
    (1, 2, 2, 128, torch.bfloat16, 0), (1, 2, 2, 64, torch.float32, 0), (1, 18, 32, 128, torch.bfloat16, 0),
    (2, 18, 32, 128, torch.bfloat16, 0), (1, 2, 2, 128, torch.bfloat16, 3), (2, 18, 32, 64, torch.bfloat16, 3),
])
def test_decode_keys_at_minus_infinity(B, L, H, D, dtype, distance):
    N, inf_rows = 90, [*range(0, 33), *range(48, 64)]
    g = torch.Generator().manual_seed(B * L + D)
    k = torch.randn((B, L, H, N, D), generator=g).abs()
    k[:, :, :, inf_rows] = -float("inf")
    v, kn, vn = (torch.randn((B, L, H, n, D), generator=g).to(dtype) for n in (N, 1, 1))
    q = (torch.randn((B, L, H, D), generator=g).abs() + 0.1).to(dtype)
    k, scale = k.to(dtype), torch.full((L,), D ** -0.5)
    order = torch.arange(N, dtype=torch.int32).expand(B, L, N).contiguous().to(DEV)
    lengths = torch.full((B, L), N, dtype=torch.int32, device=DEV)
    cap = 1 + 2 * distance
    cache = P.prefixkv_compact(k.to(DEV), v.to(DEV), order, lengths, cap, B * L * (N + cap))
    new = kn[:, :, :, 0].contiguous().to(DEV), vn[:, :, :, 0].contiguous().to(DEV)
    if distance:
        out = P.prefixkv_decode_attn_evict(cache, lengths, q.to(DEV), *new, scale.to(DEV), N, 1, distance)
    else:
        out = P.prefixkv_decode_attn(cache, q.to(DEV), *new, scale.to(DEV), N)
    keys = torch.cat([k, kn], 3).double()
    s = (keys * q.double().unsqueeze(3)).sum(-1) * D ** -0.5
    want = (torch.softmax(s, -1).unsqueeze(-1) * torch.cat([v, vn], 3).double()).sum(3)
    assert (out.cpu().double() - want).abs().max() <= OUT_ATOL


# Ranked launches of heads that do not fill workgroups of four, so that these hold units of two segments; all three classes
# of segments, none, and the index order of many short units; groups of 2, 4 and 8 query heads in fp32.
@pytest.mark.parametrize("B,L,H,Hkv,N,D,dtype,frac,steps,layers", [
    (1, 50, 27, 27, 60, 64, torch.bfloat16, 0.4, 2, None),      # 1350 units: a quarter with four wavefronts, the others two
    (4, 23, 21, 21, 90, 128, torch.bfloat16, 0.4, 2, (1, 22)),  # 1764: an eighth with four and two each, 84 segments
    (7, 60, 7, 7, 60, 128, torch.bfloat16, 0.5, 2, None),       # 2940 units of 420 segments
    (33, 64, 1, 1, 40, 128, torch.bfloat16, 0.5, 1, None),      # one head: 2112 segments in five groups
    (12, 64, 6, 6, 30, 64, torch.bfloat16, 0.5, 1, None),       # 4608 units: index order
    (6, 60, 6, 3, 40, 64, torch.float32, 0.5, 2, None),         # fp32, groups of 2
    (9, 50, 12, 3, 40, 64, torch.float32, 0.5, 2, None),        # groups of 4
    (10, 40, 24, 3, 40, 128, torch.float32, 0.5, 1, None),      # groups of 8
    (2, 32, 160, 20, 60, 64, torch.float32, 0.4, 2, None),      # groups of 8, 64 segments
])
def test_decode_ranked_classes(B, L, H, Hkv, N, D, dtype, frac, steps, layers):
    run_decode_case(B, L, H, Hkv, N, D, dtype, frac, steps, seed=B * L + H, layer_range=layers)


@pytest.mark.parametrize("B,L,H,Hkv,N,D,dtype,frac,d,steps", [
    (2, 32, 18, 18, 40, 64, torch.bfloat16, 0.5, 2, 6),         # 1152 units of 64 segments
    (2, 32, 33, 33, 30, 128, torch.bfloat16, 0.5, 3, 7),        # 2112: one, two and four wavefronts per unit
    (8, 40, 14, 7, 24, 64, torch.float32, 0.5, 2, 5),           # fp32, groups of 2: 2240 units of 320 segments
])
def test_decode_evict_ranked_classes(B, L, H, Hkv, N, D, dtype, frac, d, steps):
    run_evict_case(B, L, H, Hkv, N, D, dtype, frac, d, steps, seed=B * L + H)


# The column sums with 64 rows per wavefront where their blocks fill one round of three workgroups per compute unit, next to
# the 32-row form just below and above (256 compute units)
@pytest.mark.parametrize("B,L,H,Hkv,N,D", [
    (8, 1, 27, 27, 513, 128),            # 648 blocks of 256 keys: 64 rows
    (8, 1, 26, 26, 513, 128),            # 624: 32 rows
    (8, 4, 8, 2, 521, 128),              # 768: 64 rows
    (8, 4, 9, 3, 521, 128),              # 864: 32 rows
    (1, 3, 36, 36, 1530, 128),           # 648 of six blocks: 64 rows
])
def test_importance_columns_one_round(B, L, H, Hkv, N, D):
    run_importance_on_gpu(B, L, H, Hkv, N, D, both=False)


def run_importance_on_gpu(B, L, H, Hkv, N, D, both=True):
    """Importance with a given log-sum-exp and, `both`, without, against fp64 on the GPU (the CPU oracle is slow here)."""
    q, k, scale = rand_qk(N + H, B, L, H, Hkv, N, D, torch.bfloat16)
    lse = torch.empty((B, L, H, N), device=DEV)
    want = torch.empty((B, L, N), dtype=torch.float64, device=DEV)
    qd, kd, future = q.to(DEV), k.to(DEV), torch.ones((N, N), dtype=torch.bool, device=DEV).triu_(1)
    for b in range(B):
        for l in range(L):
            kt = kd[b, l].double().transpose(1, 2).contiguous()
            s = torch.stack([qd[b, l, h].double() @ kt[h // (H // Hkv)] for h in range(H)]) * scale[l].item()
            s.masked_fill_(future, -float("inf"))
            lse[b, l] = torch.logsumexp(s, -1)
            want[b, l] = torch.softmax(s, -1).sum(1).mean(0)
    want = want.cpu().numpy()
    check_importance(np32(P.prefixkv_importance(qd, kd, scale.to(DEV), lse=lse)), want)
    if both:
        check_importance(np32(P.prefixkv_importance(qd, kd, scale.to(DEV))), want)


# Both sweeps of the stream kernels, 256 compute units: 32 rows per wavefront and one group of wavefronts (321 to about 1000
# blocks of 128 rows) at D = 128, and 64 rows (1024 blocks of 256 and more) with a remainder and with wavefronts wholly past the
# end at both head dimensions; six and four blocks whose ranks move on from head to head (512 and 672 heads, of which the last
# 344 and 512 run longest block first)
@pytest.mark.parametrize("B,L,H,Hkv,N,D", [
    (1, 7, 20, 4, 300, 128), (1, 2, 20, 4, 1153, 128), (1, 3, 13, 13, 1281, 128),
    (4, 2, 32, 32, 801, 128), (4, 2, 32, 32, 801, 64), (5, 4, 13, 13, 1030, 128), (3, 4, 17, 17, 1409, 64),
    (5, 4, 16, 4, 769, 128), (4, 4, 32, 8, 1300, 64), (3, 7, 32, 16, 900, 128),
])
def test_importance_stream_forms(B, L, H, Hkv, N, D):
    run_importance_on_gpu(B, L, H, Hkv, N, D)


# A row that holds NaN is refused by its status word, but its order stays a permutation, whatever the bits of the NaN: with a
# shared configuration the compaction reads it.
@pytest.mark.parametrize("N", [64, 200, 1025, 4097])
def test_order_of_nan_rows(N):
    imp = synthetic_importance(1, 3, N, seed=N)
    imp[0, 0] = torch.full((N,), -1, dtype=torch.int32).view(torch.float32)
    imp[0, 1, 0] = torch.tensor(-1, dtype=torch.int32).view(torch.float32)
    imp[0, 2, N // 2] = float("nan")
    r = P.prefixkv_rank(imp.to(DEV))
    assert r.status.item() & 1
    assert torch.equal(r.order.cpu().sort(-1).values, torch.arange(N, dtype=torch.int32).expand(1, 3, N))


# The head mean takes 2^30 values (one query expanded over a million sequences, so that they need 12 GB in all)
def test_importance_f32_largest_grid():
    B, L, N, D = 1 << 20, 64, 16, 64
    q, k, scale = rand_qk(3, 1, L, 1, 1, N, D, torch.float32)
    one = P.prefixkv_importance(q.to(DEV), k.to(DEV), scale.to(DEV))
    all_ = P.prefixkv_importance(q.to(DEV).expand(B, L, 1, N, D), k.to(DEV).expand(B, L, 1, N, D), scale.to(DEV))
    assert (all_ == one).all()


# One wavefront walks 4096 fp32 rows (2048 per half of its lanes) and adds a block of four of them at a time to its running
# sums.  With equal weights and one value v everywhere the sum of n blocks errs by at most half an ulp of every partial
# result, 2^-24 * (n + 1) / 2 of the total; adding row by row errs by 3e-5 for this v, whose remainder in the last binades is
# close to half an ulp.
def test_decode_long_sums():
    B, L, H, N, D = 2, 32, 32, 4096, 128
    v = np.uint32(0x3ffd8c03).view(np.float32)
    rows = B * L * N
    cache = P.CompactResult(
        kc=torch.zeros(rows * H * D, device=DEV), vc=torch.full((rows * H * D,), float(v), device=DEV),
        kept_pos=torch.zeros(rows, dtype=torch.int32, device=DEV),
        seg_off=(torch.arange(B * L, device=DEV) * N).view(B, L).contiguous(),
        caps=torch.full((B, L), N, dtype=torch.int32, device=DEV), lens=torch.full((B, L), N, dtype=torch.int32, device=DEV),
        cache_tokens=rows, Hkv=H, D=D)
    out = P.prefixkv_decode_attn(cache, torch.ones((B, L, H, D), device=DEV), None, None, torch.ones(L, device=DEV), N)
    blocks, rest = 512, 16       # rest: the block's own sum, the row groups, the quotient
    assert (out.double() / float(v) - 1).abs().max() <= 2.0 ** -24 * ((blocks + 1) / 2 + rest)
