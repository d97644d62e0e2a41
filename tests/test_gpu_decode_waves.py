"""Decode launches whose units have one, two, four or all of a workgroup's wavefronts, the new row in any of their blocks, against the CPU oracle with the bars of the other GPU tests."""
import pytest
import torch

from paper_2412_03409_amd import binding
from paper_2412_03409_amd.pipeline import HotPath
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
    (1, 24, 32, 32, 300, 128, BF16, 0.3),    # 768, several to a workgroup
    (1, 44, 17, 17, 190, 128, BF16, 0.4),    # 748, wavefronts to spare in a segment's last workgroup
    (1, 43, 25, 25, 90, 64, BF16, 0.6),      # more than four per compute unit
    (1, 29, 25, 25, 130, 128, F32, 0.2),     # 725, an odd number of segments
])
def test_spread(B, L, H, Hkv, N, D, dt, frac):
    run_decode_case(B, L, H, Hkv, N, D, dt, frac, 3, seed=N)


@pytest.mark.parametrize("B,L,H,Hkv,N,D,dt,frac,d,steps", [
    (1, 32, 32, 32, 340, 128, BF16, 0.2, 40, 44),
    (1, 24, 20, 20, 200, 64, BF16, 0.1, 1, 5),
    (2, 15, 9, 3, 190, 128, F32, 0.3, 5, 9),
    (1, 32, 17, 17, 200, 64, BF16, 0.1, 1, 5),
])
def test_spread_with_pruning(B, L, H, Hkv, N, D, dt, frac, d, steps):
    run_evict_case(B, L, H, Hkv, N, D, dt, frac, d, steps, seed=N)


# The loop of HotPath looks at its arguments once; step by step, and from tensors that are not contiguous, the same bits.
@pytest.mark.parametrize("dt,Hkv", [(F32, 2), (BF16, 2), (BF16, 4)])
def test_loop_is_its_steps(dt, Hkv):
    B, L, H, N, D, T = 2, 3, 4, 40, 64, 5
    g = torch.Generator().manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g).to(dt).cuda()
    hp = HotPath(rnd(B, L, H, N, D), rnd(B, L, Hkv, N, D), rnd(B, L, Hkv, N, D), torch.full((L,), 0.1, device="cuda"), 30, T)
    hp.run_importance(); hp.run_select()
    dq, dk, dv = rnd(T + 1, B, L, H, D), rnd(T, B, L, Hkv, D), rnd(T, B, L, Hkv, D)
    wide = torch.zeros((T + 1, B, L, H, 2 * D), dtype=dt, device="cuda")
    wide[..., :D] = dq
    seen = []
    for form in ("loop", "steps", "lists"):
        hp.run_compact()
        hp.out.zero_()
        if form == "loop":
            hp.run_decode_loop(dq, dk, dv)
        elif form == "steps":
            for t in range(T):
                hp.run_decode_step(t, dq, dk, dv)
        else:
            hp.run_decode_loop(list(dq), list(dk), list(dv))
        torch.cuda.synchronize()
        seen.append((hp.out.clone(), hp.cache.lens.clone()))
    for out, lens in seen[1:]:
        assert torch.equal(out, seen[0][0]) and torch.equal(lens, seen[0][1])
    hp.run_compact()
    with pytest.raises(ValueError):
        hp.run_decode_loop(wide[..., :D], dk, dv)
    with pytest.raises(IndexError):
        hp.run_decode_loop(dq, dk[:T - 1], dv)


# What decode_attn_steps takes, and what it leaves to the steps: nothing is done then, and a step by itself accepts or refuses it as ever.
@pytest.mark.parametrize("Hkv", [4, 2])
def test_what_the_loop_takes(Hkv):
    B, L, H, N, D, T = 1, 3, 4, 40, 64, 3
    g = torch.Generator().manual_seed(7)
    rnd = lambda *s: torch.randn(s, generator=g).to(BF16).cuda()
    hp = HotPath(rnd(B, L, H, N, D), rnd(B, L, Hkv, N, D), rnd(B, L, Hkv, N, D), torch.full((L,), 0.1, device="cuda"), 30, T)
    hp.run_importance(); hp.run_select(); hp.run_compact()
    q, k, v = rnd(T, B, L, H, D), rnd(T, B, L, Hkv, D), rnd(T, B, L, Hkv, D)
    need = binding.prefixkv_workspace_bytes(binding.OP_DECODE, B, L, H, Hkv, N, D, binding.PKV_BF16)
    assert (need > 0) == (Hkv < H)
    lens, wide = hp.cache.lens.clone(), torch.cat([q, q], -1)
    args = dict(cache=hp.cache, q=q, k_new=k, v_new=v, scale=hp.scale, N=N, T=T, out=hp.out, ws=hp.dec_ws)
    bad = [dict(T=0), dict(T=T + 1), dict(q=q.float()), dict(k_new=k.float()), dict(out=hp.out.float()), dict(q=wide[..., :D]), dict(q=q[0]), dict(k_new=k[:, :, :2]),
           dict(out=hp.out[:, :, :, :2]), dict(q=q.cpu()), dict(k_new=None), dict(q=q.clone().requires_grad_()), dict(scale=hp.scale.double()), dict(scale=hp.scale[:2]),
           dict(scale=hp.scale.cpu()), dict(scale=torch.ones(2 * L, device="cuda")[::2]), dict(ws=None)]
    if need:
        bad.append(dict(ws=hp.dec_ws[:need - 1]))
    hp.out.fill_(7)
    for b in bad:
        assert binding.decode_attn_steps(**{**args, **b}) is False, list(b)
    torch.cuda.synchronize()
    assert torch.equal(hp.cache.lens, lens) and bool((hp.out == 7).all())
    hp.dec_ws, ws = None, hp.dec_ws                        # the steps have a workspace made then
    hp.run_decode_loop(q, k, v)
    want, hp.dec_ws = hp.out.clone(), ws
    hp.run_compact()
    assert binding.decode_attn_steps(**args) is True
    torch.cuda.synchronize()
    assert torch.equal(hp.out, want) and torch.equal(hp.cache.lens, lens + T)
    for name in ("vc", "seg_off", "caps", "lens"):         # refused by the library, by either path
        kept = getattr(hp.cache, name)
        setattr(hp.cache, name, None)
        with pytest.raises(binding.PrefixKVError):
            binding.prefixkv_decode_attn(hp.cache, q[0], k[0], v[0], hp.scale, N, ws=ws)
        with pytest.raises(binding.PrefixKVError):
            binding.decode_attn_steps(**args)
        setattr(hp.cache, name, kept)
