"""HotPath.run_decode_loop: which tensors each step gets, without a GPU (the binding's entry points are recorded)."""
import pytest
import torch

from paper_2412_03409_amd import binding, pipeline

T, B, L, H, D = 3, 1, 2, 2, 64


@pytest.fixture
def path(monkeypatch):
    q = torch.zeros((B, L, H, 16, D))
    hp = pipeline.HotPath(q, q, q, torch.ones(L), 8, T)
    hp.calls = []
    monkeypatch.setattr(binding, "prefixkv_decode_attn",
                        lambda cache, q, k, v, scale, N, out, ws: hp.calls.append((q, k, v, out)) or out.fill_(len(hp.calls)))
    return hp


def tensors():
    return [torch.randn((T, B, L, H, D)) for _ in range(3)]


def check(hp, dq, dk, dv):
    assert len(hp.calls) == T
    for t, (q, k, v, out) in enumerate(hp.calls):
        assert torch.equal(q, dq[t]) and torch.equal(k, dk[t]) and torch.equal(v, dv[t])
        assert out.data_ptr() == hp.out[t].data_ptr()


def test_tensors_lists_and_mappings(path):
    dq, dk, dv = tensors()
    for x in ((dq, dk, dv), (torch.cat([dq, dq]), dk, dv), (list(dq), tuple(dk), dv), (dict(enumerate(dq)), dk, dv)):
        path.calls.clear()
        path.run_decode_loop(*x)
        check(path, dq, dk, dv)


def test_steps_made_from_the_outputs_before(path):
    """A sequence whose step t is made from the output of step t - 1."""
    dq, dk, dv = tensors()

    class Next:
        def __getitem__(self, t):
            if not 0 <= t < T:
                raise IndexError(t)
            return dq[t] + (path.out[t - 1].mean() if t else 0)

    path.run_decode_loop(Next(), dk, dv)
    assert [float((q - dq[t]).mean().round()) for t, (q, *_) in enumerate(path.calls)] == [0.0, 1.0, 2.0]


def test_a_step_of_the_callers_own(path):
    seen = []
    dq, dk, dv = tensors()
    path.run_decode_step = lambda t, q, k, v: seen.append((t, q, k, v))
    path.run_decode_loop(dq, dk, dv)
    assert [x[0] for x in seen] == list(range(T)) and all(x[1] is dq and x[2] is dk and x[3] is dv for x in seen)
    assert not path.calls


def test_too_few_steps(path):
    dq, dk, dv = tensors()
    for x in ((dq[:2], dk, dv), (dq, list(dk)[:2], dv)):
        with pytest.raises(IndexError):
            path.run_decode_loop(*x)


def test_a_decode_call_of_the_programs_own(monkeypatch):
    """A function in the place of the binding's is called for every step, also one put there before the pipeline is imported."""
    import importlib
    calls = []
    monkeypatch.setattr(binding, "prefixkv_decode_attn", lambda *a, **k: calls.append(a))
    fresh = importlib.util.module_from_spec(pipeline.__spec__)
    pipeline.__spec__.loader.exec_module(fresh)
    monkeypatch.setattr(torch.Tensor, "is_cuda", True)     # as on the GPU, where the loop's arguments are looked at once
    monkeypatch.setattr(binding, "load", lambda *a: pytest.fail("the library was called"))
    monkeypatch.setattr(binding, "prefixkv_workspace_bytes", lambda *a: 0)
    monkeypatch.setattr(binding, "select_workspace_bytes", lambda *a: 0)
    monkeypatch.setattr(binding, "prefixkv_cache_tokens_upper_bound", lambda *a: 8)
    q = torch.zeros((B, L, H, 16, D))
    hp = fresh.HotPath(q, q, q, torch.ones(L), 8, T)
    hp.run_decode_loop(*tensors())
    assert len(calls) == T
