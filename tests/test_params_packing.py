"""Shape.params fills the parameter block in one packing call: the same block as field by field (CPU)."""
import pytest
import torch

from paper_2505_24133_amd import rkv


def _by_field(s, k=None, v=None, q=None):
    p = rkv.RkvParams(s.num_problems, s.kv_heads, s.q_heads, s.n_tokens, s.head_dim, s.alpha, s.budget, s.pool_w, s.beta,
                      s.sim_threshold, s.lam, s.eps, s.flags)
    for name, t in (("k", k), ("v", v), ("q", q)):
        if t is not None and not (name == "q" and t.is_contiguous()):
            for i, what in enumerate(("problem", "head", "token")):
                setattr(p, f"{name}_stride_{what}", t.stride(i))
    return bytes(p)


@pytest.mark.parametrize("change", [{}, dict(alpha=16, pool_w=2, beta=3, sim_threshold=0.75, lam=0.3, eps=1e-6, flags=37),
                                    dict(flags=-1), dict(flags=1 << 33), dict(n_tokens=1 << 35), dict(num_problems=-1),
                                    dict(lam=float("nan")), dict(sim_threshold=1e39)])
def test_packed_block_equals_field_by_field(change):
    s = rkv.Shape(**{**dict(num_problems=2, kv_heads=2, q_heads=4, n_tokens=40, budget=24), **change})
    cache = torch.zeros((2, 48, 2, 128), dtype=torch.bfloat16)
    dense = torch.zeros((2, 2, 40, 128), dtype=torch.bfloat16)
    view = cache.transpose(1, 2)[:, :, :40]
    q = torch.zeros((2, 8, 4, 128), dtype=torch.bfloat16).transpose(1, 2)
    for args in ({}, dict(k=dense), dict(k=view, v=dense), dict(k=dense, v=view, q=q), dict(q=dense)):
        assert bytes(s.params(**args)) == _by_field(s, **args)


def test_stream_handle_without_the_private_call(monkeypatch):
    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(rkv, "_RAW_STREAM", None)
    assert rkv._stream() == 77
    monkeypatch.setattr(rkv, "_RAW_STREAM", lambda device: 100 + device)
    assert rkv._stream() == 103
