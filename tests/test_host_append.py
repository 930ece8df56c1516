"""The native host path of an appended token: what it takes gives the bytes of the plain call through ctypes, what it does not take is left
to the binding's own checks, with their errors."""
import ctypes
import subprocess
import sys

import pytest
import torch

import paper_2505_24133_amd
from paper_2505_24133_amd import rkv


def _shape(**kw):
    return rkv.Shape(**{**dict(num_problems=2, kv_heads=2, q_heads=6, n_tokens=40, budget=24), **kw})


def _tensors(s, device, strided=False):
    gen = torch.Generator().manual_seed(5)

    def draw(*size):
        return torch.randn(size, generator=gen).bfloat16().to(device)

    P, H, Hq, N, a, d = s.num_problems, s.kv_heads, s.q_heads, s.n_tokens, s.alpha, s.head_dim
    if strided:
        k, v = draw(P, N + 3, H, d).transpose(1, 2)[:, :, :N], draw(P, H, N + 5, d)[:, :, :N]
        q = draw(P, a, Hq, d).transpose(1, 2)
    else:
        k, v, q = draw(P, H, N, d), draw(P, H, N, d), draw(P, Hq, a, d)
    return [k, v, q, draw(P, H, d), draw(P, H, d), draw(P, Hq, d)]


def test_calls_that_are_not_taken():
    rkv.load_library()
    s = _shape()
    good = _tensors(s, "cpu")
    assert rkv._append(s, *good, 0, 0) is None                                # not on a GPU
    assert rkv._append(s, None, *good[1:], 0, 0) is None
    assert rkv._append(s, *good, 0.0, 0) is None
    assert rkv._append(s, *good, 1 << 40, 0) is None
    for wrong in (dict(n_tokens=1 << 40), dict(lam=1), dict(flags=-1), dict(page_size=16)):
        assert rkv._append(_shape(**wrong), *good, 0, 0) is None
    assert rkv._append(object(), *good, 0, 0) is None
    with pytest.raises(TypeError):
        rkv._append(s, *good)
    with pytest.raises(RuntimeError, match="GPU tensors only"):
        rkv.rkv_cache_append(s, *good, 0, 0)


def _without_host(code, repo_root):
    """Runs `code` in a fresh interpreter in which the native host module does not load."""
    start = "import sys; sys.modules['paper_2505_24133_amd._host'] = None; import torch; from paper_2505_24133_amd import rkv; "
    r = subprocess.run([sys.executable, "-c", start + code], cwd=repo_root, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_the_library_works_without_the_host_module(repo_root):
    assert int(_without_host("print(rkv.rkv_workspace_size(rkv.Shape(2, 2, 6, 40, 24)))", repo_root)) == rkv.rkv_workspace_size(_shape())
    assert _without_host("rkv.load_library(); print(rkv._append(rkv.Shape(2, 2, 6, 40, 24), 0, 0, 0, 0, 0, 0, 0, 0))", repo_root) == "None\n"


@pytest.mark.gpu
def test_an_append_without_the_host_module(monkeypatch):
    print("[gpu-case] append without the host module", flush=True)
    monkeypatch.setitem(sys.modules, "paper_2505_24133_amd._host", None)
    monkeypatch.delattr(paper_2505_24133_amd, "_host", raising=False)
    monkeypatch.setattr(rkv, "_lib", None)
    monkeypatch.setattr(rkv, "_append", None)
    s = _shape()
    t = _tensors(s, "cuda")
    rkv.rkv_cache_append(s, *t, 11, 4)
    assert rkv._append(s, *t, 0, 0) is None
    assert torch.equal(t[0][:, :, 11], t[3]) and torch.equal(t[1][:, :, 11], t[4]) and torch.equal(t[2][:, :, 4], t[5])


@pytest.mark.gpu
@pytest.mark.parametrize("strided", [False, True])
def test_same_bytes_as_the_plain_call(strided):
    print(f"[gpu-case] host append strided={strided}", flush=True)
    rkv.load_library()
    s = _shape()
    native, plain = _tensors(s, "cuda", strided), _tensors(s, "cuda", strided)
    for row, slot in ((0, 0), (7, 3), (39, 7)):
        assert rkv._append(s, *native, row, slot) == rkv.RKV_OK
        prm = s.params(plain[0], plain[1], q=plain[2])
        assert rkv.load_library().rkv_cache_append(ctypes.byref(prm), *(t.data_ptr() for t in plain), row, slot, rkv._stream()) == rkv.RKV_OK
        for a, b in zip(native, plain):
            assert torch.equal(a, b)
        assert torch.equal(native[0][:, :, row], native[3]) and torch.equal(native[2][:, :, slot], native[5])


@pytest.mark.gpu
def test_stream_and_refusals():
    print("[gpu-case] host append stream and refusals", flush=True)
    rkv.load_library()
    s = _shape()
    t = _tensors(s, "cuda")
    other = torch.cuda.Stream()
    other.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(other):
        rkv.rkv_cache_append(s, *t, 5, 1)
    other.synchronize()
    assert torch.equal(t[1][:, :, 5], t[4])
    for row, slot in ((40, 0), (-1, 0), (0, 8), (0, -1)):
        with pytest.raises(rkv.RkvError) as e:
            rkv.rkv_cache_append(s, *t, row, slot)
        assert e.value.status == rkv.RKV_ERR_SHAPE
    for at, bad in ((0, t[0].float()), (3, t[3][:, :1]), (5, t[5].transpose(0, 1).contiguous().transpose(0, 1)), (2, t[2][..., :64]), (1, t[1].cpu())):
        wrong = list(t)
        wrong[at] = bad
        assert rkv._append(s, *wrong, 0, 0) is None
        with pytest.raises((ValueError, RuntimeError)):
            rkv.rkv_cache_append(s, *wrong, 0, 0)
    rkv.rkv_cache_append(s, *t, torch.tensor(6), 2)                           # not an int: the binding's own way
    assert torch.equal(t[0][:, :, 6], t[3])
    same = t[3].as_subclass(_Wrapped)                                         # nor a plain tensor
    assert rkv._append(s, t[0], t[1], t[2], same, t[4], t[5], 8, 2) is None
    rkv.rkv_cache_append(s, t[0], t[1], t[2], same, t[4], t[5], 8, 2)
    assert torch.equal(t[0][:, :, 8], t[3])


class _Wrapped(torch.Tensor):
    pass


class _Refusing(rkv.Shape):
    """A shape that fills the parameter block in its own way."""

    def params(self, *args, **kw):
        p = super().params(*args, **kw)
        p.head_dim = 64
        return p


@pytest.mark.gpu
def test_a_shape_of_another_class_is_asked_for_its_parameters():
    print("[gpu-case] host append shape subclass", flush=True)
    rkv.load_library()
    s = _Refusing(**{k: v for k, v in vars(_shape()).items()})
    t = _tensors(s, "cuda")
    before = t[0].clone()
    with pytest.raises(rkv.RkvError) as e:
        rkv.rkv_cache_append(s, *t, 5, 1)
    assert e.value.status == rkv.RKV_ERR_UNSUPPORTED and torch.equal(t[0], before)
