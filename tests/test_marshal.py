"""_marshal, the binding's fast way into the library: it does exactly the calls that the Python path accepts, with the same results, and
leaves everything else to it."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2505_09326_amd as pkg
from paper_2505_09326_amd._build import MARSHAL_PATH, build_marshal
from paper_2505_09326_amd.autograd import spherical_attention

DEV = "cuda:0"


class Refusing:
    """In _marshal's place: every call takes the Python path."""
    @staticmethod
    def forward(*args):
        return None
    backward = fp8_forward = forward


class Subclass(torch.Tensor):
    pass


@pytest.mark.parametrize("marshal", ["missing", "another torch's", "for another torch"])
def test_the_package_works_without_it(tmp_path, marshal):
    """build_library() is all that the binding needs: without _marshal, or with one that cannot be used, every call takes the Python path."""
    if not os.path.exists(pkg.LIB_PATH):
        pkg.build_library()
    copy, here = tmp_path / "paper_2505_09326_amd", os.path.dirname(pkg.__file__)
    copy.mkdir()
    for name in ("__init__.py", "_build.py", "autograd.py", "libsphattn.so"):
        os.symlink(os.path.join(here, name), copy / name)
    if marshal == "another torch's":               # (which the loader refuses)
        (copy / "_marshal.so").write_bytes(b"")
    if marshal == "for another torch":
        (copy / "_marshal.so").write_bytes(open(_built_marshal(), "rb").read())
    code = f"""
import torch
if {marshal == "for another torch"}:
    torch.__version__ = "0.0"
import paper_2505_09326_amd as pkg
assert pkg.__file__.startswith({str(tmp_path)!r}) and pkg.sphattn_version() > 0 and pkg._fast is pkg._PythonOnly
t = torch.zeros((1, 1, 8, 64), dtype=torch.bfloat16)
for call in (lambda: pkg.sphattn_fwd(t, t, t), lambda: pkg.sphattn_bwd(t, t, t, t, t, torch.zeros((1, 1, 8)))):
    try:
        call()
    except ValueError as e:
        assert "device tensor" in str(e), e
    else:
        raise AssertionError("accepted tensors of the CPU")
"""
    run = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, env={**os.environ, "PYTHONPATH": str(tmp_path)})
    assert run.returncode == 0, run.stderr[-2000:]


def _built_marshal():
    if not os.path.exists(MARSHAL_PATH):
        build_marshal()
    return MARSHAL_PATH


def test_what_is_not_right_is_left_to_python():
    _built_marshal()
    fast = pkg._bound_marshal(pkg.load_library())
    t = torch.zeros((1, 1, 8, 64), dtype=torch.bfloat16)
    fwd = lambda q, k, v, m=None, z=None, code=1: fast.forward(q, k, v, m, z, code, True, True, False)
    assert fwd(t, t, t) is None                    # not on a device
    assert fwd(t, t, None) is None and fwd(t.numpy, t, t) is None and fwd(t, t, t, 3) is None and fwd(t, t, t, code=9) is None
    assert fwd(t.as_subclass(Subclass), t, t) is None
    assert fast.backward(t, t, t, None, t, t, t, 1, True) is None and fast.fp8_forward(t, t, t, None, t) is None
    with pytest.raises(TypeError):
        fast.forward(t)
    with pytest.raises(TypeError):
        fast.forward(t, t, t, None, None, "bf16", True, True, False)


def _qkv(dtype, H, H_kv, Nq, Nk, d, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    r = lambda h, n: torch.randn((2, h, n, d), generator=g, device=DEV)
    q, k, v = r(H, Nq), r(H_kv, Nk), r(H_kv, Nk)
    if dtype in ("fp8qk_bf16v", "e4m3"):
        q, k = ((100 * x).clamp(-448, 448).to(torch.float8_e4m3fn) for x in (q, k))
    if dtype == "e4m3":
        return q, k, (100 * v).clamp(-448, 448).to(torch.float8_e4m3fn)
    t = {"f32": torch.float32, "f16": torch.float16}.get(dtype, torch.bfloat16)
    return (q if dtype == "fp8qk_bf16v" else q.to(t)), (k if dtype == "fp8qk_bf16v" else k.to(t)), v.to(t)


def _same(a, b):
    a, b = (x if isinstance(x, tuple) else (x,) for x in (a, b))
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert x.dtype == y.dtype and x.stride() == y.stride() and x.requires_grad == y.requires_grad and torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16", "fp8qk_bf16v"])
@pytest.mark.parametrize("H,H_kv,Nq,Nk,d", [(2, 2, 100, 100, 64), (4, 2, 33, 5000, 128)])
def test_forward_calls_equal_the_python_path(monkeypatch, dtype, H, H_kv, Nq, Nk, d):
    q, k, v = _qkv(dtype, H, H_kv, Nq, Nk, d, 31)
    m = torch.rand((2, Nk), device=DEV)
    z = torch.empty((2, H, Nq), device=DEV)
    calls = [lambda: pkg.sphattn_cross_fwd(q, k, v, dtype=dtype), lambda: pkg.sphattn_cross_fwd(q, k, v, m, Z=z, dtype=dtype)]
    if Nq == Nk:
        calls += [lambda: pkg.sphattn_fwd(q, k, v, dtype=dtype), lambda: pkg.sphattn_fwd_z(q, k, v, dtype=dtype), lambda: pkg.sphattn_grn_fwd(q, k, v, m, dtype=dtype)]
    fast = [c() for c in calls]
    for c in calls:                                # (it was not the Python path that did them)
        with monkeypatch.context() as patch:
            patch.setattr(pkg, "_check_forward", None)
            c()
    monkeypatch.setattr(pkg, "_fast", Refusing)
    for a, c in zip(fast, calls):
        _same(a, c())


@pytest.mark.gpu
@pytest.mark.parametrize("H,H_kv,N,counts", [(2, 2, 70, False), (4, 2, 700, True)])
def test_backward_and_training_step_equal_the_python_path(monkeypatch, H, H_kv, N, counts):
    q, k, v = (x.requires_grad_(True) for x in _qkv("f16", H, H_kv, N, N, 64, 32))
    m = torch.rand((2, N), device=DEV) if counts else None
    do = torch.randn(q.shape, device=DEV).half()

    def step():
        o = spherical_attention(q, k, v, m)
        return (o.detach(), *torch.autograd.grad(o, (q, k, v), do))
    with monkeypatch.context() as patch:
        patch.setattr(pkg, "_check_forward", None)
        patch.setattr(pkg, "_check_backward", None)
        fast = step()
    monkeypatch.setattr(pkg, "_fast", Refusing)
    _same(fast, step())


@pytest.mark.gpu
@pytest.mark.parametrize("counts", [False, True])
def test_e4m3_calls_equal_the_python_path(monkeypatch, counts):
    q, k, v = _qkv("e4m3", 4, 2, 300, 300, 64, 33)
    m = torch.rand((2, 300), device=DEV) if counts else None
    ws = torch.empty(pkg.sphattn_fp8_workspace_bytes(2, 2, 300, 64), dtype=torch.uint8, device=DEV)
    call = lambda: pkg.sphattn_fp8_grn_fwd(q, k, v, m, ws) if counts else pkg.sphattn_fp8_fwd(q, k, v, ws)
    with monkeypatch.context() as patch:
        patch.setattr(pkg, "_check_fp8", None)
        fast = call()
    monkeypatch.setattr(pkg, "_fast", Refusing)
    _same(fast, call())


@pytest.mark.gpu
def test_errors_are_the_python_paths():
    q, k, v = _qkv("bf16", 2, 2, 64, 64, 64, 34)
    with pytest.raises(ValueError, match="contiguous"):
        pkg.sphattn_fwd(q.transpose(1, 2).contiguous().transpose(1, 2), k, v)
    with pytest.raises(ValueError, match="K must have Q's N"):
        pkg.sphattn_fwd(q, k[:, :, :32].contiguous(), v[:, :, :32].contiguous())
    with pytest.raises(ValueError, match="V must have dtype"):
        pkg.sphattn_fwd(q, k, v.float())
    with pytest.raises(pkg.SphattnError):
        pkg.sphattn_fwd(*(x[..., :32].contiguous() for x in (q, k, v)))   # a head dimension the library does not have
    with pytest.raises(pkg.SphattnError):
        pkg.sphattn_fp8_fwd(*_qkv("e4m3", 2, 2, 64, 64, 64, 35), torch.empty(16, dtype=torch.uint8, device=DEV))


@pytest.mark.gpu
def test_the_current_stream_is_used():
    q, k, v = _qkv("bf16", 2, 2, 300, 300, 64, 36)
    want = pkg.sphattn_fwd(q, k, v)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        copies = [x + 0 for x in (q, k, v)]        # behind these, on the same stream
        got = pkg.sphattn_fwd(*copies)
    side.synchronize()
    assert torch.equal(got, want)


@pytest.mark.gpu
def test_modes_are_left_to_python():
    """Under a dispatch or a function mode nothing is allocated or launched in C++: the mode's own tensors go through Python's checks."""
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    q, k, v = _qkv("bf16", 2, 2, 64, 64, 64, 37)
    e4m3 = _qkv("e4m3", 2, 2, 64, 64, 64, 38)
    ws = torch.empty(pkg.sphattn_fp8_workspace_bytes(2, 2, 64, 64), dtype=torch.uint8, device=DEV)
    o, z = pkg.sphattn_fwd_z(q, k, v)

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    class Function(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    calls = [lambda: pkg._fast.forward(q, k, v, None, None, 1, True, True, False), lambda: pkg._fast.backward(q, k, v, None, o, q, z, 1, True),
             lambda: pkg._fast.fp8_forward(*e4m3, None, ws)]
    for mode in (Dispatch, Function):
        with mode():
            assert [c() for c in calls] == [None] * 3
            assert torch.equal(pkg.sphattn_fwd(q, k, v), o)
    assert all(c() is not None for c in calls)
