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


def _defects(t, of_shape=True):
    """What a tensor must not be, by name: a wrong size in each dimension, element type, layout, device, Python type."""
    out = {}
    if of_shape:
        for dim in range(t.dim()):
            out[f"size {dim}"] = t.narrow(dim, 0, t.size(dim) - 1).contiguous()
        out["dimensions"] = t[0]
    out["type"] = t.view(torch.int16) if t.element_size() == 2 else t.view(torch.int32) if t.element_size() == 4 else t.view(torch.int8)
    out["strides"] = torch.stack([t.view(out["type"].dtype)] * 2, -1)[..., 0].view(t.dtype)
    out["device"] = t.cpu()
    out["Python type"] = t.as_subclass(Subclass)
    out["no tensor"] = 3
    return out


def _refused(call, args, tensors):
    """call(*args) is done, and left to Python with any one defect in any one tensor."""
    assert call(*args) is not None
    for i, whole in tensors.items():
        for what, bad in _defects(args[i], whole).items():
            assert call(*args[:i], bad, *args[i + 1:]) is None, (i, what)
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_forward_takes_nothing_with_a_defect():
    q, k, v = _qkv("bf16", 4, 2, 64, 64, 64, 41)
    m, z = torch.rand((2, 64), device=DEV), torch.empty((2, 4, 64), device=DEV)
    fwd = pkg._fast.forward
    _refused(fwd, (q, k, v, m, z, 1, True, False, False), dict.fromkeys(range(5), True))
    _refused(fwd, (q, k, v, None, None, 1, False, False, True), {0: False, 1: False, 2: True})   # (rectangular: K's own size is N_k)
    assert fwd(q, k, v, m, z, 1, True, True, False) is None                        # shared heads where there are none
    k3, v3 = (torch.cat([x, x[:, :1]], 1) for x in (k, v))
    assert fwd(q, k3, v3, m, z, 1, True, False, False) is None                     # 3 does not divide 4
    k0, v0 = (x[:, :0].contiguous() for x in (k, v))
    assert fwd(q, k0, v0, m, z, 1, True, False, False) is None
    k63, v63 = (x[:, :, :63].contiguous() for x in (k, v))
    assert fwd(q, k63, v63, None, z, 1, True, False, False) is None and fwd(q, k63, v63, None, z, 1, False, False, False) is not None
    for code in (0, 2, 3, 4, -2, 9):
        assert fwd(q, k, v, m, z, code, True, False, False) is None, code
    for x in ("f32", "f16", "fp8qk_bf16v"):
        qx, kx, vx = _qkv(x, 4, 2, 64, 64, 64, 42)
        code = pkg._dtype_code(x)
        _refused(fwd, (qx, kx, vx, m, z, code, True, False, False), {0: True, 1: True, 2: True})
        assert fwd(qx, kx, v.to(torch.int16), m, z, code, True, False, False) is None and fwd(q, kx, vx, m, z, code, True, False, False) is None


@pytest.mark.gpu
def test_backward_takes_nothing_with_a_defect():
    q, k, v = _qkv("f16", 4, 2, 64, 64, 64, 43)
    m = torch.rand((2, 64), device=DEV)
    o, z = pkg._cross_fwd_z(q, k, v, m, "f16")
    do = torch.randn(q.shape, device=DEV).half()
    bwd, args = pkg._fast.backward, (q, k, v, m, o, do, z, 3, False)
    _refused(bwd, args, dict.fromkeys(range(7), True))
    assert bwd(q, k, v, m, o, do, z, 3, True) is None
    k3, v3 = (torch.cat([x, x[:, :1]], 1) for x in (k, v))
    assert bwd(q, k3, v3, m, o, do, z, 3, False) is None
    for code in (0, 1, 2, 4, -2):
        assert bwd(q, k, v, m, o, do, z, code, False) is None, code
    for i in (4, 5, 6):
        assert bwd(*args[:i], None, *args[i + 1:]) is None, i


@pytest.mark.gpu
def test_e4m3_takes_nothing_with_a_defect():
    q, k, v = _qkv("e4m3", 4, 2, 64, 64, 64, 44)
    m = torch.rand((2, 64), device=DEV)
    ws = torch.empty(pkg.sphattn_fp8_workspace_bytes(2, 2, 64, 64), dtype=torch.uint8, device=DEV)
    fp8 = pkg._fast.fp8_forward
    _refused(fp8, (q, k, v, m, ws), dict.fromkeys(range(4), True))
    for bad in (ws.cpu(), ws[None], torch.stack([ws, ws], -1)[:, 0], ws.as_subclass(Subclass), None):
        assert fp8(q, k, v, m, bad) is None
    k3, v3 = (torch.cat([x.view(torch.uint8), x.view(torch.uint8)[:, :1]], 1).view(torch.float8_e4m3fn) for x in (k, v))
    assert fp8(q, k3, v3, m, ws) is None
    with pytest.raises(pkg.SphattnError):          # (its size is the library's to check)
        fp8(q, k, v, m, ws[:-1])


@pytest.mark.gpu
def test_without_memory_for_the_workspace_a_call_runs_uncut(monkeypatch):
    """The allocator is held to 24 MB more than it has: enough for the outputs, not for the workspace (more than 30)."""
    q, k, v = _qkv("f32", 8, 2, 256, 16384, 128, 45)
    tq, tk, tv = _qkv("f16", 2, 2, 2048, 2048, 128, 46)
    to, tz = pkg.sphattn_fwd_z(tq, tk, tv, dtype="f16")
    lib = pkg.load_library()
    assert lib.sphattn_cross_splitkv_workspace_bytes(2, 8, 2, 256, 16384, 128, 0) >= 30 << 20
    assert lib.sphattn_bwd_workspace_bytes(2, 2, 2, 2048, 128, 3) >= 30 << 20
    forward, backward = lambda **kw: pkg.sphattn_cross_fwd(q, k, v, dtype="f32", **kw), lambda **kw: pkg.sphattn_bwd(tq, tk, tv, to, to, tz, dtype="f16", **kw)
    current = torch.cuda.current_stream().cuda_stream
    want = (forward(stream=current), backward(stream=current))   # uncut, as a call with a stream of its own is
    monkeypatch.setattr(pkg, "_check_forward", None)
    monkeypatch.setattr(pkg, "_check_backward", None)
    cut = (forward(), backward())
    torch.cuda.synchronize()
    assert not all(torch.equal(a, b) for a, b in zip((cut[0], *cut[1]), (want[0], *want[1])))
    del cut
    for call, ref in ((forward, want[0]), (backward, want[1])):
        torch.cuda.empty_cache()                   # room for the outputs, in one segment of 20 MB and a small one
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (24 << 20)) / torch.cuda.get_device_properties(0).total_memory)
        try:
            with pytest.raises(torch.OutOfMemoryError):
                torch.empty(30 << 20, dtype=torch.uint8, device=DEV)
            got = call()
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)
        _same(got, ref)


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
