"""Spherical attention forward for AMD MI355X: thin binding over libsphattn.so.

Every step of the computation runs in the HIP kernels behind the C ABI of
include/sphattn.h; this module only marshals torch tensors (device memory and
streams) into that ABI.  There is no fallback: if the library has not been
built, importing the entry points raises.

Every entry point has a function of its name here except sphattn_cross_splitkv_fwd, sphattn_grn_bwd_split and
their _workspace_bytes: the forward and backward functions call those themselves where the library would cut
the launch into slices, provided that they allocate all outputs (no O, no gradients, no delta given) and no
stream handle is given.  The slices' workspace then comes from torch's allocator, at most 17 MB for a
forward call (68 MB in fp32) and 512 MiB for a backward call; where it gives none the call runs the uncut launch
without a word, as does a call that brings an output or a stream.  Cut and uncut launches agree to rounding,
not bit for bit, so sphattn_fwd_tile_rows, sphattn_normalized_fwd with "l2" and the like, which never cut, may
differ from sphattn_fwd in the last place.

Calls that allocate their outputs and give no stream go through _marshal (csrc/marshal.cpp), which does in C++ what the
functions here do in Python and does nothing where anything about a call is not as it has to be; the Python below it then
finds out what, and takes the calls that bring an output or a stream.  It takes all calls, at more host time each, where
_marshal is not built or was built for another torch.

The C ABI cannot see how large a buffer behind a pointer is, so the binding checks what it
can see before any launch: every tensor's shape against the shapes the entry point's header
states, its torch dtype against the `dtype` code, contiguity and device.  A mismatch raises
ValueError; nothing is enqueued.
"""
from __future__ import annotations

import ctypes
import functools
import os

from ._build import LIB_PATH, MARSHAL_PATH, build_library

SPHATTN_F32 = 0
SPHATTN_BF16 = 1
SPHATTN_FP8QK_BF16V = 2
SPHATTN_F16 = 3

_DTYPE_NAMES = {"f32": SPHATTN_F32, "bf16": SPHATTN_BF16, "fp8qk_bf16v": SPHATTN_FP8QK_BF16V,
                "f16": SPHATTN_F16}

EXPORTED_SYMBOLS = ("sphattn_fwd", "sphattn_fwd_z", "sphattn_fwd_tile_rows", "sphattn_grn_fwd",
                    "sphattn_normalized_fwd", "sphattn_softmax_fwd", "sphattn_cross_fwd", "sphattn_partial_fwd",
                    "sphattn_combine", "sphattn_splitkv_fwd", "sphattn_splitkv_workspace_bytes",
                    "sphattn_splitkv_heuristic", "sphattn_splitkv_fwd_noalloc",
                    "sphattn_cross_splitkv_workspace_bytes", "sphattn_cross_splitkv_fwd",
                    "sphattn_bwd", "sphattn_grn_bwd", "sphattn_bwd_workspace_bytes", "sphattn_grn_bwd_split",
                    "sphattn_fp8_workspace_bytes", "sphattn_fp8_fwd", "sphattn_fp8_grn_fwd", "sphattn_fp8_softmax_fwd",
                    "sphattn_strerror", "sphattn_version")

NORMALIZERS = {"l2": 0, "softmax": 1, "l1": 2, "sqrelu": 3}

_lib = None
_fast = None                                       # _marshal, bound to _lib's entry points, or _PythonOnly


class _PythonOnly:
    """In _marshal's place: every call takes the Python path."""
    @staticmethod
    def forward(*args):
        return None
    backward = fp8_forward = forward


class SphattnError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__(f"sphattn error {code}: {text}")
        self.code = code


def load_library() -> ctypes.CDLL:
    """Load the built library; raise if it is missing (no CPU fallback exists)."""
    global _lib, _fast
    if _lib is None:
        path = os.environ.get("SPHATTN_LIBRARY", LIB_PATH)   # another build of the same library
        if not os.path.exists(path):
            raise ImportError(
                f"{path} is not built; run `python -c 'import __graft_entry__ as g; g.build()'`")
        lib = ctypes.CDLL(path)
        vp, ip, sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t
        for name in ("sphattn_fwd", "sphattn_softmax_fwd"):
            fn = getattr(lib, name)
            fn.restype = ip
            fn.argtypes = [vp, vp, vp, vp, ip, ip, ip, ip, ip, vp]
        lib.sphattn_grn_fwd.restype = ip
        lib.sphattn_grn_fwd.argtypes = [vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_normalized_fwd.restype = ip
        lib.sphattn_normalized_fwd.argtypes = [vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_fwd_z.restype = ip
        lib.sphattn_fwd_z.argtypes = [vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, vp]
        lib.sphattn_fwd_tile_rows.restype = ip
        lib.sphattn_fwd_tile_rows.argtypes = [vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_cross_fwd.restype = ip
        lib.sphattn_cross_fwd.argtypes = [vp, vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_partial_fwd.restype = ip
        lib.sphattn_partial_fwd.argtypes = [vp, vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_combine.restype = ip
        lib.sphattn_combine.argtypes = [vp, vp, ip, vp, vp, ip, ip, ip, ip, ip, vp]
        lib.sphattn_splitkv_fwd.restype = ip
        lib.sphattn_splitkv_fwd.argtypes = [vp, vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, ip, vp, sz, vp]
        lib.sphattn_splitkv_fwd_noalloc.restype = ip
        lib.sphattn_splitkv_fwd_noalloc.argtypes = [vp, vp, vp, vp, vp, vp, ip, ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_splitkv_workspace_bytes.restype = sz
        lib.sphattn_splitkv_workspace_bytes.argtypes = [ip, ip, ip, ip, ip]
        lib.sphattn_splitkv_heuristic.restype = ip
        lib.sphattn_splitkv_heuristic.argtypes = [ip, ip, ip, ip, ip]
        lib.sphattn_cross_splitkv_workspace_bytes.restype = sz
        lib.sphattn_cross_splitkv_workspace_bytes.argtypes = [ip] * 7
        lib.sphattn_cross_splitkv_fwd.restype = ip
        lib.sphattn_cross_splitkv_fwd.argtypes = [vp] * 6 + [ip] * 7 + [vp, sz, vp]
        lib.sphattn_bwd.restype = ip
        lib.sphattn_bwd.argtypes = [vp] * 10 + [ip, ip, ip, ip, ip, vp]
        lib.sphattn_grn_bwd.restype = ip
        lib.sphattn_grn_bwd.argtypes = [vp] * 11 + [ip, ip, ip, ip, ip, ip, vp]
        lib.sphattn_bwd_workspace_bytes.restype = sz
        lib.sphattn_bwd_workspace_bytes.argtypes = [ip] * 6
        lib.sphattn_grn_bwd_split.restype = ip
        lib.sphattn_grn_bwd_split.argtypes = [vp] * 11 + [ip] * 6 + [vp, sz, vp]
        lib.sphattn_fp8_workspace_bytes.restype = sz
        lib.sphattn_fp8_workspace_bytes.argtypes = [ip, ip, ip, ip]
        for name in ("sphattn_fp8_fwd", "sphattn_fp8_softmax_fwd"):
            fn = getattr(lib, name)
            fn.restype = ip
            fn.argtypes = [vp, vp, vp, vp, vp, sz, ip, ip, ip, ip, ip, vp]
        lib.sphattn_fp8_grn_fwd.restype = ip
        lib.sphattn_fp8_grn_fwd.argtypes = [vp, vp, vp, vp, vp, vp, sz, ip, ip, ip, ip, ip, vp]
        lib.sphattn_strerror.restype = ctypes.c_char_p
        lib.sphattn_strerror.argtypes = [ip]
        lib.sphattn_version.restype = ip
        lib.sphattn_version.argtypes = []
        _fast = _bound_marshal(lib)                # (first: whoever sees _lib uses _fast)
        _lib = lib
    return _lib


def _bound_marshal(lib):
    """_marshal on the library's entry points, or _PythonOnly where it is not there for this torch."""
    if not os.path.exists(MARSHAL_PATH):
        return _PythonOnly
    try:
        import torch                               # (whose libraries it links against)
        from . import _marshal
    except ImportError:                            # no torch, or one with other symbols
        return _PythonOnly
    if getattr(_marshal, "built_for", None) != torch.__version__:
        return _PythonOnly
    names = ("sphattn_cross_fwd", "sphattn_cross_splitkv_fwd", "sphattn_cross_splitkv_workspace_bytes", "sphattn_grn_bwd",
             "sphattn_grn_bwd_split", "sphattn_bwd_workspace_bytes", "sphattn_fp8_grn_fwd")
    _marshal.bind(_raise_on, *(ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in names))
    return _marshal


def sphattn_strerror(code: int) -> str:
    return load_library().sphattn_strerror(int(code)).decode()


def sphattn_version() -> int:
    return int(load_library().sphattn_version())


def _dtype_code(dtype) -> int:
    if isinstance(dtype, str):
        return _DTYPE_NAMES[dtype]
    return int(dtype)


# The smallest calls are bound by what happens on the host before the launch, so the checks run
# twice at most: one pass of plain comparisons that accepts what is right (`_fits_forward`), and, only when
# that says no, the checks below it, which find out what is wrong and say so.  One call of
# sphattn_fwd on 64 rows: 13.6 us of host time with the second kind alone, 8.5 with both.

@functools.lru_cache(maxsize=None)
def _type_tables():
    """Element types of (Q and K, V and O) by dtype code."""
    import torch
    f32, f16, bf16 = (torch.float32,), (torch.float16,), (torch.bfloat16,)
    return {SPHATTN_F32: (f32, f32), SPHATTN_F16: (f16, f16), SPHATTN_BF16: (bf16, bf16),
            SPHATTN_FP8QK_BF16V: ((torch.float8_e4m3fn, torch.uint8), bf16)}


def _fits_forward(Q, K, V, O, mult, Z, code, same_n, same_h):
    """(B, H, N_q, d, H_kv, N_k) if everything about a forward call's tensors is as it has to be, else None."""
    if Q is None or K is None or V is None or O is None:
        return None
    sq, sk = Q.shape, K.shape
    if len(sq) != 4 or len(sk) != 4 or V.shape != sk or O.shape != sq:
        return None
    B, H, Nq, d = sq
    Bk, H_kv, Nk, dk = sk
    if Bk != B or dk != d or H_kv <= 0 or H % H_kv or (same_n and Nk != Nq) or (same_h and H_kv != H):
        return None
    qk, vo = _type_tables().get(code, ((), ()))
    if Q.dtype not in qk or K.dtype not in qk or V.dtype not in vo or O.dtype not in vo:
        return None
    gpu = Q.get_device()
    if not (Q.is_cuda and K.get_device() == gpu and V.get_device() == gpu and O.get_device() == gpu and
            K.is_cuda and V.is_cuda and O.is_cuda and
            Q.is_contiguous() and K.is_contiguous() and V.is_contiguous() and O.is_contiguous()):
        return None
    for t, shape in ((mult, (B, Nk)), (Z, (B, H, Nq))):
        if t is not None and not (t.shape == shape and t.dtype in _f32_types() and t.is_contiguous() and
                                  t.is_cuda and t.get_device() == gpu):
            return None
    return B, H, Nq, d, H_kv, Nk


def _fits_backward(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, code):
    """(B, H, N, d, H_kv) if everything about a backward call's tensors is as it has to be, else None."""
    like_q, like_k = (Q, O, dO, dQ), (K, V, dK, dV)
    if any(t is None for t in like_q + like_k + (Z, delta)) or code not in (SPHATTN_BF16, SPHATTN_F16):
        return None
    sq, sk = Q.shape, K.shape
    if len(sq) != 4 or len(sk) != 4:
        return None
    B, H, N, d = sq
    Bk, H_kv, Nk, dk = sk
    if Bk != B or dk != d or Nk != N or H_kv <= 0 or H % H_kv or not Q.is_cuda:
        return None
    gpu, (t16,), (f32,) = Q.get_device(), _vo_types(code), _f32_types()
    for ts, shape, dtype in ((like_q, sq, t16), (like_k, sk, t16), ((Z,), (B, H, N), f32), ((delta,), (2, B, H, N), f32),
                             (() if mult is None else (mult,), (B, N), f32)):
        for t in ts:
            if t.shape != shape or t.dtype != dtype or not t.is_contiguous() or not t.is_cuda or t.get_device() != gpu:
                return None
    return B, H, N, d, H_kv


# ---- what the binding can check and the C ABI cannot: shapes and element types -------------

def _qk_types(code):
    return _type_tables()[code][0]


def _vo_types(code):
    import torch
    return _type_tables().get(code, ((), (torch.bfloat16,)))[1]


def _e4m3_types():
    import torch
    return (torch.float8_e4m3fn, torch.uint8)


@functools.lru_cache(maxsize=None)
def _f32_types():
    import torch
    return (torch.float32,)


def _need(name, t, shape, types, optional=False):
    """Shape, element type and contiguity of one argument (its device: _on_device, once the
    shapes of all arguments have been checked)."""
    if t is None:
        if optional:
            return
        raise ValueError(f"{name} is required")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} must have shape {tuple(shape)}, got {tuple(t.shape)}")
    if t.dtype not in types:
        raise ValueError(f"{name} must have dtype {' or '.join(str(x) for x in types)}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")


def _on_device(**tensors):
    """All the (non-None) arguments of a call must live on one GPU."""
    first = None
    for name, t in tensors.items():
        if t is None:
            continue
        if not t.is_cuda:
            raise ValueError(f"{name} must be a device tensor")
        if first is None:
            first = (name, t.device)
        elif t.device != first[1]:
            raise ValueError(f"{name} is on {t.device}, {first[0]} on {first[1]}")


def _shape4(name, t):
    if t is None or t.dim() != 4:
        raise ValueError(f"{name} must be a [B,H,N,d] tensor")
    return tuple(int(x) for x in t.shape)


def _kv_shape(Q, K, same_n):
    """(B, H, N_q, d, H_kv, N_k) from Q [B,H,N_q,d] and K [B,H_kv,N_k,d]."""
    B, H, Nq, d = _shape4("Q", Q)
    Bk, H_kv, Nk, dk = _shape4("K", K)
    if Bk != B or dk != d:
        raise ValueError(f"K must be [B,H_kv,N_k,d] with Q's B and d, got {tuple(K.shape)} for Q {tuple(Q.shape)}")
    if H_kv <= 0 or H % H_kv != 0:
        raise ValueError(f"the number of K/V heads ({H_kv}) must divide the number of query heads ({H})")
    if same_n and Nk != Nq:
        raise ValueError(f"K must have Q's N ({Nq}), got {Nk}: this entry point is self-attention")
    return B, H, Nq, d, H_kv, Nk


def _check_forward(Q, K, V, O, mult, Z, code, same_n=True, same_h=False):
    fits = _fits_forward(Q, K, V, O, mult, Z, code, same_n, same_h)
    if fits is not None:
        return fits
    B, H, Nq, d, H_kv, Nk = _kv_shape(Q, K, same_n)
    if same_h and H_kv != H:
        raise ValueError(f"K must have Q's {H} heads, got {H_kv}")
    _need("Q", Q, (B, H, Nq, d), _qk_types(code))
    _need("K", K, (B, H_kv, Nk, d), _qk_types(code))
    _need("V", V, (B, H_kv, Nk, d), _vo_types(code))
    _need("O", O, (B, H, Nq, d), _vo_types(code))
    _need("mult", mult, (B, Nk), _f32_types(), optional=True)
    _need("Z", Z, (B, H, Nq), _f32_types(), optional=True)
    _on_device(Q=Q, K=K, V=V, O=O, mult=mult, Z=Z)
    return B, H, Nq, d, H_kv, Nk


def _alloc_out(Q, dtype):
    import torch
    out = _vo_types(_dtype_code(dtype))[0]
    if Q.dtype == out and Q.is_contiguous():
        return torch.empty_like(Q)
    return torch.empty(Q.shape, dtype=out, device=Q.device)


def _stream_of(t, stream):
    """The stream handle of a call: the one given, or torch's current stream on the tensor's GPU."""
    if stream is not None:
        return stream
    import torch
    return torch._C._cuda_getCurrentRawStream(t.device.index)


def _ptr(t):
    return t.data_ptr() if t is not None else None


def _raise_on(rc):
    if rc != 0:
        raise SphattnError(rc, sphattn_strerror(rc))


@functools.lru_cache(maxsize=1024)
def _cut_workspace_bytes(device_index, B, H, H_kv, Nq, Nk, d, code):
    """Workspace of the library's choice of key slices: a function of the shape and the GPU."""
    return load_library().sphattn_cross_splitkv_workspace_bytes(B, H, H_kv, Nq, Nk, d, code)


def _workspace(need, like):
    """`need` bytes on the GPU of `like`, or None: for 0 bytes, and where memory is too short for them
    (the uncut launches need none)."""
    if not need:
        return None
    import torch
    try:
        return torch.empty(need, dtype=torch.uint8, device=like.device)
    except torch.OutOfMemoryError:
        return None


def _launch_cross(lib, Q, K, V, mult, O, Z, B, H, H_kv, Nq, Nk, d, code, stream, own_output):
    """sphattn_cross_fwd on checked arguments.  Where the library would cut the key axis (few query
    rows against many keys) and this call allocates its output anyway, the slices' workspace (17 MB at most, 68
    in fp32) comes from torch's allocator too: on the current stream, so its reuse is ordered behind the launch.
    A caller that brings O or a stream handle of its own gets no allocation and the unsplit launch."""
    args = (Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult), O.data_ptr(), _ptr(Z), B, H, H_kv, Nq, Nk, d, code)
    need = _cut_workspace_bytes(Q.device.index, B, H, H_kv, Nq, Nk, d, code) if own_output and stream is None else 0
    ws = _workspace(need, Q)
    if ws is None:
        _raise_on(lib.sphattn_cross_fwd(*args, _stream_of(Q, stream)))
    else:
        _raise_on(lib.sphattn_cross_splitkv_fwd(*args, ws.data_ptr(), need, _stream_of(Q, None)))


# ---- entry points, same names as the C ABI ----------------------------------------------------

def sphattn_fwd(Q, K, V, O=None, dtype="bf16", stream=None):
    """O = (Q K^T) V with each score row divided by its L2 norm; tensors are [B,H,N,d]."""
    lib, code, own_output = load_library(), _dtype_code(dtype), O is None
    if O is None:
        done = _fast.forward(Q, K, V, None, None, code, True, True, False) if stream is None else None
        if done is not None:
            return done
        O = _alloc_out(Q, dtype)
    B, H, N, d, _, _ = _check_forward(Q, K, V, O, None, None, code, same_h=True)
    _launch_cross(lib, Q, K, V, None, O, None, B, H, H, N, N, d, code, stream, own_output)
    return O


def sphattn_softmax_fwd(Q, K, V, O=None, dtype="bf16", stream=None):
    """Comparison twin: softmax(Q K^T / sqrt(d)) V on the same tiling."""
    lib, code = load_library(), _dtype_code(dtype)
    if O is None:
        O = _alloc_out(Q, dtype)
    B, H, N, d, _, _ = _check_forward(Q, K, V, O, None, None, code, same_h=True)
    _raise_on(lib.sphattn_softmax_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(),
                                      B, H, N, d, code, _stream_of(Q, stream)))
    return O


def sphattn_fwd_z(Q, K, V, O=None, Z=None, dtype="bf16", stream=None):
    """sphattn_fwd that also returns the row aggregates z_i = sum_j s_ij^2: (O, Z [B,H,N] fp32)."""
    import torch
    lib, code, own_output = load_library(), _dtype_code(dtype), O is None
    if O is None:
        done = _fast.forward(Q, K, V, None, Z, code, True, True, Z is None) if stream is None else None
        if done is not None:
            return done if Z is None else (done, Z)
        O = _alloc_out(Q, dtype)
    if Z is None:
        Z = torch.empty(Q.shape[:3], dtype=torch.float32, device=Q.device)
    B, H, N, d, _, _ = _check_forward(Q, K, V, O, None, Z, code, same_h=True)
    _launch_cross(lib, Q, K, V, None, O, Z, B, H, H, N, N, d, code, stream, own_output)
    return O, Z


def sphattn_fwd_tile_rows(Q, K, V, O=None, Z=None, dtype="bf16", tile_rows=0, stream=None):
    """sphattn_fwd_z in one launch, with the workgroup shape forced to 128 or 256 query rows (0: the library's
    choice); returns (O, Z), Z being None unless given."""
    lib, code = load_library(), _dtype_code(dtype)
    if O is None:
        O = _alloc_out(Q, dtype)
    B, H, N, d, _, _ = _check_forward(Q, K, V, O, None, Z, code, same_h=True)
    _raise_on(lib.sphattn_fwd_tile_rows(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), _ptr(Z),
                                        B, H, N, d, code, int(tile_rows), _stream_of(Q, stream)))
    return O, Z


def sphattn_grn_fwd(Q, K, V, mult=None, O=None, dtype="bf16", stream=None):
    """Gene-regulatory-network variant: keys scaled by per-gene multiplicity mult[B,N] (fp32 or
    None) and K, V of shape [B,H_kv,N,d] shared by groups of H/H_kv query heads."""
    lib, code, own_output = load_library(), _dtype_code(dtype), O is None
    if O is None:
        done = _fast.forward(Q, K, V, mult, None, code, True, False, False) if stream is None else None
        if done is not None:
            return done
        O = _alloc_out(Q, dtype)
    B, H, N, d, H_kv, _ = _check_forward(Q, K, V, O, mult, None, code)
    _launch_cross(lib, Q, K, V, mult, O, None, B, H, H_kv, N, N, d, code, stream, own_output)
    return O


def sphattn_normalized_fwd(Q, K, V, O=None, dtype="bf16", normalizer="l2", stream=None):
    """Attention with the normalizer "l2", "softmax", "l1" or "sqrelu" in place of the SoftMax."""
    lib, code = load_library(), _dtype_code(dtype)
    if O is None:
        O = _alloc_out(Q, dtype)
    B, H, N, d, _, _ = _check_forward(Q, K, V, O, None, None, code, same_h=True)
    norm = NORMALIZERS[normalizer] if isinstance(normalizer, str) else int(normalizer)
    _raise_on(lib.sphattn_normalized_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(),
                                         B, H, N, d, code, norm, _stream_of(Q, stream)))
    return O


def sphattn_cross_fwd(Q, K, V, mult=None, O=None, Z=None, dtype="bf16", stream=None):
    """Spherical attention of Q [B,H,N_q,d] over the keys K, V [B,H_kv,N_k,d] (optional
    multiplicities mult [B,N_k], optional row aggregates Z [B,H,N_q]); returns O [B,H,N_q,d]."""
    lib, code, own_output = load_library(), _dtype_code(dtype), O is None
    if O is None:
        done = _fast.forward(Q, K, V, mult, Z, code, False, False, False) if stream is None else None
        if done is not None:
            return done
        O = _alloc_out(Q, dtype)
    B, H, Nq, d, H_kv, Nk = _check_forward(Q, K, V, O, mult, Z, code, same_n=False)
    _launch_cross(lib, Q, K, V, mult, O, Z, B, H, H_kv, Nq, Nk, d, code, stream, own_output)
    return O


def _cross_fwd_z(Q, K, V, mult, dtype):
    """sphattn_cross_fwd of a self-attention shape that also returns the row aggregates: (O, Z)."""
    import torch
    load_library()
    done = _fast.forward(Q, K, V, mult, None, _dtype_code(dtype), True, False, True)
    if done is not None:
        return done
    Z = torch.empty(Q.shape[:3], dtype=torch.float32, device=Q.device)
    return sphattn_cross_fwd(Q, K, V, mult, Z=Z, dtype=dtype), Z


def sphattn_partial_fwd(Q, K, V, mult=None, o_part=None, z_part=None, dtype="bf16", stream=None):
    """Unnormalised accumulator pair of Q [B,H,N_q,d] over the keys K, V [B,H_kv,N_k,d]:
    (o_part [B,H,N_q,d] fp32, z_part [B,H,N_q] fp32)."""
    import torch
    lib, code = load_library(), _dtype_code(dtype)
    if o_part is None:
        o_part = torch.empty(Q.shape, dtype=torch.float32, device=Q.device)
    if z_part is None:
        z_part = torch.empty(Q.shape[:3], dtype=torch.float32, device=Q.device)
    B, H, Nq, d, H_kv, Nk = _kv_shape(Q, K, same_n=False)
    _need("Q", Q, (B, H, Nq, d), _qk_types(code))
    _need("K", K, (B, H_kv, Nk, d), _qk_types(code))
    _need("V", V, (B, H_kv, Nk, d), _vo_types(code))
    _need("mult", mult, (B, Nk), _f32_types(), optional=True)
    _need("o_part", o_part, (B, H, Nq, d), _f32_types())
    _need("z_part", z_part, (B, H, Nq), _f32_types())
    _on_device(Q=Q, K=K, V=V, mult=mult, o_part=o_part, z_part=z_part)
    _raise_on(lib.sphattn_partial_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult),
                                      o_part.data_ptr(), z_part.data_ptr(), B, H, H_kv, Nq, Nk, d,
                                      code, _stream_of(Q, stream)))
    return o_part, z_part


def sphattn_combine(o_parts, z_parts, O=None, Z=None, dtype="bf16", stream=None):
    """Tail of the summed accumulators: o_parts [P,B,H,N,d], z_parts [P,B,H,N] (fp32) -> O."""
    import torch
    lib, code = load_library(), _dtype_code(dtype)
    if o_parts is None or o_parts.dim() != 5:
        raise ValueError("o_parts must be a [P,B,H,N,d] tensor")
    P, B, H, N, d = (int(x) for x in o_parts.shape)
    if O is None:
        O = torch.empty((B, H, N, d), dtype=_vo_types(code)[0], device=o_parts.device)
    _need("o_parts", o_parts, (P, B, H, N, d), _f32_types())
    _need("z_parts", z_parts, (P, B, H, N), _f32_types())
    _need("O", O, (B, H, N, d), _vo_types(code))
    _need("Z", Z, (B, H, N), _f32_types(), optional=True)
    _on_device(o_parts=o_parts, z_parts=z_parts, O=O, Z=Z)
    _raise_on(lib.sphattn_combine(o_parts.data_ptr(), z_parts.data_ptr(), P, O.data_ptr(), _ptr(Z),
                                  B, H, N, d, code, _stream_of(o_parts, stream)))
    return O


def sphattn_splitkv_workspace_bytes(B, H, N, d, n_splits) -> int:
    return int(load_library().sphattn_splitkv_workspace_bytes(B, H, N, d, n_splits))


def sphattn_splitkv_heuristic(B, H, N, d, dtype="bf16") -> int:
    return int(load_library().sphattn_splitkv_heuristic(B, H, N, d, _dtype_code(dtype)))


def _need_workspace(workspace):
    """Size in bytes of a workspace argument (its device is checked with the other arguments')."""
    if workspace is None or workspace.dim() != 1:
        raise ValueError("workspace must be a one-dimensional device byte tensor")
    _need("workspace", workspace, workspace.shape, (workspace.dtype,))
    return workspace.numel() * workspace.element_size()


def sphattn_splitkv_fwd(Q, K, V, workspace, mult=None, O=None, Z=None, n_splits=0, dtype="bf16", stream=None):
    """sphattn_grn_fwd with the key axis cut into n_splits slices (0: the library's choice);
    `workspace` is a device byte tensor of at least sphattn_splitkv_workspace_bytes(...)."""
    lib, code = load_library(), _dtype_code(dtype)
    if O is None:
        O = _alloc_out(Q, dtype)
    ws_bytes = _need_workspace(workspace)
    B, H, N, d, H_kv, _ = _check_forward(Q, K, V, O, mult, Z, code)
    _on_device(Q=Q, workspace=workspace)
    _raise_on(lib.sphattn_splitkv_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult), O.data_ptr(), _ptr(Z),
                                      B, H, H_kv, N, d, code, int(n_splits),
                                      workspace.data_ptr(), ws_bytes, _stream_of(Q, stream)))
    return O


NOALLOC_SCRATCH_BYTES = 64 << 20   # SPHATTN_NOALLOC_SCRATCH_BYTES of include/sphattn.h


def sphattn_splitkv_fwd_noalloc(Q, K, V, O, mult=None, Z=None, n_splits=0, dtype="bf16", stream=None):
    """sphattn_splitkv_fwd on the library's own scratch array (NOALLOC_SCRATCH_BYTES): no
    workspace argument and no allocation anywhere in the call, so O must be given."""
    lib, code = load_library(), _dtype_code(dtype)
    B, H, N, d, H_kv, _ = _check_forward(Q, K, V, O, mult, Z, code)
    _raise_on(lib.sphattn_splitkv_fwd_noalloc(Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult), O.data_ptr(),
                                              _ptr(Z), B, H, H_kv, N, d, code, int(n_splits), _stream_of(Q, stream)))
    return O


def sphattn_fp8_workspace_bytes(B, H_kv, N, d) -> int:
    """Workspace of sphattn_fp8_fwd for K, V of shape [B,H_kv,N,d]."""
    return int(load_library().sphattn_fp8_workspace_bytes(B, H_kv, N, d))


def _check_fp8(Q, K, V, O, mult):
    import torch
    B, H, N, d, H_kv, _ = _kv_shape(Q, K, same_n=True)
    _need("Q", Q, (B, H, N, d), _e4m3_types())
    _need("K", K, (B, H_kv, N, d), _e4m3_types())
    _need("V", V, (B, H_kv, N, d), _e4m3_types())
    _need("O", O, (B, H, N, d), (torch.bfloat16,))
    _need("mult", mult, (B, N), _f32_types(), optional=True)
    _on_device(Q=Q, K=K, V=V, O=O, mult=mult)
    return B, H, N, d, H_kv


def sphattn_fp8_fwd(Q, K, V, workspace, O=None, stream=None, _entry="sphattn_fp8_fwd"):
    """Spherical attention with Q [B,H,N,d], K and V [B,H_kv,N,d] all stored in E4M3
    (float8_e4m3fn tensors) and both contractions on the fp8 matrix instructions; O is bfloat16.
    `workspace` is a device byte tensor of at least sphattn_fp8_workspace_bytes(B, H_kv, N, d)."""
    import torch
    lib = load_library()
    if O is None:
        done = _fast.fp8_forward(Q, K, V, None, workspace) if stream is None and _entry == "sphattn_fp8_fwd" else None
        if done is not None:
            return done
        O = torch.empty(Q.shape, dtype=torch.bfloat16, device=Q.device)
    ws_bytes = _need_workspace(workspace)
    B, H, N, d, H_kv = _check_fp8(Q, K, V, O, None)
    _on_device(Q=Q, workspace=workspace)
    _raise_on(getattr(lib, _entry)(Q.data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), workspace.data_ptr(),
                                   ws_bytes, B, H, H_kv, N, d, _stream_of(Q, stream)))
    return O


def sphattn_fp8_softmax_fwd(Q, K, V, workspace, O=None, stream=None):
    """SoftMax comparison twin of sphattn_fp8_fwd (same arguments): for timing, on inputs of
    moderate size."""
    return sphattn_fp8_fwd(Q, K, V, workspace, O=O, stream=stream, _entry="sphattn_fp8_softmax_fwd")


def sphattn_fp8_grn_fwd(Q, K, V, mult, workspace, O=None, stream=None):
    """sphattn_fp8_fwd with per-gene multiplicities mult [B,N] (fp32, or None) on the scores."""
    import torch
    lib = load_library()
    if O is None:
        done = _fast.fp8_forward(Q, K, V, mult, workspace) if stream is None else None
        if done is not None:
            return done
        O = torch.empty(Q.shape, dtype=torch.bfloat16, device=Q.device)
    ws_bytes = _need_workspace(workspace)
    B, H, N, d, H_kv = _check_fp8(Q, K, V, O, mult)
    _on_device(Q=Q, workspace=workspace)
    _raise_on(lib.sphattn_fp8_grn_fwd(Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult), O.data_ptr(),
                                      workspace.data_ptr(), ws_bytes, B, H, H_kv, N, d, _stream_of(Q, stream)))
    return O


def _check_backward(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, code):
    fits = _fits_backward(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, code)
    if fits is not None:
        return fits
    if code not in (SPHATTN_BF16, SPHATTN_F16):
        raise ValueError("the backward pass takes 16-bit storage (bf16 or f16)")
    B, H, N, d, H_kv, _ = _kv_shape(Q, K, same_n=True)
    t = _vo_types(code)
    for name, x in (("Q", Q), ("O", O), ("dO", dO), ("dQ", dQ)):
        _need(name, x, (B, H, N, d), t)
    for name, x in (("K", K), ("V", V), ("dK", dK), ("dV", dV)):
        _need(name, x, (B, H_kv, N, d), t)
    _need("Z", Z, (B, H, N), _f32_types())
    _need("delta", delta, (2, B, H, N), _f32_types())
    _need("mult", mult, (B, N), _f32_types(), optional=True)
    _on_device(Q=Q, K=K, V=V, mult=mult, O=O, dO=dO, Z=Z, dQ=dQ, dK=dK, dV=dV, delta=delta)
    return B, H, N, d, H_kv


@functools.lru_cache(maxsize=1024)
def _bwd_workspace_bytes(device_index, B, H, H_kv, N, d, code):
    """Workspace of the library's choice of slices for the backward: a function of the shape and the GPU."""
    return load_library().sphattn_bwd_workspace_bytes(B, H, H_kv, N, d, code)


def _launch_bwd(lib, Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, d, code, stream, own_outputs):
    """sphattn_grn_bwd on checked arguments, cut into slices under the conditions of _launch_cross (up to
    256 MiB of partial sums for dQ and as much for dK and dV)."""
    args = (Q.data_ptr(), K.data_ptr(), V.data_ptr(), _ptr(mult), O.data_ptr(), dO.data_ptr(), Z.data_ptr(),
            dQ.data_ptr(), dK.data_ptr(), dV.data_ptr(), delta.data_ptr(), B, H, H_kv, N, d, code)
    need = _bwd_workspace_bytes(Q.device.index, B, H, H_kv, N, d, code) if own_outputs and stream is None else 0
    ws = _workspace(need, Q)
    if ws is None:
        _raise_on(lib.sphattn_grn_bwd(*args, _stream_of(Q, stream)))
    else:
        _raise_on(lib.sphattn_grn_bwd_split(*args, ws.data_ptr(), need, _stream_of(Q, None)))


def sphattn_grn_bwd(Q, K, V, mult, O, dO, Z, dQ=None, dK=None, dV=None, delta=None, dtype="bf16", stream=None):
    """Gradients (dQ, dK, dV) of sum(O * dO) for O = sphattn_grn_fwd(Q, K, V, mult): per-gene
    multiplicities mult[B,N] (or None) and K, V of shape [B,H_kv,N,d]."""
    import torch
    lib, code = load_library(), _dtype_code(dtype)
    own_outputs = dQ is None and dK is None and dV is None and delta is None
    if own_outputs and stream is None:
        done = _fast.backward(Q, K, V, mult, O, dO, Z, code, False)
        if done is not None:
            return done
    dQ = torch.empty_like(Q) if dQ is None else dQ
    dK = torch.empty_like(K) if dK is None else dK
    dV = torch.empty_like(V) if dV is None else dV
    if delta is None:
        delta = torch.empty((2, *Q.shape[:3]), dtype=torch.float32, device=Q.device)
    B, H, N, d, H_kv = _check_backward(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, code)
    _launch_bwd(lib, Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, d, code, stream, own_outputs)
    return dQ, dK, dV


def sphattn_bwd(Q, K, V, O, dO, Z, dQ=None, dK=None, dV=None, delta=None, dtype="bf16", stream=None):
    """Gradients (dQ, dK, dV) of sum(O * dO) for O, Z = sphattn_fwd_z(Q, K, V); 16-bit storage."""
    import torch
    lib, code = load_library(), _dtype_code(dtype)
    own_outputs = dQ is None and dK is None and dV is None and delta is None
    if own_outputs and stream is None:
        done = _fast.backward(Q, K, V, None, O, dO, Z, code, True)
        if done is not None:
            return done
    dQ = torch.empty_like(Q) if dQ is None else dQ
    dK = torch.empty_like(K) if dK is None else dK
    dV = torch.empty_like(V) if dV is None else dV
    if delta is None:
        delta = torch.empty((2, *Q.shape[:3]), dtype=torch.float32, device=Q.device)
    if Q.dim() == 4 and K.dim() == 4 and K.shape[1] != Q.shape[1]:
        raise ValueError(f"K must have Q's {Q.shape[1]} heads, got {K.shape[1]} (sphattn_grn_bwd takes shared heads)")
    B, H, N, d, H_kv = _check_backward(Q, K, V, None, O, dO, Z, dQ, dK, dV, delta, code)
    _launch_bwd(lib, Q, K, V, None, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, d, code, stream, own_outputs)
    return dQ, dK, dV
