"""The backward with its streamed axes cut into slices (shapes that leave CUs idle): gradients against
the oracle element by element, with test_gpu_backward.py's bound (the slices' fp32 sums add nothing to
it: they are rounded to 16 bits once, like the uncut kernels' accumulators), and against the uncut
launch.  Shared K/V heads run as one block of rows in both."""
import ctypes

import numpy as np
import pytest
import torch

import synthetic_inputs as si

pytestmark = pytest.mark.gpu

INNER = {"bf16": 1.5e-2, "f16": 3e-3}
HALF_ULP = {"bf16": 2.0 ** -9, "f16": 2.0 ** -12}
DEV = "cuda:0"
P = ctypes.c_void_p

# B, H, H_kv, N, d, dtype, multiplicities: dQ cut, dK/dV cut, or both; ragged last tiles and last slices
CASES = [(1, 1, 1, 513, 64, "bf16", False), (1, 4, 2, 700, 128, "bf16", True), (2, 3, 1, 600, 64, "f16", True),
         (1, 6, 2, 1025, 64, "bf16", False), (1, 2, 2, 900, 128, "f16", True), (1, 8, 1, 257, 128, "bf16", False)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


@pytest.mark.parametrize("B,H,H_kv,N,d,dtype,with_mult", CASES)
def test_cut_backward_against_the_oracle(pkg, oracle, B, H, H_kv, N, d, dtype, with_mult):
    print(f"case bwd slices B={B} H={H} H_kv={H_kv} N={N} d={d} {dtype} mult={with_mult}", flush=True)
    lib, code = pkg.load_library(), pkg._dtype_code(dtype)
    need = lib.sphattn_bwd_workspace_bytes(B, H, H_kv, N, d, code)
    assert need > 0
    q, _, _ = si.make_qkv(B, H, N, d, dtype, seed=5000 + N)
    _, k, v = si.make_qkv(B, H_kv, N, d, dtype, seed=5100 + N)
    g = torch.Generator(device="cpu").manual_seed(5200 + N)
    dO = torch.randn((B, H, N, d), generator=g, dtype=torch.float32).to(q.dtype)
    mult = None
    if with_mult:
        mult = torch.poisson(torch.full((B, N), 1.5), generator=g).to(torch.float32)
        mult[:, 0] = 2.0
    qd, kd, vd, gd, md = (t.to(DEV) if t is not None else None for t in (q, k, v, dO, mult))
    Z = torch.empty((B, H, N), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(qd, kd, vd, md, Z=Z, dtype=dtype)
    got = pkg.sphattn_grn_bwd(qd, kd, vd, md, O, gd, Z, dtype=dtype)
    uncut = [torch.empty_like(t) for t in (qd, kd, vd)]
    delta = torch.empty((2, B, H, N), dtype=torch.float32, device=DEV)
    pkg.sphattn_grn_bwd(qd, kd, vd, md, O, gd, Z, *uncut, delta, dtype=dtype)
    # straight through the C entry, on a NaN-filled workspace with guard bytes behind it
    ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
    again = [torch.full_like(t, float("nan")) for t in (qd, kd, vd)]
    rc = lib.sphattn_grn_bwd_split(*(P(t.data_ptr()) if t is not None else P(0) for t in (qd, kd, vd, md, O, gd, Z, *again, delta)),
                                   B, H, H_kv, N, d, code, P(ws.data_ptr()), need, None)
    torch.cuda.synchronize()
    assert rc == 0 and bool((ws[need:] == 0xFF).all())
    bits = [si.storage_bits(t)[0] for t in (q, k, v, dO)]
    kind = si.storage_bits(q)[1]
    ref = oracle.grn_attention_bwd(*bits, mult.numpy() if with_mult else None, kinds=(kind,) * 4)
    row_scale = 1.0 / np.maximum(mult.numpy(), 1.0)[:, None, :, None] if with_mult else 1.0
    for name, a, a2, u, b in zip(("dQ", "dK", "dV"), got, again, uncut, ref):
        assert torch.equal(a, a2), name              # the same launch: no atomics, a fixed order
        for x in (a, u):
            x = x.cpu().double().numpy()
            assert np.all(np.isfinite(x)), name
            y = b
            if name != "dQ":
                x, y = x * row_scale, y * row_scale
            rms = np.sqrt((y ** 2).mean())
            err = np.abs(x - y).max() / rms
            assert err <= HALF_ULP[dtype] * np.abs(y).max() / rms + INNER[dtype], (name, err)


def test_full_launches_are_not_cut(pkg):
    lib = pkg.load_library()
    assert lib.sphattn_bwd_workspace_bytes(2, 16, 16, 8192, 128, 1) == 0
    assert lib.sphattn_bwd_workspace_bytes(1, 1, 1, 200, 64, 1) == 0      # nothing to cut: 4 tiles
