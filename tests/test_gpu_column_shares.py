"""Launches whose workgroups have 64 rows and a half or a quarter of the columns of V and O each (column_shares in sphattn_choice.hpp): ragged rows and
keys, odd numbers of tiles, shared K/V heads, as many workgroups as CUs, whole results and partial accumulators, cut key axes.
Compared with 64 bits within what the storage type allows, as in test_gpu_forward_forms.py."""
import pytest
import torch

import launch_choice
import synthetic_inputs as si

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}

# H, H_kv, N_q, N_k, d, shares
SHAPES = [(1, 1, 1, 1100, 128, 4), (2, 2, 64, 129, 128, 4), (5, 5, 300, 300, 128, 4), (4, 2, 63, 1025, 128, 4), (52, 52, 64, 1281, 128, 4),
          (4, 4, 1999, 1999, 128, 2), (64, 64, 64, 1281, 128, 2), (64, 64, 64, 700, 128, 4), (128, 128, 33, 1088, 128, 2), (1, 1, 70, 4161, 128, 2),
          (2, 2, 100, 385, 64, 2), (2, 1, 65, 1281, 64, 2), (128, 128, 64, 1400, 64, 2), (3, 3, 700, 2049, 64, 2)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("H,H_kv,Nq,Nk,d,shares", SHAPES)
def test_against_64_bits(pkg, H, H_kv, Nq, Nk, d, shares, dtype, counts):
    print(f"case column shares {H} on {H_kv}, {Nq} of {Nk} x {d} {dtype} counts={counts}", flush=True)
    assert {launch_choice.column_shares(H, H_kv, Nq, Nk, d, dtype, counts, partial) for partial in (False, True)} == {shares}
    q, _, _ = si.make_qkv(1, H, Nq, d, dtype, seed=8100 + Nq)
    _, k, v = si.make_qkv(1, H_kv, Nk, d, dtype, seed=8200 + Nk)
    m = torch.poisson(torch.full((1, Nk), 1.5), generator=torch.Generator(device="cpu").manual_seed(8300 + Nk)) if counts else None
    q, k, v = q.to(DEV), k.to(DEV), v.to(DEV)
    m = m.to(DEV) if counts else None
    guard = 64
    Z = torch.full((1, H, Nq), -1.0, device=DEV)
    flat = torch.full((H * Nq * d + guard,), 7.0, dtype=v.dtype, device=DEV)   # (what is not written shows)
    O = flat[:H * Nq * d].view(1, H, Nq, d)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype=dtype)
    o, z = pkg.sphattn_partial_fwd(q, k, v, m, dtype=dtype)
    cut = pkg.sphattn_cross_fwd(q, k, v, m, dtype=dtype)   # (where the library cuts it, else the same)
    torch.cuda.synchronize()
    assert (flat[H * Nq * d:] == 7.0).all()
    for h in sorted({0, H // 2, H - 1}):
        kh = k[0, h // (H // H_kv)].double()
        kh = kh * m[0].double()[:, None] if counts else kh
        V, Q, KT = v[0, h // (H // H_kv)].double(), q[0, h].double(), kh.t().contiguous()
        S = Q @ KT
        n = (S * S).sum(1, keepdim=True).sqrt()
        ref = S @ V / n
        slack = (S.abs() * U[dtype]) @ V.abs() / n + 1e-4 * ref.abs()
        for got in (O, cut):
            assert ((got[0, h].double() - ref).abs() <= slack + U[dtype] * ref.abs() + 1e-5).all(), h
        assert ((o[0, h].double() / n - ref).abs() <= slack + 1e-5).all(), h
        for got in (Z, z):
            assert ((got[0, h].double() - n[:, 0] ** 2).abs() <= 2e-4 * n[:, 0] ** 2 + 1e-7 * (n ** 2).max()).all(), h
