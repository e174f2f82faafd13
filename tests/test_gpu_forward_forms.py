"""Launches that take the key-split kernel's forms of four key groups, of one row group and of 256 rows (choose_form in
sphattn_choice.hpp), at the sizes where they can go wrong: a single step of 128 keys and parts of one, odd numbers of
tiles, ragged last rows, as many workgroups as CUs, whole results and partial accumulators, with and without counts.
Every element is compared with 64 bits within what the storage type allows: one rounding of every score and of the
result (u of them at most), 2e-4 of z, and for E4M3 scores the matrix instruction's own error, 2^-16 of the sum of the
products' magnitudes."""
import pytest
import torch

import synthetic_inputs as si

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "fp8qk_bf16v": 2.0 ** -8}

# H, H_kv, N_q, N_k, d
# (what each takes depends on storage and counts as well; test_launch_choice.py holds that every form of every storage is among them)
SHAPES = [(2, 2, 64, 641, 64), (3, 3, 130, 575, 64), (4, 2, 200, 1025, 64), (256, 256, 33, 700, 64),   # 64 rows, two and four key groups
          (2, 2, 63, 900, 128), (4, 1, 65, 1153, 128), (250, 250, 64, 1600, 128),
          (1, 1, 70, 150, 128), (2, 2, 64, 257, 128), (50, 50, 300, 4600, 128), (128, 64, 17, 4097, 128),   # the same, and one row group
          (20, 20, 999, 1300, 64), (6, 3, 3000, 1281, 64),                                             # 128 rows, four key groups with counts
          (64, 64, 290, 1985, 64), (64, 64, 289, 310, 64), (16, 8, 2000, 1990, 128), (64, 64, 290, 61, 128),   # four without, and two
          (64, 64, 290, 61, 64), (1, 1, 33, 60, 64), (1, 1, 33, 61, 128),                              # two workgroups on a CU; a single tile
          (100, 100, 400, 1000, 64), (64, 64, 1024, 449, 64), (12, 3, 5003, 129, 64),                  # 256 rows, two key groups
          (1, 1, 33, 150, 64), (6, 6, 1900, 1217, 128), (8, 4, 1985, 961, 128), (4, 4, 2000, 4600, 128)]   # 64 rows that do not share their columns


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "fp8qk_bf16v"])
@pytest.mark.parametrize("H,H_kv,Nq,Nk,d", SHAPES)
def test_every_form_against_64_bits(pkg, H, H_kv, Nq, Nk, d, dtype, counts):
    print(f"case forms {H} on {H_kv}, {Nq} of {Nk} x {d} {dtype} counts={counts}", flush=True)
    q, _, _ = si.make_qkv(1, H, Nq, d, dtype, seed=5100 + Nq)
    _, k, v = si.make_qkv(1, H_kv, Nk, d, dtype, seed=5200 + Nk)
    g = torch.Generator(device="cpu").manual_seed(5300 + Nk)
    m = torch.poisson(torch.full((1, Nk), 1.5), generator=g) if counts else None
    q, k, v = q.to(DEV), k.to(DEV), v.to(DEV)
    m = m.to(DEV) if counts else None
    Z = torch.empty((1, H, Nq), dtype=torch.float32, device=DEV)
    O = torch.empty((1, H, Nq, d), dtype=v.dtype, device=DEV)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype=dtype)
    o, z = pkg.sphattn_partial_fwd(q, k, v, m, dtype=dtype)
    torch.cuda.synchronize()
    for h in sorted({0, H // 2, H - 1}):
        kh = k[0, h // (H // H_kv)].double()
        kh = kh * m[0].double()[:, None] if counts else kh
        V, Q, KT = v[0, h // (H // H_kv)].double(), q[0, h].double(), kh.t().contiguous()
        S = Q @ KT
        n = (S * S).sum(1, keepdim=True).sqrt()
        ref = S @ V / n
        slack = S.abs() * U[dtype]
        if dtype == "fp8qk_bf16v":
            slack = slack + 2.0 ** -16 * (Q.abs() @ KT.abs())
        slack = slack @ V.abs() / n + 1e-4 * ref.abs()
        assert ((O[0, h].double() - ref).abs() <= slack + U[dtype] * ref.abs() + 1e-5).all(), h
        assert ((o[0, h].double() / n - ref).abs() <= slack + 1e-5).all(), h
        for got in (Z, z):
            assert ((got[0, h].double() - n[:, 0] ** 2).abs() <= 2e-4 * n[:, 0] ** 2 + 1e-7 * (n ** 2).max()).all(), h
