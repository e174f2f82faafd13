"""The d = 64 forward with 512 rows in eight waves (rows512_pay in sphattn_choice.hpp): one round and several (every other batch of which
streams the keys backwards), ragged last rows and keys, one key tile, shared K/V heads, whole results and partial
accumulators.  Without counts and in one round the sums are those of the 256-row workgroups bit for bit; everything is compared with 64 bits
within what the storage type allows, as in test_gpu_forward_forms.py."""
import pytest
import torch

import launch_choice
import synthetic_inputs as si

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "fp8qk_bf16v": 2.0 ** -8}

# H, H_kv, N_q, N_k
ALL = [(100, 100, 700, 700), (120, 120, 513, 577), (70, 35, 1537, 641), (250, 250, 300, 640), (60, 60, 1500, 705), (256, 256, 1000, 1100), (64, 32, 4000, 1281), (100, 20, 700, 8129), (100, 100, 513, 193)]
NO_COUNTS = [(120, 120, 513, 130), (250, 250, 300, 192), (60, 60, 1500, 129), (100, 100, 513, 60)]   # the shortest key axes
LONG = [(64, 32, 4000, 8257)]                                                    # 16-bit storage without counts, past 128 key tiles
CASES = [(s, t, c) for t, c in (("bf16", False), ("bf16", True), ("f16", False), ("f16", True), ("fp8qk_bf16v", False))
         for s in ALL + (NO_COUNTS if not c else []) + (LONG if not c and t != "fp8qk_bf16v" else [])]


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


@pytest.mark.parametrize("shape,dtype,counts", CASES)
def test_against_64_bits(pkg, shape, dtype, counts):
    H, H_kv, Nq, Nk = shape
    print(f"case rows512 {H} on {H_kv}, {Nq} of {Nk} {dtype} counts={counts}", flush=True)
    assert launch_choice.rows512(H, H_kv, Nq, Nk, dtype, counts) and launch_choice.rows512(H, H_kv, Nq, Nk, dtype, counts, whole=False)
    d = 64
    q, _, _ = si.make_qkv(1, H, Nq, d, dtype, seed=7100 + Nq)
    _, k, v = si.make_qkv(1, H_kv, Nk, d, dtype, seed=7200 + Nk)
    m = torch.poisson(torch.full((1, Nk), 1.5), generator=torch.Generator(device="cpu").manual_seed(7300 + Nk)) if counts else None
    q, k, v = q.to(DEV), k.to(DEV), v.to(DEV)
    m = m.to(DEV) if counts else None
    O, Z = torch.empty((1, H, Nq, d), dtype=v.dtype, device=DEV), torch.empty((1, H, Nq), dtype=torch.float32, device=DEV)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype=dtype)
    o, z = pkg.sphattn_partial_fwd(q, k, v, m, dtype=dtype)
    torch.cuda.synchronize()
    if not counts and Nq == Nk and H_kv * -(-Nq // 512) <= launch_choice.CUS:
        O256, Z256 = pkg.sphattn_fwd_tile_rows(q, k, v, Z=torch.empty_like(Z), dtype=dtype, tile_rows=256)
        assert torch.equal(O, O256) and torch.equal(Z, Z256)
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
