"""fp32 storage: three-part bf16 products (sphattn_f32.hpp) in 128- and 256-row workgroups, and the fp32
instruction in 16- and 32-row ones, on shapes that choose each: ragged queries and keys, multiplicities, shared heads, accumulators.  The bound is
that of fp32 arithmetic itself, not the 1e-4 of the entry point: relative 2-norm error against 64 bits
at most 3e-8 sqrt(N_k) / 4 + 2e-7, which the fp32 matrix instruction measures at (2.1e-7 at 256 keys,
6.1e-7 at 4096) and which one missing low part (2^-17) or a rounded score would exceed tenfold."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _reference(q, k, v, mult):
    B, H, _, _ = q.shape
    G = H // k.shape[1]
    o = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
    z = torch.zeros(q.shape[:3], dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(H):
            K, V = k[b, h // G].double(), v[b, h // G].double()
            if mult is not None:
                K = K * mult[b].double()[:, None]
            S = q[b, h].double() @ K.t().contiguous()
            o[b, h], z[b, h] = S @ V, (S * S).sum(-1)
    return o, z


# B, H, H_kv, N_q, N_k, d, multiplicities, scale of Q and of V
CASES = [(1, 9, 9, 4000, 33, 128, False, 1.0, 1.0), (1, 17, 17, 4097, 97, 128, True, 1.0, 1.0),
         (1, 12, 4, 3001, 700, 64, True, 1.0, 1.0), (2, 16, 16, 2100, 1025, 64, False, 1.0, 1.0),
         (1, 8, 8, 2049, 1, 128, False, 1.0, 1.0), (1, 8, 8, 4096, 4100, 128, False, 1e15, 1e-20),
         (1, 16, 16, 4096, 640, 128, False, 1e-12, 1e30),
         # 16 rows: one tile, fewer tiles than waves, several per wave; 32 rows: between 4096 and 8192 rows
         (1, 1, 1, 1, 33, 64, False, 1.0, 1.0), (2, 4, 2, 100, 333, 64, True, 1.0, 1.0), (1, 3, 3, 257, 130, 128, True, 1.0, 1.0),
         (1, 2, 1, 17, 600, 128, False, 1.0, 1.0), (1, 5, 5, 1400, 70, 64, True, 1.0, 1.0), (1, 5, 5, 1399, 40, 128, False, 1.0, 1.0)]


@pytest.mark.parametrize("B,H,H_kv,Nq,Nk,d,with_mult,sq,sv", CASES)
def test_fp32_error_against_64_bits(pkg, B, H, H_kv, Nq, Nk, d, with_mult, sq, sv):
    print(f"case f32 B={B} H={H} H_kv={H_kv} Nq={Nq} Nk={Nk} d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(Nq + Nk)
    q = torch.randn((B, H, Nq, d), generator=g, device=DEV) * sq
    k, v = (torch.randn((B, H_kv, Nk, d), generator=g, device=DEV) for _ in range(2))
    v = v * sv
    mult = torch.poisson(torch.full((B, Nk), 1.5, device=DEV), generator=g) if with_mult else None
    if with_mult:
        mult[:, 0] = 2.0
    Z = torch.empty((B, H, Nq), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(q, k, v, mult, Z=Z, dtype="f32")
    op, zp = pkg.sphattn_partial_fwd(q, k, v, mult, dtype="f32")
    torch.cuda.synchronize()
    ref_o, ref_z = _reference(q, k, v, mult)
    nrm = ref_z.sqrt()[..., None]
    bound = 0.75e-8 * math.sqrt(Nk) + 2e-7
    if Nk == 1:
        nrm = torch.ones_like(nrm)               # a single score may nearly cancel: compare unnormalised

    def rel(a, b):
        return ((a - b).norm() / b.norm()).item()
    if Nk > 1:
        err = rel(O.double(), ref_o / nrm)
        print(f"  O rel {err:.2e} of {bound:.2e}", flush=True)
        assert err <= bound
    assert rel(op.double() / nrm, ref_o / nrm) <= bound
    assert rel(Z.double(), ref_z) <= 4 * bound and rel(zp.double(), ref_z) <= 4 * bound
