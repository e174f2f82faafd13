"""Groups of query heads too large to be launched as one block of rows: the heads that share a K/V head are
packed into one only while the block stays below 2^31 bytes at 4 bytes an element (4.2 million rows of 128),
and beyond that the kernels find the K/V head of every query head, and the backward's dK/dV kernel walks
the heads of a group (its slices starting in the middle of a group), themselves.  Everything else
that shares K/V heads in these tests runs packed.  Against 64 bits on the GPU, tolerances as in
test_gpu_parity.py and test_gpu_backward.py, accumulators within their rounding bound."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL_O = {"bf16": 2e-2, "fp8qk_bf16v": 6e-2, "f16": 5e-3, "f32": 1e-4}
TORCH = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
INNER, HALF_ULP = 1.5e-2, 2.0 ** -9


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _randn(shape, dtype, g):
    x = torch.randn(shape, generator=g, device=DEV)
    return x.clamp(-448, 448).to(torch.float8_e4m3fn) if dtype == "fp8" else x.to(TORCH[dtype])


def _counts(Nk, g):
    m = torch.poisson(torch.full((1, Nk), 1.5, device=DEV), generator=g)
    m[:, 0] = 2.0
    return m


# query heads per K/V head, N_q, N_k, d, dtype, multiplicities, accumulators only.  4417 x 2 heads of 8 tiles leave
# 16 tiles behind full rounds of 512: the half-tile launch
@pytest.mark.parametrize("G,Nq,Nk,d,dtype,with_mult,partial", [
    (2100, 2000, 130, 128, "bf16", False, False), (4417, 1900, 65, 64, "f16", False, False),
    (2100, 2000, 200, 128, "fp8qk_bf16v", True, False), (2100, 2000, 70, 128, "f32", True, False),
    (4417, 1900, 100, 64, "bf16", True, True)])
def test_forward(pkg, G, Nq, Nk, d, dtype, with_mult, partial):
    print(f"case unpacked forward G={G} Nq={Nq} Nk={Nk} d={d} {dtype} mult={with_mult} partial={partial}", flush=True)
    assert G * Nq * d * 4 > 0x7fffffff
    H = 2 * G
    g = torch.Generator(device=DEV).manual_seed(G + Nk)
    qk, vt = ("fp8", "bf16") if dtype == "fp8qk_bf16v" else (dtype, dtype)
    q = torch.cat([_randn((1, G, Nq, d), qk, g) for _ in range(2)], dim=1)
    k, v = _randn((1, 2, Nk, d), qk, g), _randn((1, 2, Nk, d), vt, g)
    mult = _counts(Nk, g) if with_mult else None
    if partial:
        got, _ = pkg.sphattn_partial_fwd(q, k, v, mult, dtype=dtype)
    else:
        got = pkg.sphattn_cross_fwd(q, k, v, mult, dtype=dtype)
    torch.cuda.synchronize()
    heads = {0, 1, G // 2, G - 1, G, G + 1, H - 1} | {H * x // 8 + e for x in range(1, 8) for e in (-2, -1, 0, 1)}
    for h in sorted(heads):
        K, V = k[0, h // G].double(), v[0, h // G].double()
        if with_mult:
            K = K * mult[0].double()[:, None]
        S = q[0, h].double() @ K.t().contiguous()
        norm = S.norm(dim=1, keepdim=True)
        ref = S @ V / norm
        if partial:
            # every element: each score is rounded to bf16 (2^-8 of it at most) before its product with V; fp32 sums beside that
            bound = 2.0 ** -8 * (S.abs() @ V.abs()) + 1e-5 * norm
            excess = ((got[0, h].double() - S @ V).abs() - bound).max().item()
            assert excess <= 0.0, (h, excess)
        else:
            err = ((got[0, h].double() - ref).abs().max() / ref.square().mean().sqrt()).item()
            assert err <= TOL_O[dtype], (h, err)


def test_backward_uncut_and_cut(pkg):
    G, N, d, H_kv = 7000, 600, 128, 2
    H = G * H_kv
    print(f"case unpacked backward G={G} N={N} d={d}", flush=True)
    assert G * N * d * 4 > 0x7fffffff
    need = pkg.load_library().sphattn_bwd_workspace_bytes(1, H, H_kv, N, d, pkg._dtype_code("bf16"))
    part = 2 * H_kv * N * d * 4                    # dK and dV of one slice; dQ has tiles enough and is not cut
    slices = need // part
    per = -(-(G * 10) // slices)                   # 10 query tiles to a head
    assert slices > 1 and need < part * 100 and any(s * per % 10 for s in range(slices))
    g = torch.Generator(device=DEV).manual_seed(11)
    q, dO = (torch.cat([_randn((1, G, N, d), "bf16", g) for _ in range(H_kv)], dim=1) for _ in range(2))
    k, v = _randn((1, H_kv, N, d), "bf16", g), _randn((1, H_kv, N, d), "bf16", g)
    mult = _counts(N, g)
    Z = torch.empty((1, H, N), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(q, k, v, mult, Z=Z, dtype="bf16")
    cut = pkg.sphattn_grn_bwd(q, k, v, mult, O, dO, Z, dtype="bf16")
    uncut = [torch.empty_like(t) for t in (q, k, v)]
    pkg.sphattn_grn_bwd(q, k, v, mult, O, dO, Z, *uncut, torch.empty((2, 1, H, N), dtype=torch.float32, device=DEV), dtype="bf16")
    torch.cuda.synchronize()
    assert torch.equal(cut[0], uncut[0])
    m, rows = mult[0].double()[:, None], 50 * N
    scale = 1.0 / m.clamp_min(1.0)                 # rows of dK and dV and their errors scale with the multiplicity
    for hk in range(H_kv):
        K, V = k[0, hk].double() * m, v[0, hk].double()
        Kt, Vt = K.t().contiguous(), V.t().contiguous()
        Q, D, dQ = (t[0, hk * G:(hk + 1) * G].reshape(G * N, d) for t in (q, dO, cut[0]))
        dK, dV = torch.zeros_like(K), torch.zeros_like(V)
        worst = biggest = square = 0.0
        for i in range(0, G * N, rows):
            Qi, Di = Q[i:i + rows].double(), D[i:i + rows].double()
            S = Qi @ Kt
            r = S.square().sum(1, keepdim=True).rsqrt()
            W = S * r
            dS = r * (Di @ Vt) - (Di * (W @ V)).sum(1, keepdim=True) * r * W
            ref = dS @ K
            dK += m * (dS.t().contiguous() @ Qi)
            dV += W.t().contiguous() @ Di
            worst = max(worst, (dQ[i:i + rows].double() - ref).abs().max().item())
            biggest, square = max(biggest, ref.abs().max().item()), square + ref.square().sum().item()
        rms = np.sqrt(square / (G * N * d))
        assert worst / rms <= HALF_ULP * biggest / rms + INNER, ("dQ", worst / rms)
        for name, ref, got in (("dK", dK, (cut[1], uncut[1])), ("dV", dV, (cut[2], uncut[2]))):
            for x in got:
                a, b = x[0, hk].double() * scale, ref * scale
                rms = b.square().mean().sqrt()
                err = ((a - b).abs().max() / rms).item()
                assert err <= (HALF_ULP * b.abs().max() / rms).item() + INNER, (name, err)
