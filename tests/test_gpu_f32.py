"""fp32 storage: three-part bf16 products (sphattn_f32.hpp; from 512 keys, d = 64 1792, on two-part fp16 ones) in 128- and 256-row workgroups, and the fp32
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


# Values that have no three bf16 parts: below 2^-100 (1e-36 is 2^-119.6), scores among them, and those that round to
# infinity in bf16.  Shapes of the 128- and the 256-row kernel, d = 64 and 128; N_q, N_k, d, heads, multiplicities.
WIDE = [(2049, 97, 128, 8, False), (4097, 70, 128, 17, True), (3001, 130, 64, 12, True), (2100, 333, 64, 32, False)]
KINDS = ["v_small", "v_smaller", "q_small_k_large", "one_value_small", "one_score_small", "one_value_largest", "q_row_small"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Nq,Nk,d,H,with_mult", WIDE)
def test_fp32_outside_the_range_of_three_parts(pkg, Nq, Nk, d, H, with_mult, kind):
    """The bound of test_fp32_error_against_64_bits over the whole output and, for the column that
    only the one odd value reaches, over that column; the accumulators likewise."""
    print(f"case f32 range {kind} Nq={Nq} Nk={Nk} d={d} H={H}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(Nq + Nk)
    q = torch.randn((1, H, Nq, d), generator=g, device=DEV)
    k, v = (torch.randn((1, H, Nk, d), generator=g, device=DEV) for _ in range(2))
    mult = torch.poisson(torch.full((1, Nk), 1.5, device=DEV), generator=g) + 1.0 if with_mult else None
    odd = Nk - 3                                   # a key of the last tile: seen after the others
    column = slice(None)
    if kind == "v_small":
        v = v * 1e-36
    elif kind == "v_smaller":
        v = v * 1e-37
    elif kind == "q_small_k_large":
        q, k = q * 1e-36, k * 1e36
    elif kind == "q_row_small":
        q[:, :, 5] *= 1e-35
        k = k * 1e16
    else:
        column = slice(7, 8)
        v[..., 7] = 0.0
        if kind == "one_value_small":
            v[:, :, odd, 7] = 1.2345e-36
        elif kind == "one_score_small":
            k[:, :, odd] *= 1e-34
            v[:, :, odd, 7] = 1.2345e30
        else:
            q = q * 1e-4
            v[:, :, odd, 7] = 3.4e38
    Z = torch.empty((1, H, Nq), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(q, k, v, mult, Z=Z, dtype="f32")
    op, zp = pkg.sphattn_partial_fwd(q, k, v, mult, dtype="f32")
    torch.cuda.synchronize()
    ref_o, ref_z = _reference(q, k, v, mult)
    nrm = ref_z.sqrt()[..., None]
    bound = 0.75e-8 * math.sqrt(Nk) + 2e-7

    def rel(a, b):                                 # scaled first, for the squares
        a, b = a[..., column] / b[..., column].abs().max(), b[..., column] / b[..., column].abs().max()
        return ((a - b).norm() / b.norm()).item()
    for name, got in (("O", O.double()), ("o / sqrt(z)", op.double() / nrm)):
        err = rel(got, ref_o / nrm)
        print(f"  {name} rel {err:.2e} of {bound:.2e}", flush=True)
        assert err <= bound, name
    column = slice(None)
    assert rel(Z.double(), ref_z) <= 4 * bound and rel(zp.double(), ref_z) <= 4 * bound


def test_fp32_infinite_value_stays_in_its_column(pkg):
    """An infinity in V gives an infinity of its score's sign in that column and nothing elsewhere."""
    g = torch.Generator(device=DEV).manual_seed(3)
    q = torch.randn((1, 8, 2049, 128), generator=g, device=DEV)
    k, v = (torch.randn((1, 8, 97, 128), generator=g, device=DEV) for _ in range(2))
    print("case f32 infinite value", flush=True)
    ref = pkg.sphattn_cross_fwd(q, k, v, dtype="f32")
    v[:, :, 40, 7] = math.inf
    O = pkg.sphattn_cross_fwd(q, k, v, dtype="f32")
    torch.cuda.synchronize()
    s = q.double() @ k[:, :, 40].double()[..., None]
    assert torch.equal(O[..., 7].double(), torch.copysign(torch.full_like(s[..., 0], math.inf), s[..., 0]))
    others = torch.arange(128, device=DEV) != 7
    # the other columns: two fp32 results of the same sums, each within the bound above
    assert ((O - ref)[..., others].double().norm() / ref[..., others].double().norm()).item() <= 2 * (0.75e-8 * math.sqrt(97) + 2e-7)


def test_fp32_product_is_good_to_a_rounding(pkg):
    """Rows with one element each against one key of as many: every score is a single product.  The partial
    products left out come to 2^-24 of it, the sum of the others to one rounding (2^-24, or 2^-23 if the
    matrix core cuts instead); o = s v with v = 1 is exact."""
    H, N, d = 64, 4096, 64
    g = torch.Generator(device=DEV).manual_seed(4)
    q, k = torch.zeros((1, H, N, d), device=DEV), torch.zeros((1, H, 1, d), device=DEV)
    q[..., 3] = 1.0 + torch.rand((1, H, N), generator=g, device=DEV)
    k[..., 3] = 1.0 + torch.rand((1, H, 1), generator=g, device=DEV)
    print("case f32 single products", flush=True)
    o, z = pkg.sphattn_partial_fwd(q, k, torch.ones_like(k), dtype="f32")
    torch.cuda.synchronize()
    exact = q[..., 3].double() * k[..., 3].double()
    err = ((o[..., 0].double() - exact) / exact).abs().max().item()
    print(f"  largest error {err:.2e}", flush=True)
    assert err <= 3 * 2.0 ** -24


def test_fp32_longest_key_axis(pkg):
    """4 194 303 keys of 128, the most that a head's 2^31 - 1 bytes hold: the byte offsets of the last tiles are
    the largest there are.  Sampled rows against 64 bits (32 keys left out would show as 2.8e-3)."""
    Nq, Nk, d = 16384, 0x7fffffff // 512, 128
    print(f"case f32 longest Nq={Nq} Nk={Nk} d={d}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn((1, 1, Nq, d), generator=g, device=DEV)
    k, v = (torch.randn((1, 1, Nk, d), generator=g, device=DEV) for _ in range(2))
    op, zp = pkg.sphattn_partial_fwd(q, k, v, dtype="f32")
    torch.cuda.synchronize()
    rows = torch.tensor([0, 1, 777, 8191, 16383], device=DEV)
    o, z = torch.zeros((5, d), dtype=torch.float64, device=DEV), torch.zeros(5, dtype=torch.float64, device=DEV)
    for i in range(0, Nk, 1 << 19):
        S = q[0, 0, rows].double() @ k[0, 0, i:i + (1 << 19)].double().t().contiguous()
        o += S @ v[0, 0, i:i + (1 << 19)].double()
        z += (S * S).sum(-1)
    # z: a lane adds the squares of Nk / 8 keys one after the other, half a rounding of the running sum each on the
    # average over its growth at worst (they have one sign, so nothing averages out as it does in o)
    bound, bound_z = 0.75e-8 * math.sqrt(Nk) + 2e-7, Nk / 8 * 2.0 ** -25
    err_o = ((op[0, 0, rows].double() - o).norm() / o.norm()).item()
    err_z = ((zp[0, 0, rows].double() - z).norm() / z.norm()).item()
    print(f"  o rel {err_o:.2e} of {bound:.2e}, z rel {err_z:.2e} of {bound_z:.2e}", flush=True)
    assert err_o <= bound and err_z <= bound_z
