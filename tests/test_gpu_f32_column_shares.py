"""The smallest fp32 launches, whose 16-row workgroups share the columns of V (f32_small_column_shares in sphattn_choice.hpp): four, two and
one to a row tile give the same bits, and what 64 bits give within 2^-23 of the sums of magnitudes (24 bits a value and a product, sums in
any order at random signs)."""
import pytest
import torch

import launch_choice

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _call(pkg, q, k, v, m):
    O, Z = torch.full_like(q, 7.0), torch.full(q.shape[:3], 7.0, device=DEV)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype="f32")
    return (O, Z, *pkg.sphattn_partial_fwd(q, k, v, m, dtype="f32"))


@pytest.mark.parametrize("counts", [False, True])
@pytest.mark.parametrize("Nq,Nk", [(250, 33), (256, 1), (241, 300), (256, 256)])
@pytest.mark.parametrize("d", [64, 128])
def test_shares_of_the_columns(pkg, d, Nq, Nk, counts):
    print(f"case f32 shares {Nq} of {Nk} x {d} counts={counts}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(9100 + Nq + Nk + d)
    q, k, v = (torch.randn((1, 10, n, d), generator=g, device=DEV) for n in (Nq, Nk, Nk))
    m = torch.rand((1, Nk), generator=g, device=DEV) + 0.5 if counts else None
    assert [launch_choice.f32_shares(h, Nq) for h in (1, 4, 6, 8, 10)] == [4, 4, 2, 2, 1] and launch_choice.f32_rows(10, Nq, Nk, d)[0] == 16
    whole = _call(pkg, q, k, v, m)
    for h in (1, 4, 6, 8):
        for a, b in zip(whole, _call(pkg, *(x[:, :h].contiguous() for x in (q, k, v)), m)):
            assert torch.equal(a[:, :h], b), h
    kd = k[0].double() * (m[0].double()[:, None] if counts else 1.0)
    S = q[0].double() @ kd.transpose(1, 2).contiguous()
    A = q[0].double().abs() @ kd.abs().transpose(1, 2).contiguous()
    n = S.norm(dim=2, keepdim=True)
    ref = S @ v[0].double() / n
    bound = 2.0 ** -23 * (4 * A @ v[0].double().abs() / n + 4 * ref.abs() * (A / n).norm(dim=2, keepdim=True) + 4 * ref.abs())
    assert ((whole[0][0].double() - ref).abs() <= bound).all() and ((whole[2][0].double() / n - ref).abs() <= bound).all()
    for z in (whole[1], whole[3]):
        assert ((z[0].double() - n[..., 0] ** 2).abs() <= 2.0 ** -21 * (S.abs() * A).sum(2)).all()
