"""The all-E4M3 forward's workgroup shapes (choose_fp8 in sphattn_choice.hpp).  test_gpu_fp8.py holds the calls of few rows, which
take 64 rows, against the oracle; here calls of many heads take each of the other shapes, and some of their heads
are called alone.  A row's scores, their rounding and its sums do not depend on the workgroup it is in, so the results are equal bit for
bit; where the launch has several rounds, of which every other streams the keys backwards, the order of the fp32 sums differs, and an
element may round to the neighbouring bf16."""
import pytest
import torch

import launch_choice

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# H, H_kv, N, d, counts, (query blocks per wave, waves), key stream reversed somewhere
CASES = [(64, 64, 300, 128, False, (1, 8), False), (64, 16, 257, 128, True, (1, 8), False), (100, 100, 129, 64, True, (1, 8), False), (130, 130, 65, 64, False, (1, 8), False),
         (100, 50, 290, 128, False, (2, 8), False), (250, 250, 140, 128, True, (2, 8), False), (100, 100, 300, 64, False, (2, 8), False), (100, 25, 511, 64, True, (2, 8), False),
         (300, 300, 130, 128, True, (2, 8), True), (250, 50, 400, 64, False, (4, 4), False), (260, 260, 300, 64, False, (2, 4), True), (270, 90, 260, 64, True, (2, 4), True)]


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _call(pkg, q, k, v, m):
    B, H_kv, N, d = k.shape
    ws = torch.empty(pkg.sphattn_fp8_workspace_bytes(B, H_kv, N, d), dtype=torch.uint8, device=DEV)
    return pkg.sphattn_fp8_grn_fwd(q, k, v, m, ws)


@pytest.mark.parametrize("H,H_kv,N,d,counts,shape,reversed_keys", CASES)
def test_heads_of_a_launch_equal_heads_alone(pkg, H, H_kv, N, d, counts, shape, reversed_keys):
    print(f"case fp8 shapes {H} on {H_kv} of {N} x {d} counts={counts} {shape}", flush=True)
    assert launch_choice.fp8_shape(H, N, d, counts) == shape
    g = torch.Generator(device="cpu").manual_seed(900 + H + N)
    q, k, v = ((torch.randn((1, h, N, d), generator=g) * 100).clamp(-448, 448).to(torch.float8_e4m3fn).to(DEV) for h in (H, H_kv, H_kv))
    m = torch.poisson(torch.full((1, N), 1.5), generator=g).to(DEV) if counts else None
    whole = _call(pkg, q, k, v, m)
    group = H // H_kv
    for kv in sorted({0, 1, H_kv // 2, H_kv - 1}):
        heads = slice(kv * group, (kv + 1) * group)
        alone = _call(pkg, *(x[:, s].contiguous() for x, s in ((q, heads), (k, slice(kv, kv + 1)), (v, slice(kv, kv + 1)))), m)
        assert launch_choice.fp8_shape(group, N, d, counts) == (1, 4)
        if not reversed_keys:
            assert torch.equal(whole[:, heads], alone), kv
        else:                                      # 2^-8 of the element, and 2 N 2^-24 of the sum of magnitudes (sqrt(N) sigma at most)
            err = (whole[:, heads].double() - alone.double()).abs()
            bound = 2.0 ** -7 * alone.double().abs() + 2 * N * 2.0 ** -24 * N ** 0.5 * v.float().abs().max().item()
            assert (err <= bound).all(), (kv, err.max().item())
