"""The 128- and 64-row forward kernel whose two wave pairs share out every key tile (sphattn_keysplit.hpp):
odd and even tile counts, ragged last tiles, tiles past the end, rows past the last query; every
storage type, multiplicities, row aggregates and partial accumulators, element by element against
the oracle.  Tolerances are those of test_gpu_parity.py and test_gpu_partial_splitkv.py."""
import numpy as np
import pytest
import torch

import synthetic_inputs as si

pytestmark = pytest.mark.gpu

TOL_O = {"bf16": 2e-2, "fp8qk_bf16v": 6e-2, "f16": 5e-3}
TOL_PART = {"bf16": 1e-2, "fp8qk_bf16v": 1e-2, "f16": 2e-3}
DEV = "cuda:0"


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _rel_err(got, ref):
    return np.abs(got - ref).max() / np.sqrt((ref ** 2).mean())


def _bits(*ts):
    pairs = [si.storage_bits(t) for t in ts]
    return [p[0] for p in pairs], tuple(p[1] for p in pairs)


SHAPES = [(n, d, t) for t in ("f16", "fp8qk_bf16v") for d in (64, 128) for n in (1, 31, 64, 65, 129, 257, 383)] + \
         [(1025, 128, "bf16"), (449, 128, "bf16"), (513, 64, "bf16"), (100, 64, "bf16")]


@pytest.mark.parametrize("tile_rows", [0, 128])
@pytest.mark.parametrize("N,d,dtype", SHAPES)
def test_both_widths_against_the_oracle(pkg, oracle, N, d, dtype, tile_rows):
    """tile_rows 0: launches this small take 64 rows per workgroup (fp8 Q/K at d = 128: 128)."""
    print(f"case keysplit N={N} d={d} {dtype} tile_rows={tile_rows}", flush=True)
    q, k, v = si.make_qkv(1, 2, N, d, dtype, seed=4000 + N + d)
    Z = torch.empty((1, 2, N), dtype=torch.float32, device=DEV)
    O, _ = pkg.sphattn_fwd_tile_rows(q.to(DEV), k.to(DEV), v.to(DEV), Z=Z, dtype=dtype, tile_rows=tile_rows)
    torch.cuda.synchronize()
    bits, kinds = _bits(q, k, v)
    ref, _, ref_z = oracle.spherical_attention_full(*bits, kinds=kinds)
    got = O.cpu().double().numpy()
    assert np.all(np.isfinite(got))
    assert _rel_err(got, ref) <= TOL_O[dtype]
    if dtype == "fp8qk_bf16v":
        # the fp8 matrix instruction sums its 128 products with fewer bits than fp32 (a score may be
        # off by about 2^-16 of the sum of its products' magnitudes, far more than 1e-4 of itself
        # where they cancel, and a row of one key does not average that out): the same scores as the
        # 256-row kernel's, squared and summed in another order, N 2^-24 at most
        _, Z256 = pkg.sphattn_fwd_tile_rows(q.to(DEV), k.to(DEV), v.to(DEV), Z=torch.empty_like(Z), dtype=dtype, tile_rows=256)
        np.testing.assert_allclose(Z.cpu().double().numpy(), Z256.cpu().double().numpy(), rtol=(N + 8) * 2.0 ** -24)
    else:
        # a single key: z carries the fp32 rounding of one score that may nearly cancel
        np.testing.assert_allclose(Z.cpu().double().numpy(), ref_z, rtol=2e-4, atol=1e-7 * ref_z.max())


@pytest.mark.parametrize("H,Nq,Nk,d", [(64, 300, 300, 128), (12, 1500, 1500, 128), (100, 300, 300, 64), (20, 129, 1000, 128),
                                       (3, 50, 64, 128), (2, 64, 1, 64), (30, 1050, 640, 64)])
def test_short_key_axes_take_the_narrow_form_of_the_256_row_kernel(pkg, H, Nq, Nk, d):
    """bf16 launches that 64-row workgroups would overfill, with few key tiles, and single tiles: every element
    within what rounding each score and the result to bf16 (2^-8 of them at most) allows against 64 bits, and
    bit for bit what 256 rows give (the key-split kernel adds the halves of a tile separately and does not)."""
    print(f"case narrow H={H} Nq={Nq} Nk={Nk} d={d}", flush=True)
    q, _, _ = si.make_qkv(1, H, Nq, d, "bf16", seed=4800 + Nq)
    _, k, v = si.make_qkv(1, H, Nk, d, "bf16", seed=4900 + Nk)
    q, k, v = q.to(DEV), k.to(DEV), v.to(DEV)
    Z = torch.empty((1, H, Nq), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(q, k, v, O=torch.empty_like(q), Z=Z, dtype="bf16")
    torch.cuda.synchronize()
    for h in range(H):
        V, S = v[0, h].double(), q[0, h].double() @ k[0, h].double().t().contiguous()
        z = (S * S).sum(1, keepdim=True)
        ref = S @ V / z.sqrt()
        bound = 2.0 ** -8 * (ref.abs() + S.abs() @ V.abs() / z.sqrt()) + 1e-5
        assert ((O[0, h].double() - ref).abs() <= bound).all(), h
        assert ((Z[0, h].double() - z[:, 0]).abs() <= 2e-4 * z[:, 0] + 1e-7 * z.max()).all(), h
    if Nq == Nk:
        whole, _ = pkg.sphattn_fwd_tile_rows(q, k, v, tile_rows=256)
        assert torch.equal(O, whole)


@pytest.mark.parametrize("Nq,Nk,d,dtype", [(130, 1, 64, "f16"), (127, 65, 128, "f16"), (200, 191, 128, "bf16"),
                                           (129, 448, 64, "bf16"), (300, 130, 128, "fp8qk_bf16v"), (1, 320, 64, "fp8qk_bf16v")])
def test_partial_accumulators_with_multiplicities(pkg, oracle, Nq, Nk, d, dtype):
    print(f"case keysplit partial Nq={Nq} Nk={Nk} d={d} {dtype}", flush=True)
    q, _, _ = si.make_qkv(1, 4, Nq, d, dtype, seed=4100 + Nq)
    _, k, v = si.make_qkv(1, 2, Nk, d, dtype, seed=4200 + Nk)
    g = torch.Generator(device="cpu").manual_seed(4300 + Nk)
    mult = torch.poisson(torch.full((1, Nk), 1.5), generator=g).to(torch.float32)
    mult[:, 0] = 2.0
    o, z = pkg.sphattn_partial_fwd(q.to(DEV), k.to(DEV), v.to(DEV), mult.to(DEV), dtype=dtype)
    O = pkg.sphattn_cross_fwd(q.to(DEV), k.to(DEV), v.to(DEV), mult.to(DEV), dtype=dtype)
    torch.cuda.synchronize()
    bits, kinds = _bits(q, k, v)
    ref_o, ref_z = oracle.spherical_accumulate(*bits, mult.numpy(), kinds=kinds)
    nrm = np.sqrt(ref_z)[..., None]
    assert _rel_err(o.cpu().double().numpy() / nrm, ref_o / nrm) <= TOL_PART[dtype]
    np.testing.assert_allclose(z.cpu().double().numpy(), ref_z, rtol=2e-4, atol=1e-7 * ref_z.max())
    assert _rel_err(O.cpu().double().numpy(), oracle.spherical_tail(ref_o[None], ref_z[None])) <= TOL_O[dtype]


def test_several_batches_of_128_row_items_walk_the_keys_both_ways(pkg, oracle):
    """More items than run at once: the second batch of a persistent workgroup reuses its LDS and
    streams the (ragged) keys backwards."""
    B, H, N, d = 1, 40, 1100, 128                # 360 items for 256 workgroups
    q, k, v = si.make_qkv(B, H, N, d, "f16", seed=4400)
    O, _ = pkg.sphattn_fwd_tile_rows(q.to(DEV), k.to(DEV), v.to(DEV), dtype="f16", tile_rows=128)
    torch.cuda.synchronize()
    bits, kinds = _bits(q, k, v)
    assert _rel_err(O.cpu().double().numpy(), oracle.spherical_attention(*bits, kinds=kinds)) <= TOL_O["f16"]


# B, H, H_kv, N_q, N_k, d, dtype, multiplicities: shapes that the calls below cut into slices (few query
# rows against many keys), rows of a group of heads packed into whole and ragged tiles
CUT = [(1, 4, 2, 33, 3001, 128, "bf16", False), (2, 6, 2, 100, 2500, 64, "f16", True), (1, 1, 1, 1, 5000, 128, "bf16", True),
       (1, 8, 1, 200, 4096, 64, "fp8qk_bf16v", False), (1, 1, 1, 3000, 3000, 128, "f16", False), (1, 3, 1, 77, 6000, 64, "f32", True)]


@pytest.mark.parametrize("B,H,H_kv,Nq,Nk,d,dtype,with_mult", CUT)
def test_few_query_rows_cut_the_key_axis(pkg, oracle, B, H, H_kv, Nq, Nk, d, dtype, with_mult):
    """sphattn_cross_fwd with an output of its own (slices and their combination) and into a given
    output (one launch): both against the oracle; z as well."""
    print(f"case cut B={B} H={H} H_kv={H_kv} Nq={Nq} Nk={Nk} d={d} {dtype}", flush=True)
    lib = pkg.load_library()
    need = lib.sphattn_cross_splitkv_workspace_bytes(B, H, H_kv, Nq, Nk, d, pkg._dtype_code(dtype))
    assert need >= 2 * B * H * Nq * (d + 1) * 4
    q, _, _ = si.make_qkv(B, H, Nq, d, dtype, seed=4500 + Nq)
    _, k, v = si.make_qkv(B, H_kv, Nk, d, dtype, seed=4600 + Nk)
    mult = None
    if with_mult:
        g = torch.Generator(device="cpu").manual_seed(4700 + Nk)
        mult = torch.poisson(torch.full((B, Nk), 1.5), generator=g).to(torch.float32)
        mult[:, 0] = 2.0
    qd, kd, vd, md = (t.to(DEV) if t is not None else None for t in (q, k, v, mult))
    Z = torch.empty((B, H, Nq), dtype=torch.float32, device=DEV)
    O = pkg.sphattn_cross_fwd(qd, kd, vd, md, Z=Z, dtype=dtype)
    given = torch.full_like(O, float("nan"))
    pkg.sphattn_cross_fwd(qd, kd, vd, md, O=given, dtype=dtype)
    torch.cuda.synchronize()
    bits, kinds = _bits(q, k, v)
    ref_o, ref_z = oracle.spherical_accumulate(*bits, None if mult is None else mult.numpy(), kinds=kinds)
    ref = oracle.spherical_tail(ref_o[None], ref_z[None])
    tol = {**TOL_O, "f32": 1e-4}[dtype]
    assert _rel_err(O.cpu().double().numpy(), ref) <= tol
    assert _rel_err(given.cpu().double().numpy(), ref) <= tol
    np.testing.assert_allclose(Z.cpu().double().numpy(), ref_z, rtol=2e-4, atol=1e-7 * ref_z.max())


def test_cut_launch_writes_inside_its_workspace_and_repeats(pkg):
    """The slices' workspace, NaN-filled with guard bytes behind it: every slot read was written,
    nothing past the stated size is, and two calls give the same bits."""
    import ctypes
    lib, P = pkg.load_library(), ctypes.c_void_p
    B, H, H_kv, Nq, Nk, d = 1, 4, 2, 130, 4000, 128
    q, k, v = (torch.randn(B, h, n, d, device=DEV).to(torch.bfloat16) for h, n in ((H, Nq), (H_kv, Nk), (H_kv, Nk)))
    need = lib.sphattn_cross_splitkv_workspace_bytes(B, H, H_kv, Nq, Nk, d, 1)
    outs = []
    for _ in range(2):
        ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
        O = torch.empty_like(q)
        rc = lib.sphattn_cross_splitkv_fwd(P(q.data_ptr()), P(k.data_ptr()), P(v.data_ptr()), P(0), P(O.data_ptr()), P(0),
                                           B, H, H_kv, Nq, Nk, d, 1, P(ws.data_ptr()), need, None)
        torch.cuda.synchronize()
        assert rc == 0 and bool((ws[need:] == 0xFF).all()) and bool(torch.isfinite(O.float()).all())
        outs.append(O)
    assert torch.equal(outs[0], outs[1])


def test_cut_calls_replay_from_a_graph(pkg):
    """Forward and backward calls that are cut, with outputs and workspaces from torch's allocator,
    captured into a graph: three replays on fresh inputs, eager work in between, bit for bit the
    eager results."""
    B, H, H_kv, N, d = 1, 4, 2, 4000, 64
    lib = pkg.load_library()
    assert lib.sphattn_bwd_workspace_bytes(B, H, H_kv, N, d, 1) > 0
    assert lib.sphattn_cross_splitkv_workspace_bytes(B, H, H_kv, 40, N, d, 1) > 0
    g = torch.Generator(device=DEV).manual_seed(1)

    def fresh(h, n):
        return torch.randn((B, h, n, d), generator=g, device=DEV).to(torch.bfloat16)
    q, k, v, dO, qs = fresh(H, N), fresh(H_kv, N), fresh(H_kv, N), fresh(H, N), fresh(H, 40)

    def step():
        Z = torch.empty((B, H, N), dtype=torch.float32, device=DEV)
        O = pkg.sphattn_cross_fwd(q, k, v, Z=Z, dtype="bf16")
        return [pkg.sphattn_cross_fwd(qs, k, v, dtype="bf16"), O, *pkg.sphattn_grn_bwd(q, k, v, None, O, dO, Z, dtype="bf16")]

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = step()
    for _ in range(3):
        for t, h, n in ((q, H, N), (k, H_kv, N), (v, H_kv, N), (dO, H, N), (qs, H, 40)):
            t.copy_(fresh(h, n))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in outs]
        want = step()
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b) and bool(torch.isfinite(a.float()).all())
