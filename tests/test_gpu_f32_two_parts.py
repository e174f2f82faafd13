"""fp32 storage in two fp16 parts (sphattn_f32.hpp): the shortest key axes that take them, odd numbers of tiles, parts of
one, and values that a pair of fp16 numbers holds only with the powers of two of rows, keys and columns, or not at all
(then three bf16 parts or the fp32 instruction do the work).  Every output column of a head is compared with 64 bits on
its own.  With A = sqrt(q^2 . k^2) for the size of a score's terms, a score is off by rounding q and k (2^-24 in the root mean square of each) and by
at most 12 to 24 additions (2^-25 each in the root mean square): 1.5e-7 A.  Independent errors of the scores move an
output by sqrt(sum A^2 v^2) / n and, through n, by o sum |S| A / n^2, and adding up 57 groups of keys moves it by 2^-25 sqrt(57)
of its own size, 2.3e-7.
5e-7 of the three together is asked for.  A single z has no mean over rows: each of 24 additions may be 2^-24 short
of a partial sum of twice A, so 3e-6 of 2 sum |S| A."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pkg():
    import paper_2505_09326_amd as p
    p.load_library()
    return p


def _inputs(kind, H, Nq, Nk, d, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    q, k, v = (torch.randn((1, H, n, d), generator=g, device=DEV) for n in (Nq, Nk, Nk))
    m = None
    if kind == "columns":                          # every column of V in a binade of its own
        v *= torch.pow(2.0, torch.arange(d, device=DEV) % 61 - 30.0)
    elif kind == "zero columns":
        v[..., 5::16] = 0.0
    elif kind == "rows":                           # rows of Q far apart, all keys small; a row of zeros
        q *= torch.pow(2.0, torch.arange(Nq, device=DEV) % 41 - 20.0)[:, None]
        q[:, :, 7] = 0.0
        k *= 1e-9
    elif kind == "outliers":                       # the first key a hundred times the others, its value a thousand
        k[:, :, 0] *= 100.0
        v[:, :, 0] *= 1000.0
    elif kind == "unseen value":                   # a value of 1e7 that no score touches
        k[:, :, 0] = 0.0
        v[:, :, 0] = 1e7
    elif kind == "unscored":                       # the same of every other key, the others' values a thousandth
        k[:, :, ::2], v[:, :, ::2], v[:, :, 1::2] = 0.0, 100.0, v[:, :, 1::2] * 1e-3
    elif kind == "unvalued":                       # every other value zero, the other keys a thousandth
        v[:, :, ::2], k[:, :, 1::2] = 0.0, k[:, :, 1::2] * 1e-3
    elif kind == "growing":                        # later keys a hundred times the first, later values a thousandth
        k[:, :, Nk // 2:] *= 100.0
        v[:, :, Nk // 3:] *= 1e-3
    elif kind == "late":                           # one late key beyond fp16 at the first tile's scale
        k[:, :, -1] *= 1e6
    elif kind == "tiny column":                    # a column whose one value vanishes beside the others
        v[..., 5] = 0.0
        v[:, :, 7, 5] = 1e-30
    elif kind == "counts":
        m = torch.poisson(torch.full((1, Nk), 1.5, device=DEV), generator=g)
        m[:, 0], m[:, Nk // 2] = 2.0, 5000.0
    return q, k, v, m


@pytest.mark.parametrize("kind", ["plain", "columns", "zero columns", "rows", "outliers", "unseen value", "unscored", "unvalued", "growing", "late", "tiny column", "counts"])
@pytest.mark.parametrize("H,Nq,Nk,d", [(32, 512, 512, 128), (40, 391, 577, 128), (130, 300, 640, 128), (16, 4000, 1100, 128), (32, 512, 1792, 64), (64, 257, 1825, 64), (16, 4000, 1900, 64)])
def test_columns_against_64_bits(pkg, H, Nq, Nk, d, kind):
    print(f"case two parts {H} x {Nq} of {Nk} x {d} {kind}", flush=True)
    q, k, v, m = _inputs(kind, H, Nq, Nk, d, 6000 + Nk + d)
    O, Z = torch.empty_like(q), torch.empty((1, H, Nq), device=DEV)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype="f32")
    o, z = pkg.sphattn_partial_fwd(q, k, v, m, dtype="f32")
    torch.cuda.synchronize()
    for h in (0, H // 2, H - 1):
        kh = k[0, h].double() * m[0].double()[:, None] if m is not None else k[0, h].double()
        S = q[0, h].double() @ kh.t().contiguous()
        A = ((q[0, h].double() ** 2) @ (kh ** 2).t().contiguous()).sqrt()
        n2, dz = (S * S).sum(1), 2.0 * (S.abs() * A).sum(1)
        n = n2.sqrt()[:, None].clamp_min(1e-140)
        V = v[0, h].double()
        ref = S @ V / n
        size = (ref.abs() + (A * A @ V ** 2).sqrt() / n + ref.abs() * dz[:, None] / 2.0 / n ** 2).norm(dim=0)
        for got in (O[0, h].double(), o[0, h].double() / n):
            assert torch.isfinite(got).all()
            err = (got - ref).norm(dim=0)
            assert (err <= 5e-7 * size).all(), (h, (err / size).max().item())
        for got in (Z[0, h].double(), z[0, h].double()):
            assert ((got - n2).abs() <= 3e-6 * dz).all(), (h, ((got - n2).abs() / dz.clamp_min(1e-300)).max().item())


def _one_key(kind, size, value, H, Nq, Nk, d, seed):
    """Inputs in which one key among the first has `size` times the others' scores (by its elements, by its count, or for one
    query row alone) and `value` times their values in a quarter of V's columns."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    q, k, v = (torch.randn((1, H, n, d), generator=g, device=DEV) for n in (Nq, Nk, Nk))
    m = None
    if kind == "key":
        q += 2.0
        k[:, :, 3] = k[:, :, 3].abs() * size
    elif kind == "late key":
        q += 2.0
        k[:, :, Nk - 3] = k[:, :, Nk - 3].abs() * size
    elif kind == "count":
        m = torch.poisson(torch.full((1, Nk), 1.5, device=DEV), generator=g)
        m[:, 3] = size
    elif kind == "one row":                        # element 0 belongs to this key and this row
        q[..., 0] = 0.0
        q[:, :, 21, 0] = size
        k[..., 0] = 0.0
        k[:, :, 3, 0] = 1.0
    v[:, :, Nk - 3 if kind == "late key" else 3, :d // 4] *= value
    return q, k, v, m


@pytest.mark.parametrize("kind,size", [("key", 1e2), ("key", 1e4), ("key", 1e5), ("key", 1e6), ("key", 1e7), ("key", 1e9), ("key", 1e11),
                                       ("late key", 1e5), ("count", 1e3), ("count", 1e5), ("count", 1e7), ("one row", 1e3), ("one row", 1e5), ("one row", 1e8)])
@pytest.mark.parametrize("value", [0.0, 1e-6])
@pytest.mark.parametrize("H,Nq,Nk,d", [(32, 512, 512, 128), (16, 4000, 1100, 128), (64, 257, 1825, 64), (16, 4000, 1900, 64)])
def test_columns_without_the_largest_key(pkg, H, Nq, Nk, d, kind, size, value):
    """Columns as above.  Rows over the quarter of the columns: a row's errors in the scores are common to its columns, so its
    norm over 16 or 32 of them scatters; twice the bound.  The largest key's products may all have one sign, so partial sums reach the
    score itself as well as twice A: z within 3e-6 of 2 sum |S| (A + |S|)."""
    print(f"case two parts {H} x {Nq} of {Nk} x {d} {kind} {size:g}, {value:g}", flush=True)
    q, k, v, m = _one_key(kind, size, value, H, Nq, Nk, d, 6100 + Nk + d)
    O, Z = torch.empty_like(q), torch.empty((1, H, Nq), device=DEV)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, Z=Z, dtype="f32")
    o, z = pkg.sphattn_partial_fwd(q, k, v, m, dtype="f32")
    torch.cuda.synchronize()
    for h in (0, H - 1):
        kh = k[0, h].double() * m[0].double()[:, None] if m is not None else k[0, h].double()
        S = q[0, h].double() @ kh.t().contiguous()
        A = ((q[0, h].double() ** 2) @ (kh ** 2).t().contiguous()).sqrt()
        n2, dz = (S * S).sum(1), 2.0 * (S.abs() * A).sum(1)
        n = n2.sqrt()[:, None]
        V = v[0, h].double()
        ref = S @ V / n
        size = ref.abs() + (A * A @ V ** 2).sqrt() / n + ref.abs() * dz[:, None] / 2.0 / n ** 2
        for got in (O[0, h].double(), o[0, h].double() / n):
            err = got - ref
            columns = err.norm(dim=0) / size.norm(dim=0)
            rows = err[:, :d // 4].norm(dim=1) / size[:, :d // 4].norm(dim=1)
            print(f"  columns {columns.max().item():.2e} rows {rows.max().item():.2e}", flush=True)
            assert (columns <= 5e-7).all() and (rows <= 1e-6).all()
        for got in (Z[0, h].double(), z[0, h].double()):
            assert ((got - n2).abs() <= 3e-6 * (dz + 2.0 * n2)).all()


def _ordinary(kind, H, Nq, Nk, d, seed):
    """Inputs that programs have, with zeros where a sample of the first keys would look."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    q, k, v = (torch.randn((1, H, n, d), generator=g, device=DEV) for n in (Nq, Nk, Nk))
    m = None
    if kind.startswith("left padding"):
        n = int(kind.split()[-1])
        k[:, :, :n], v[:, :, :n] = 0.0, 0.0
    elif kind == "right padding":
        k[:, :, 100:], v[:, :, 100:] = 0.0, 0.0
    elif kind == "no values at first":
        v[:, :, :40] = 0.0
    elif kind == "one late column":
        v[:, :, :40, 5] = 0.0
    elif kind == "cut at one":
        v = (v - 1.0).clamp_min(0.0)
    elif kind == "one value in twenty":
        v = v * (torch.rand(v.shape, generator=g, device=DEV) < 0.05)
    elif kind == "one-hot":
        v = torch.nn.functional.one_hot(torch.randint(0, d, v.shape[:3], generator=g, device=DEV), d).float()
    elif kind == "no counts at first":
        m = torch.poisson(torch.full((1, Nk), 1.5, device=DEV), generator=g)
        m[:, :100] = 0.0
    elif kind == "zero columns":
        v[..., 5::16] = 0.0
    elif kind == "late key":                       # (not ordinary: fp16 does not hold it)
        k[:, :, -1] *= 1e6
    return q, k.contiguous(), v.contiguous(), m


@pytest.mark.parametrize("kind", ["plain", "zero columns", "left padding 31", "left padding 100", "left padding 600", "right padding", "no values at first", "one late column",
                                  "cut at one", "one value in twenty", "one-hot", "no counts at first", "late key"])
@pytest.mark.parametrize("H,Nq,Nk,d", [(32, 512, 1024, 128), (16, 4000, 1100, 128), (64, 257, 1825, 64), (16, 4000, 1900, 64)])
def test_ordinary_values_take_two_parts(pkg, H, Nq, Nk, d, kind):
    """A value of 1e30 in the last row of column 0 sends every workgroup to three parts, whose other columns do not
    depend on it: results that differ from them in their last bits were formed in two.  And the bound of the columns."""
    print(f"case two parts {H} x {Nq} of {Nk} x {d} {kind}", flush=True)
    q, k, v, m = _ordinary(kind, H, Nq, Nk, d, 6200 + Nk + d)
    three = v.clone()
    three[:, :, -1, 0] = 1e30
    O, T = torch.empty_like(q), torch.empty_like(q)
    pkg.sphattn_cross_fwd(q, k, v, m, O=O, dtype="f32")
    pkg.sphattn_cross_fwd(q, k, three, m, O=T, dtype="f32")
    torch.cuda.synchronize()
    # of every 128 rows (whole workgroups take one way or the other)
    differs = (O[0, :, :, 1:] != T[0, :, :, 1:]).any(-1).float()
    blocks = [differs[:, r:r + 128].mean(1) for r in range(0, Nq, 128)]
    for share in blocks:
        print("  rows in two parts", share.min().item(), share.max().item(), flush=True)
        assert (share > 0.5).all() if kind != "late key" else (share == 0.0).all()
    for h in (0, H - 1):
        kh = k[0, h].double() * m[0].double()[:, None] if m is not None else k[0, h].double()
        S = q[0, h].double() @ kh.t().contiguous()
        A = ((q[0, h].double() ** 2) @ (kh ** 2).t().contiguous()).sqrt()
        dz, n = 2.0 * (S.abs() * A).sum(1)[:, None], S.norm(dim=1, keepdim=True)
        V = v[0, h].double()
        ref = S @ V / n
        size = (ref.abs() + (A * A @ V ** 2).sqrt() / n + ref.abs() * dz / 2.0 / n ** 2).norm(dim=0)
        assert ((O[0, h].double() - ref).norm(dim=0) <= 5e-7 * size).all()
