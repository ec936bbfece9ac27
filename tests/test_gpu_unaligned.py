"""Rows of any stride and offset go through the same passes as 16-byte aligned ones: every result equals, bit for bit, that of
an aligned copy of S. What lies outside S (padding columns, rows behind it) is NaN."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = dfl.dfisher_ctx_create(0)
    yield c
    c.close()


def both(n, m, stride, off):
    """S behind `off` floats with rows `stride` apart, and a copy with aligned rows."""
    g = torch.Generator(device="cuda").manual_seed(n + 7 * m)
    vals = torch.randn(n, m, device="cuda", generator=g) / n ** 0.5
    flat = torch.full((off + (n + 3) * stride,), float("nan"), device="cuda")
    odd = flat[off:off + n * stride].view(n, stride)[:, :m]
    odd.copy_(vals)
    even = torch.full((n + 3, (m + 7) // 4 * 4), float("nan"), device="cuda")[:n, :m]
    even.copy_(vals)
    return odd, even


# strides and offsets of every alignment; last blocks of 1 .. 32 columns; 8, 16 and 32 rows a lane and more than 2048 rows
SHAPES = [(1, 33, 33, 1), (17, 1001, 1001, 0), (64, 4099, 4102, 3), (513, 2050, 2051, 2), (1000, 9999, 9999, 0),
          (1025, 4127, 4129, 1), (2049, 8193, 8194, 3)]


@pytest.mark.parametrize("n,m,stride,off", SHAPES)
@pytest.mark.parametrize("prec", [dfl.DFISHER_GRAM_BF16X3])
def test_gram(ctx, n, m, stride, off, prec):
    odd, even = both(n, m, stride, off)
    assert torch.equal(dfl.dfisher_gram(ctx, odd, prec, 0.5), dfl.dfisher_gram(ctx, even, prec, 0.5))


@pytest.mark.parametrize("n,m,stride,off", SHAPES)
def test_passes(ctx, n, m, stride, off):
    odd, even = both(n, m, stride, off)
    g = torch.Generator(device="cuda").manual_seed(5)
    vbuf = torch.randn(m + 3, device="cuda", generator=g)
    v = vbuf[3:]
    b = dfl.dfisher_gemv(ctx, odd, v)
    assert torch.equal(b, dfl.dfisher_gemv(ctx, even, v.clone()))
    ref = odd.double() @ v.double()
    bound = odd.double().abs() @ v.double().abs()
    assert bool(((b - ref).abs() <= 4 * m * 2.0 ** -53 * bound).all())   # FP64 sums of m exact products, either order
    y = torch.randn(n, device="cuda", dtype=torch.float64, generator=g)
    assert torch.equal(dfl.dfisher_apply(ctx, odd, v, y, 0.5), dfl.dfisher_apply(ctx, even, v.clone(), y, 0.5))


@pytest.mark.parametrize("n,m,stride,off", SHAPES)
def test_solve(ctx, n, m, stride, off):
    odd, even = both(n, m, stride, off)
    v = torch.randn(m, device="cuda", generator=torch.Generator(device="cuda").manual_seed(6))
    kw = dict(gram_prec=dfl.DFISHER_GRAM_BF16X3, sweeps=2)
    x, xe = (dfl.dfisher_solve(ctx, S, v, 1e-2, **kw)[0] for S in (odd, even))
    assert torch.equal(x, xe)


@pytest.mark.parametrize("n,m,stride,off", SHAPES[:6])
@pytest.mark.parametrize("nrhs", [1, 5, 20])
def test_factor_solve(ctx, n, m, stride, off, nrhs):
    odd, even = both(n, m, stride, off)
    V = torch.randn(nrhs, m + 1, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7))[:, :m]
    xs = []
    for S in (odd, even):
        f, _ = dfl.dfisher_factor_create(ctx, S, 1e-2, gram_prec=dfl.DFISHER_GRAM_BF16X3, sweeps=1)
        xs.append(dfl.dfisher_factor_solve(f, V))
    x, xe = (t[0] if isinstance(t, tuple) else t for t in xs)
    assert torch.equal(x, xe)


def test_no_room_for_planes(tmp_path):
    """A workspace held by a capture, without room for the planes: the tile kernel splits the rows, as it does when told to."""
    n, m, stride = 64, 70001, 70003
    odd, _ = both(n, m, stride, 1)

    def context(split):   # tuning: precision, tiles, floor(log2 m), aligned, slices / 8, split mode
        c = dfl.dfisher_ctx_create(0)
        f = tmp_path / f"tune{split}"
        f.write_text(f"0 1 16 0 4 -1\n1 1 16 0 4 {split}\n")
        dfl.dfisher_ctx_load_tuning(c, str(f))
        return c

    a, b = context(-1), context(0)
    dfl.dfisher_gram(a, odd, dfl.DFISHER_GRAM_FP32, 0.5)   # sizes the workspace: the partial tiles, no planes
    S, V = odd[:8, :200], torch.randn(1, 200, device="cuda")
    kw = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=0, shift_policy=dfl.DFISHER_SHIFT_NONE)
    X, _ = dfl.dfisher_solve_batched(a, S, [1.0], V, **kw)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dfl.dfisher_solve_batched(a, S, [1.0], V, X=X, enqueue_only=True, **kw)
    torch.cuda.synchronize()
    W = dfl.dfisher_gram(a, odd, dfl.DFISHER_GRAM_BF16X3, 0.5)
    assert torch.equal(W, dfl.dfisher_gram(b, odd, dfl.DFISHER_GRAM_BF16X3, 0.5))
    ref = odd.double() @ odd.double().T.contiguous() + 0.5 * torch.eye(n, dtype=torch.float64, device="cuda")
    assert float((W - ref).abs().max() / ref.abs().max()) <= 3e-5   # dropped lo.lo products
    del g
    a.close()
    b.close()
