"""The Gram's slice counts that are no multiple of the eight XCDs, its partly stored tiles and both forms
of its reduction, against torch's FP64 Gram."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = dfl.dfisher_ctx_create(0)
    yield c
    c.close()


# one tile and many slices (n <= 256), a last tile of 1 row, several tiles with 14, 21 ... slices, more than 16
# tiles (the other reduction), a slice of few columns, rows not 16-byte aligned
@pytest.mark.parametrize("n,m,pad", [(3, 5000, 0), (64, 70001, 3), (255, 33333, 3), (256, 40000, 0), (257, 30000, 0),
                                     (600, 20000, 0), (1281, 9000, 0), (1500, 7777, 2), (2048, 5000, 0), (520, 300, 0)])
@pytest.mark.parametrize("prec", [dfl.DFISHER_GRAM_FP32, dfl.DFISHER_GRAM_BF16X3, dfl.DFISHER_GRAM_MXFP8])
def test_gram(ctx, n, m, pad, prec):
    if prec == dfl.DFISHER_GRAM_MXFP8 and (m + pad) % 4:
        pytest.skip("the FP8 Gram takes 16-byte aligned rows")
    g = torch.Generator(device="cuda").manual_seed(n + m)
    S = torch.randn(n, m + pad, device="cuda", generator=g)[:, :m]
    W = dfl.dfisher_gram(ctx, S, prec, 0.5)
    ref = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    for c in range(0, m, 16384):
        blk = S[:, c:c + 16384].double()
        ref += blk @ blk.T.contiguous()
    ref += 0.5 * torch.eye(n, dtype=torch.float64, device="cuda")
    assert torch.equal(W, W.T)
    assert float(((W - ref).diagonal().abs() / ref.diagonal()).max()) <= 1e-13   # the diagonal is exact
    # FP32 sums of a slice; the dropped lo.lo products; E4M3 rounding of both operands
    tol = {dfl.DFISHER_GRAM_FP32: 2e-6, dfl.DFISHER_GRAM_BF16X3: 3e-5, dfl.DFISHER_GRAM_MXFP8: 0.13}[prec]
    d = ref.diagonal().sqrt()
    assert float(((W - ref).abs() / (d[:, None] * d[None, :])).max()) <= tol
