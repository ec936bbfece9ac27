"""The FP32 Gram's diagonal tiles, partial panels, odd step counts and slice ends, with whole numbers whose sums are exact:
the result equals the FP64 product bit for bit. What lies outside S (padding columns, rows behind it) is NaN."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = dfl.dfisher_ctx_create(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", [1, 31, 33, 97, 129, 223, 225, 256, 257, 300, 512, 775])
@pytest.mark.parametrize("m,pad", [(1, 3), (4, 0), (35, 5), (64, 8), (68, 0), (132, 4), (1000, 24), (4093, 7)])
def test_exact(ctx, n, m, pad):
    g = torch.Generator(device="cuda").manual_seed(100 * n + m)
    buf = torch.full((n + 9, m + pad), float("nan"), device="cuda")
    buf[:n, :m] = torch.randint(-8, 9, (n, m), device="cuda", generator=g).float()
    S = buf[:n, :m]   # |sums| <= 64 * 4093 < 2^24: exact in FP32 in any order
    W = dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_FP32, 0.0)
    D = S.double()
    assert torch.equal(W, D @ D.T.contiguous())
