"""The one-launch Cholesky (csrc/chol.hip) at the edges of its 64 x 64 tiles and 16-column panels, against
torch's FP64 factor of the same matrix, and the pivot index of a breakdown at those edges."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = dfl.dfisher_ctx_create(0)
    yield c
    c.close()


def _spd(n, cond_shift=1e-2):
    g = torch.Generator(device="cuda").manual_seed(n)
    B = torch.randn(n, n + 8, dtype=torch.float64, device="cuda", generator=g)
    return B @ B.T.contiguous() / n + cond_shift * torch.eye(n, dtype=torch.float64, device="cuda")


# one block column, two (no off-diagonal task), three (the first one), odd remainders of 1 .. 63 rows, and
# more tasks than workgroups fit on the device at once (n = 2900: 1036 tasks)
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257, 500, 1023, 2900])
def test_factor(ctx, n):
    W = _spd(n)
    L = W.clone()
    assert dfl.dfisher_potrf(ctx, L) == 0
    ref = torch.linalg.cholesky(W)
    # n products of a row, each off by at most an FP64 rounding, times the factor's conditioning (< 1e2)
    assert float((L - ref).norm() / ref.norm()) <= 1e-12
    again = W.clone()
    assert dfl.dfisher_potrf(ctx, again) == 0
    assert torch.equal(again, L)   # the order of every sum is fixed


@pytest.mark.parametrize("n", [40, 130, 200])
@pytest.mark.parametrize("value", [-1.0, 0.0, float("nan")])
def test_first_bad_pivot(ctx, n, value):
    for bad in {1, 16, 17, min(n, 64), min(n, 65), min(n, 129), n}:
        W = 2.0 * torch.eye(n, dtype=torch.float64, device="cuda")
        W[bad - 1, bad - 1] = value
        if bad < n:
            W[n - 1, n - 1] = value   # a later breakdown is not the one reported
        assert dfl.dfisher_potrf(ctx, W) == bad
    W = 2.0 * torch.eye(n, dtype=torch.float64, device="cuda")   # and nothing is left behind
    assert dfl.dfisher_potrf(ctx, W) == 0
