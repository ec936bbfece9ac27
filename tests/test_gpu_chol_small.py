"""dfisher_potrf of matrices with diagonal entries so small that the reciprocal of a pivot is not a number of FP64 any more."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


def pow2(e):   # exact, in two factors: 2^-600 alone times 2^-600 would be lost in the wrong order
    return torch.ldexp(torch.ones_like(e, dtype=torch.float64), e)


@pytest.mark.parametrize("n", [1, 3, 16, 70, 200, 500])
@pytest.mark.parametrize("kind", ["-513", "-520", "-530", "mixed", "last"])
def test_small_pivots(n, kind):
    """W = D M D with D = 2^e: |L L^T - W| <= 4 n (2^-53 sqrt(W_ii W_jj) + 2^-1074), the rounding of n sums and of subnormals."""
    ctx = dfl.dfisher_ctx_create(0)
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, n + 8, device="cuda", generator=g, dtype=torch.float64)
    M = A @ A.T.contiguous() / (n + 8) + torch.eye(n, device="cuda", dtype=torch.float64)
    if kind == "mixed":
        e = -torch.randint(0, 525, (n,), device="cuda", generator=g)
    elif kind == "last":
        e = torch.zeros(n, dtype=torch.int64, device="cuda")
        e[-1] = -520
    else:
        e = torch.full((n,), int(kind), device="cuda")
    W = M * pow2(e)[:, None] * pow2(e)[None, :]
    L = W.clone()
    assert dfl.dfisher_potrf(ctx, L) == 0
    Ls = L * pow2(-e)[:, None]
    Ws = W * pow2(-e)[:, None] * pow2(-e)[None, :]
    bound = 4 * n * (2.0 ** -53 * float(M.diagonal().max()) + pow2((-1074 - e[:, None] - e[None, :]).clamp(min=-1020)))
    assert bool(((Ls @ Ls.T.contiguous() - Ws).abs() <= bound).all())
    ctx.close()
