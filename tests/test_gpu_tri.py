"""The triangular solves of the library's own factors (csrc/tri.hip) at the edges of their 128-row blocks
and of the groups of four vectors, against torch's FP64 solves with the factor's own L."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu

LAM = 1e-2


@pytest.fixture(scope="module")
def ctx():
    c = dfl.dfisher_ctx_create(0)
    yield c
    c.close()


def _S(n, m, seed=0):
    g = torch.Generator(device="cuda").manual_seed(1000 * n + seed)
    return torch.randn(n, m, device="cuda", generator=g) / n ** 0.5


def _x(S, v, L):
    """(v - S^T L^-T L^-1 S v) / lambda with the given factor, in FP64."""
    S, v = S.double(), v.double()
    y = torch.cholesky_solve((S @ v)[:, None], L)[:, 0]
    return (v - S.T.contiguous() @ y) / LAM


# one block (no chain), two, three, more than the panels held in registers, odd remainders
@pytest.mark.parametrize("n,nrhs", [(1, 1), (100, 3), (127, 1), (128, 5), (129, 1), (129, 2), (255, 1), (256, 4),
                                    (257, 5), (385, 1), (640, 9), (1000, 1), (1001, 4)])
def test_factor_solve_matches_its_factor(ctx, n, nrhs):
    m = 4 * n + 37
    S = _S(n, m)
    f, _ = dfl.dfisher_factor_create(ctx, S, LAM, sweeps=0, x_fp64=True)
    L = dfl.dfisher_factor_copy_L(f)
    assert not torch.triu(L, diagonal=1).any()   # the factor holds L^T there, its copy does not
    g = torch.Generator(device="cuda").manual_seed(n)
    V = torch.randn(nrhs, m, device="cuda", generator=g)
    X = dfl.dfisher_factor_solve(f, V)
    for r in range(nrhs):
        ref = _x(S, V[r], L)
        # FP64 sums of n and m terms through a factor of condition < 1e2
        assert float((X[r] - ref).norm() / ref.norm()) <= 1e-12
    f.close()


@pytest.mark.parametrize("sizes", [[5, 129, 300], [128, 1, 257, 64], [700, 130, 131]])
def test_uneven_matches_single(ctx, sizes):
    """Every problem of a grouped solve equals its own single solve (other launches, the same sums)."""
    Ss = [_S(n, 4 * n + 128, 1) for n in sizes]
    vs = [torch.randn(S.shape[1], device="cuda", generator=torch.Generator(device="cuda").manual_seed(7)) for S in Ss]
    xs, _ = dfl.dfisher_solve_uneven(ctx, Ss, vs, [LAM] * len(sizes), sweeps=2, x_fp64=True)
    for S, v, x in zip(Ss, vs, xs):
        one, _ = dfl.dfisher_solve(ctx, S, v, LAM, sweeps=2, x_fp64=True)
        # both refined to FP64 level from Grams that may be split differently over the columns
        assert float((x - one).norm() / one.norm()) <= 1e-12
