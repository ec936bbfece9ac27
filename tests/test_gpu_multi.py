"""The passes that serve many vectors: every number of groups of 16 vectors a pass takes, with part groups, odd sizes and rows
of any alignment, against dense FP64 solves."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu

KW = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=4, shift_policy=dfl.DFISHER_SHIFT_NONE, x_fp64=True)
# four conjugate-gradient sweeps from an FP32 Gram (1e-6 of W, condition < 100) end at FP64 rounding times the condition
TOL = 1e-11


def problem(n, m, pad, nrhs, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed + 31 * n + m)
    buf = torch.full((n + 2, m + pad), float("nan"), device="cuda")
    buf[:n, :m] = torch.randn(n, m, device="cuda", generator=g) / m ** 0.5
    V = torch.randn(nrhs, m, device="cuda", generator=g)
    return buf[:n, :m], V


def reference(S, lams, V):
    D, B = S.double(), V.double()
    W = D @ D.T.contiguous()
    out = []
    for lam in lams:   # x = (v - S^T (W + lam)^-1 S v) / lam
        y = torch.linalg.solve(W + lam * torch.eye(len(W), dtype=W.dtype, device=W.device), D @ B.T.contiguous())
        out.append((B - (D.T.contiguous() @ y).T) / lam)
    return torch.stack(out)


def check(X, R):
    assert bool(torch.isfinite(X).all())
    assert float((X - R).abs().max() / R.abs().max()) <= TOL


@pytest.mark.parametrize("n,m,pad", [(5, 40, 0), (17, 63, 1), (64, 130, 2), (129, 999, 0), (200, 4097, 3), (150, 40000, 0)])
@pytest.mark.parametrize("nlam,nrhs", [(1, 1), (2, 8), (1, 17), (3, 11), (7, 7), (5, 13), (9, 8)])
def test_batched(n, m, pad, nlam, nrhs):   # 1, 16, 17, 33, 49, 65 and 72 vectors
    ctx = dfl.dfisher_ctx_create(0)
    S, V = problem(n, m, pad, nrhs)
    lams = [0.05 * 1.3 ** k for k in range(nlam)]
    X, _ = dfl.dfisher_solve_batched(ctx, S, lams, V, **KW)
    check(X, reference(S, lams, V))
    ctx.close()


@pytest.mark.parametrize("nrhs", [1, 2, 16, 31, 33, 64, 70])
def test_factor_solve(nrhs):
    ctx = dfl.dfisher_ctx_create(0)
    S, V = problem(333, 5003, 1, nrhs)
    f, _ = dfl.dfisher_factor_create(ctx, S, 0.05, **KW)
    X = dfl.dfisher_factor_solve(f, V)
    check(X[0] if isinstance(X, tuple) else X, reference(S, [0.05], V)[0])


def test_two_groups_without_the_memory():
    """In a capture whose workspace only holds two groups of vectors, the passes take two at a time."""
    n, m, nrhs = 64, 20000, 32
    lams = [0.05, 0.1]
    ctx = dfl.dfisher_ctx_create(0)
    Sw, Vw = problem(n, 24000, 0, nrhs, 1)
    dfl.dfisher_solve_batched(ctx, Sw, [0.1], Vw, **KW)   # sizes the workspace: two groups of a longer problem
    S, V = problem(n, m, 0, nrhs)
    X = torch.zeros(2, nrhs, m, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dfl.dfisher_solve_batched(ctx, S, lams, V, X=X, enqueue_only=True, **KW)
    for _ in range(2):
        X.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        check(X, reference(S, lams, V))
    del g
    ctx.close()


@pytest.mark.parametrize("n", [1, 65, 200])
@pytest.mark.parametrize("nlam", [1, 32, 33])
@pytest.mark.parametrize("policy", [dfl.DFISHER_SHIFT_NONE, dfl.DFISHER_SHIFT_ALWAYS])
def test_many_dampings(n, nlam, policy):
    """The factorisations read one shared Gram, each with its own damping (and shift), up to 32 at a time."""
    ctx = dfl.dfisher_ctx_create(0)
    S, V = problem(n, 700, 0, 1)
    lams = [0.05 * 1.05 ** k for k in range(nlam)]
    X, infos = dfl.dfisher_solve_batched(ctx, S, lams, V, **{**KW, "shift_policy": policy})
    assert all(i["potrf_info"] == 0 and (i["shift"] > 0) == (policy == dfl.DFISHER_SHIFT_ALWAYS) for i in infos)
    check(X, reference(S, lams, V))
    x, info = dfl.dfisher_solve(ctx, S, V[0], lams[-1], **{**KW, "shift_policy": policy})
    assert (info["shift"] > 0) == (policy == dfl.DFISHER_SHIFT_ALWAYS)
    check(x, X[-1, 0])
    ctx.close()
