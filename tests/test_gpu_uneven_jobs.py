"""The uneven call's shared launches: more problems than one launch's job list holds, tiny and large ones, both forms of the
Gram reduction, few and many column blocks, against dense FP64 solves."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


def make(shapes):
    Ss, vs = [], []
    for k, (n, m) in enumerate(shapes):
        g = torch.Generator(device="cuda").manual_seed(977 + k)
        S = torch.randn(n, m, device="cuda", generator=g) / m ** 0.5
        if n > 1:   # (one row centered is zero)
            S = (S.double() - S.double().mean(0)).float()
        buf = torch.full((n, (m + 3) // 4 * 4 + 4), float("nan"), device="cuda")
        buf[:, :m] = S
        Ss.append(buf[:, :m])
        vs.append(torch.randn(m, device="cuda", generator=g))
    return Ss, vs


def reference(S, v, lam):
    D, b = S.double(), v.double()
    W = D @ D.T.contiguous() + lam * torch.eye(len(D), dtype=torch.float64, device="cuda")
    return (b - D.T.contiguous() @ torch.linalg.solve(W, D @ b)) / lam


MANY = [(1 + (37 * k) % 260, 300 + 97 * k) for k in range(37)]
LARGE = [(1300, 60001), (1281, 50002), (700, 300003), (64, 900001), (257, 800001)]


@pytest.mark.parametrize("shapes", [MANY, LARGE, MANY[:23], MANY[:24], LARGE[:1]])
@pytest.mark.parametrize("centered,x64", [(False, False), (True, True)])
def test_uneven(shapes, centered, x64):
    ctx = dfl.dfisher_ctx_create(0)
    Ss, vs = make(shapes)
    lams = [0.1 * 1.1 ** (k % 9) for k in range(len(shapes))]
    kw = dict(gram_prec=dfl.DFISHER_GRAM_MXFP8, sweeps=-1, centered=centered, x_fp64=x64)
    xs, infos = dfl.dfisher_solve_uneven(ctx, Ss, vs, lams, **kw)
    again, _ = dfl.dfisher_solve_uneven(ctx, Ss, vs, lams, **kw)
    for S, v, lam, x, a, info in zip(Ss, vs, lams, xs, again, infos):
        assert info["potrf_info"] == 0
        assert torch.equal(x, a)
        r = reference(S, v, lam)
        # the library's refinement target (1e-7), the final correction's image (below it) and FP32 rounding of x
        assert float((x.double() - r).norm() / r.norm()) <= 1e-6, (S.shape, lam)
    ctx.close()
