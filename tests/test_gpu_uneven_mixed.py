"""An uneven call whose column passes partly share a launch and partly go alone, against dense FP64 solves."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(8, 2200001), (1500, 3001), (3, 70)],        # 1500 rows: alone
                                    [(700, 2001), (8, 1100001), (9, 1100003)],
                                    [(8, 1000), (30, 5001)]])                      # too few blocks: each alone
@pytest.mark.parametrize("x64", [False, True])
def test_uneven(shapes, x64):
    ctx = dfl.dfisher_ctx_create(0)
    g = torch.Generator(device="cuda").manual_seed(5)
    Ss = [torch.randn(n, m, device="cuda", generator=g) / m ** 0.5 for n, m in shapes]
    vs = [torch.randn(m, device="cuda", generator=g) for _, m in shapes]
    lams = [0.5] * len(shapes)   # (S S^T is near the identity or, for m near n, of norm 3: condition < 10)
    xs, infos = dfl.dfisher_solve_uneven(ctx, Ss, vs, lams, gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=3, x_fp64=x64)
    for S, v, lam, x, info in zip(Ss, vs, lams, xs, infos):
        assert info["potrf_info"] == 0
        D, b = S.double(), v.double()
        W = D @ D.T.contiguous() + lam * torch.eye(len(D), dtype=torch.float64, device="cuda")
        r = (b - D.T.contiguous() @ torch.linalg.solve(W, D @ b)) / lam
        # three sweeps from an FP32 Gram end at FP64 rounding; x in FP32 is rounded once
        assert float((x.double() - r).norm() / r.norm()) <= (1e-12 if x64 else 1e-7), S.shape
    ctx.close()
