"""S as the last columns of a wider matrix, whose storage ends with S's last element: the same bits as from a copy of S."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


# odd widths (the last block of 32 or 128 columns is partial) at 8, 16, 32 rows a lane and more than 2048 rows
@pytest.mark.parametrize("n,m,c", [(17, 1001, 3), (64, 4099, 1), (513, 2050, 37), (1025, 4127, 128), (2049, 8193, 5)])
def test_last_columns(n, m, c):
    ctx = dfl.dfisher_ctx_create(0)
    g = torch.Generator(device="cuda").manual_seed(n)
    big = torch.randn(n, c + m, device="cuda", generator=g) / n ** 0.5
    S = big[:, c:]
    copy = S.contiguous()
    V = torch.randn(5, m, device="cuda", generator=g)
    kw = dict(gram_prec=dfl.DFISHER_GRAM_BF16X3, sweeps=2)
    got = []
    for A in (S, copy):
        x, _ = dfl.dfisher_solve(ctx, A, V[0], 1e-2, **kw)
        f, _ = dfl.dfisher_factor_create(ctx, A, 1e-2, **kw)
        X = dfl.dfisher_factor_solve(f, V)
        got.append((x, X[0] if isinstance(X, tuple) else X))
        f.close()
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    ctx.close()
