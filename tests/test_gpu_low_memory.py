"""Calls whose preferred layout there is no memory for: the smaller one runs, gives the same answer, and is not looked for anew by
the next call."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu


def hold(ctx):
    """Captures a small call: from here on the workspace of ctx stays what it is."""
    S, V = torch.randn(8, 64, device="cuda"), torch.randn(1, 64, device="cuda")
    kw = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=0, shift_policy=dfl.DFISHER_SHIFT_NONE)
    X, _ = dfl.dfisher_solve_batched(ctx, S, [1.0], V, **kw)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dfl.dfisher_solve_batched(ctx, S, [1.0], V, X=X, enqueue_only=True, **kw)
    return g


def kernels(call):
    """The names of the kernels that a call runs."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.key for e in p.key_averages())


@pytest.mark.parametrize("n", [1000, 1500])   # the packed copy takes 4 and 10 MB, the held workspace 1
def test_cholesky_in_place(n):
    a, b = dfl.dfisher_ctx_create(0), dfl.dfisher_ctx_create(0)
    g = hold(a)
    M = torch.randn(n, n, device="cuda", dtype=torch.float64, generator=torch.Generator(device="cuda").manual_seed(n))
    W = M @ M.T.contiguous() / n + torch.eye(n, dtype=torch.float64, device="cuda")
    A, B = W.clone(), W.clone()
    ran = kernels(lambda: dfl.dfisher_potrf(a, A))
    assert "potf2_kernel" in ran and "chol_kernel" not in ran
    ran = kernels(lambda: dfl.dfisher_potrf(b, B))
    assert "chol_kernel" in ran and "potf2_kernel" not in ran
    for L in (A, B):   # backward stable: n eps |W|, whatever the order of the sums
        assert float((L @ L.T.contiguous() - W).abs().max()) <= 4 * n * 2.0 ** -53 * float(W.abs().max())
    del g
    a.close()
    b.close()


def test_planes_do_not_fit():
    """Little free memory (not a held workspace): rows that are not 16-byte aligned go without planes, twice alike."""
    n, m = 64, (1 << 24) + 1   # 4 GB, and as much for the planes
    S = torch.empty(n, m, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(2))
    ctx = dfl.dfisher_ctx_create(0)
    small = S[:8, :4096]
    dfl.dfisher_gram(ctx, small, dfl.DFISHER_GRAM_BF16X3, 0.5)   # (code and scratch are there before the memory goes)
    W = torch.empty(n, n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    hog = torch.empty(max(0, free - (3 << 30)), dtype=torch.uint8, device="cuda")
    ran = []
    for _ in range(2):
        ran.append(kernels(lambda: W.copy_(dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_BF16X3, 0.5))))
        left = torch.cuda.mem_get_info()[0]
    assert all("gram_kernel_split" not in r and "gram_kernel<1" in r for r in ran)
    one = W.clone()
    dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_BF16X3, 0.5)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == left
    del hog
    torch.cuda.empty_cache()
    got = dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_BF16X3, 0.5)
    assert "gram_kernel_split" in kernels(lambda: dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_BF16X3, 0.5))
    assert float((got - one).abs().max() / one.abs().max()) <= 3e-5   # dropped lo.lo products
    ctx.close()
