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


def sized(tmp_path, n, call):
    """A context whose held workspace just fits `call` of a longer problem with the base plan's slices (see test_base_plan)."""
    ctx = dfl.dfisher_ctx_create(0)
    f = tmp_path / "tune"
    f.write_text("".join(f"{prec} 1 17 {al} 4 0\n" for prec in (0, 1) for al in (0, 1)))
    dfl.dfisher_ctx_load_tuning(ctx, str(f))
    call(ctx, 131072)
    return ctx, hold(ctx)


@pytest.mark.parametrize("what", ["solve", "rowspace", "factor", "gram"])
def test_base_plan(tmp_path, what):
    """n = 64, m = 70000: the plan takes more than 200 slices; the workspace holds the base plan's 32."""
    n = 64
    gen = torch.Generator(device="cuda").manual_seed(1)
    big = torch.randn(n, 131072, device="cuda", generator=gen) / 131072 ** 0.5
    v = torch.randn(1, 131072, device="cuda", generator=gen)
    f = torch.randn(n, device="cuda", dtype=torch.float64, generator=gen)
    kw = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=4, x_fp64=True)

    def call(ctx, m):
        S, V = big[:, :m].contiguous(), v[:, :m].contiguous()
        if what == "solve":
            return dfl.dfisher_solve(ctx, S, V[0], 0.1, **kw)[0]
        if what == "rowspace":
            return dfl.dfisher_solve_rowspace(ctx, S, f, 0.1, **kw)[0]
        if what == "gram":
            return dfl.dfisher_gram(ctx, S, dfl.DFISHER_GRAM_FP32, 0.1)
        fac, _ = dfl.dfisher_factor_create(ctx, S, 0.1, **kw)
        L = dfl.dfisher_factor_copy_L(fac)
        fac.close()
        return L

    held, graph = sized(tmp_path, n, call)
    got = call(held, 70000)
    free = dfl.dfisher_ctx_create(0)
    want = call(free, 70000)
    # solves: four refinement sweeps from either Gram end at FP64 rounding; Gram and factor: FP32 sums of a slice
    tol = 1e-5 if what in ("gram", "factor") else 1e-11
    assert float((got - want).abs().max() / want.abs().max()) <= tol
    del graph
    held.close()
    free.close()


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


@pytest.mark.parametrize("what,m", [("batched", 23000), ("factor", 60000)])
def test_two_groups_a_pass(what, m):
    """64 vectors on a workspace that the call for 32 vectors, or the factor, of a problem with m = 24000 left: two groups of 16 a
    pass instead of four."""
    n = 64
    gen = torch.Generator(device="cuda").manual_seed(4)
    big, V = torch.randn(n, 60000, device="cuda", generator=gen) / 200, torch.randn(64, 60000, device="cuda", generator=gen)
    kw = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=4, shift_policy=dfl.DFISHER_SHIFT_NONE, x_fp64=True)

    def prepare(ctx, m, nrhs):
        S, W = big[:, :m].contiguous(), V[:nrhs, :m].contiguous()
        if what == "batched":
            return lambda: dfl.dfisher_solve_batched(ctx, S, [0.1, 0.2][:max(1, nrhs // 32)], W[:32], **kw)[0]
        f, _ = dfl.dfisher_factor_create(ctx, S, 0.1, **kw)
        return lambda: dfl.dfisher_factor_solve(f, W)

    held, free = dfl.dfisher_ctx_create(0), dfl.dfisher_ctx_create(0)
    prepare(held, 24000, 32)()
    graph = hold(held)
    X = []
    for ctx, groups in ((held, 2), (free, 4)):
        call = prepare(ctx, m, 64)
        ran = kernels(lambda: X.append(call()))
        assert f"rowpass_multi_tm_kernel<{groups}, false>" in ran and f"rowpass_multi_tm_kernel<{6 - groups}, false>" not in ran
    a, b = (x[0] if isinstance(x, tuple) else x for x in X)
    assert float((a - b).abs().max() / b.abs().max()) <= 1e-11   # four sweeps end at FP64 rounding, in either order of the sums
    del graph


def test_uneven_in_place(tmp_path):
    """The packed copy of a factor of 1000 rows (4 MB) does not fit a workspace sized for a shorter problem."""
    f = tmp_path / "tune"
    f.write_text("0 4 17 1 1 -1\n0 4 18 1 1 -1\n")   # (the same slices for both lengths)
    S = torch.randn(1000, 400000, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5)) / 400000 ** 0.5
    v = torch.randn(400000, device="cuda")
    kw = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=3, x_fp64=True)
    xs, names = [], []
    for held in (True, False):
        ctx = dfl.dfisher_ctx_create(0)
        dfl.dfisher_ctx_enable_graphs(ctx, False)
        dfl.dfisher_ctx_load_tuning(ctx, str(f))
        if held:
            dfl.dfisher_solve_uneven(ctx, [S[:, :200000].contiguous()], [v[:200000].contiguous()], [0.1], **kw)
            graph = hold(ctx)
        names.append(kernels(lambda: xs.append(dfl.dfisher_solve_uneven(ctx, [S], [v], [0.1], **kw)[0][0])))
    assert "potf2_kernel" in names[0] and "mirror_kernel" in names[0] and "chol_kernel" not in names[0]
    assert "chol_kernel" in names[1] and "potf2_kernel" not in names[1]
    assert float((xs[0] - xs[1]).abs().max() / xs[1].abs().max()) <= 1e-11
    del graph
