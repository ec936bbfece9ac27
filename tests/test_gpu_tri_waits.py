"""A wait of the triangular solves that gives up (here: at the first value that is not there yet) is reported, once, by the call
itself where it synchronises afterwards and else by the next one that does."""
import pytest
import torch

import paper_2310_17556_amd as dfl

pytestmark = pytest.mark.gpu
N, M = 1000, 3000   # eight blocks in a chain
KW = dict(gram_prec=dfl.DFISHER_GRAM_FP32, sweeps=1, shift_policy=dfl.DFISHER_SHIFT_NONE)


@pytest.fixture
def case():
    ctx = dfl.dfisher_ctx_create(0)
    g = torch.Generator(device="cuda").manual_seed(3)
    S = torch.randn(N, M, device="cuda", generator=g) / M ** 0.5
    v = torch.randn(M, device="cuda", generator=g)
    x, _ = dfl.dfisher_solve(ctx, S, v, 0.1, **KW)
    yield ctx, S, v, x
    torch.cuda.synchronize()
    ctx.close()


def gives_up(call):
    with pytest.raises(dfl.DfisherError) as e:
        call()
    assert e.value.status == dfl.DFISHER_E_DEVICE and "gave up" in str(e.value)


def fine(ctx, S, v, x):
    assert torch.equal(dfl.dfisher_solve(ctx, S, v, 0.1, **KW)[0], x)


def test_solve(case, monkeypatch):
    ctx, S, v, x = case
    monkeypatch.setenv("DFISHER_TRI_SPIN", "0")
    gives_up(lambda: dfl.dfisher_solve(ctx, S, v, 0.1, **KW))
    monkeypatch.delenv("DFISHER_TRI_SPIN")
    torch.cuda.synchronize()
    fine(ctx, S, v, x)


def test_uneven(case, monkeypatch):
    ctx, S, v, x = case
    call = lambda: dfl.dfisher_solve_uneven(ctx, [S, S[:300]], [v, v], [0.1, 0.1], **KW)
    dfl.dfisher_ctx_enable_graphs(ctx, False)
    monkeypatch.setenv("DFISHER_TRI_SPIN", "0")
    gives_up(call)
    monkeypatch.delenv("DFISHER_TRI_SPIN")
    torch.cuda.synchronize()
    call()
    fine(ctx, S, v, x)


@pytest.mark.parametrize("nrhs", [1, 3])
def test_later(case, monkeypatch, nrhs):
    """The kept factor's solves do not synchronise."""
    ctx, S, v, x = case
    f, _ = dfl.dfisher_factor_create(ctx, S, 0.1, **KW)
    V = v.repeat(nrhs, 1)
    monkeypatch.setenv("DFISHER_TRI_SPIN", "0")
    X = dfl.dfisher_factor_solve(f, V)
    X = X[0] if isinstance(X, tuple) else X
    assert bool(torch.isnan(X).any())
    monkeypatch.delenv("DFISHER_TRI_SPIN")
    gives_up(lambda: dfl.dfisher_solve(ctx, S, v, 0.1, **KW))
    torch.cuda.synchronize()
    fine(ctx, S, v, x)
    f.close()


def test_enqueue_only(case, monkeypatch):
    ctx, S, v, x = case
    call = lambda: dfl.dfisher_solve_batched(ctx, S, [0.1, 0.2], v[None], enqueue_only=True, **KW)[1]

    def statuses(infos):
        torch.cuda.synchronize()
        return [i["potrf_info"] for i in dfl.batch_infos(infos)]

    monkeypatch.setenv("DFISHER_TRI_SPIN", "0")
    lost = call()
    monkeypatch.delenv("DFISHER_TRI_SPIN")
    good = call()
    assert statuses(lost) == [-1, -1] and statuses(good) == [0, 0]
    fine(ctx, S, v, x)
