"""Calls after one that ended with DPG_ENOMEM under a memory budget: they are refused or
give what they give on a context on which nothing failed, bit for bit.

Each budget is taken from a context with a very large one that goes through the same
calls, so that the call named by the test, and nothing before it, passes it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _D():
    from paper_2304_01728_amd import dpgmg as D
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return D


def _loads(n):
    rng = np.random.default_rng(5)
    return [dict(dir=d / np.linalg.norm(d), amp=1.0) for d in rng.standard_normal((n, 3))]


def _ctx(D, N, p, c, loads, budget=int(200e9), **kw):
    print(f"[after enomem] N={N} p={p} loads={len(loads)} budget={budget} {kw}", flush=True)
    opt = D.dpg_default_options(nu_pre=2, nu_post=2, hbm_budget=budget, **kw)
    ctx = D.dpg_setup(N, p, 2 * np.pi * N / 5, loads, c=c, options=opt)
    D.dpg_assemble(ctx)
    D.dpg_build_hierarchy(ctx)
    return ctx


def _resident(D, ctx):
    return int(D.dpg_info(ctx).resident_bytes)


def _refused(D, code, f, *a, **kw):
    with pytest.raises(D.DPGError) as e:
        f(*a, **kw)
    assert e.value.code == code


def test_setup_after_failed_release():
    """The load maps do not fit: the work areas are gone all the same, and assembly and
    hierarchy are refused (they ran on freed memory); solves go on."""
    D = _D()
    c = 1.0 + np.random.default_rng(1).random(8)
    ctx = _ctx(D, 2, 2, c, _loads(1))
    budget = _resident(D, ctx)
    ctx.close()
    ctx = _ctx(D, 2, 2, c, _loads(1), budget)
    x = D.dpg_solve(ctx, tol=1e-10)[0]
    _refused(D, D.DPG_ENOMEM, D.dpg_release_setup, ctx)
    _refused(D, D.DPG_ESTATE, D.dpg_assemble, ctx)
    _refused(D, D.DPG_ESTATE, D.dpg_build_hierarchy, ctx)
    y = D.dpg_solve(ctx, tol=1e-10)[0]
    ctx.close()
    assert np.array_equal(x, y)


@pytest.mark.parametrize("shared", [False, True])
def test_loads_after_failed_element_plan(shared):
    """A load update with many loads that does not fit the element stage's work areas,
    then one with as many loads as before: planned anew, not taken for the plan that the
    failed one replaced.  Media of more than 512 kinds of elements, whose load updates go
    through the element stage: all elements different, or half of them equal."""
    D = _D()
    N, p, many = 12, 1, 48
    rng = np.random.default_rng(2)
    c = 1.0 + rng.random(N ** 3)
    if shared:
        c[rng.random(N ** 3) < 0.5] = 1.0
    one, other, more = _loads(1), _loads(3)[2:], _loads(many)
    ctx = _ctx(D, N, p, c, one)
    before = _resident(D, ctx)
    D.dpg_load_rhs(ctx, more)
    after = _resident(D, ctx)
    want = D.dpg_load_rhs(ctx, other)
    ctx.close()
    # the work areas are the last allocations of the update
    ctx = _ctx(D, N, p, c, one, after - 4096)
    print(f"  resident {before}, with {many} loads {after}", flush=True)
    _refused(D, D.DPG_ENOMEM, D.dpg_load_rhs, ctx, more)
    got = D.dpg_load_rhs(ctx, other)
    x, it, rr, code = D.dpg_solve(ctx, tol=1e-8)
    ctx.close()
    assert np.array_equal(got, want) and code == D.DPG_OK


@pytest.mark.parametrize("flags,precision", [(0, "fp64"), (0, "mixed"), (8, "fp64")])
def test_solves_after_a_block_solve_that_does_not_fit(flags, precision):
    """32 columns that do not fit, in the middle of the block vectors: solves of one and two
    columns, and a batch of two, go on as before (recomputed patches share a buffer between
    block and single-column solves)."""
    D = _D()
    N, p = 4, 2
    kw = dict(flags=flags, precision=D.DPG_MIXED if precision == "mixed" else D.DPG_FP64)
    ctx = _ctx(D, N, p, None, _loads(1), **kw)
    n = D.dpg_info(ctx).n_trace
    rng = np.random.default_rng(8)
    b = rng.standard_normal((32, n)) + 1j * rng.standard_normal((32, n))
    x2 = D.dpg_solve(ctx, rhs=b[:2], nrhs=2, tol=1e-8)[0]
    small = _resident(D, ctx)
    D.dpg_solve(ctx, rhs=b, nrhs=32, tol=1e-8)
    large = _resident(D, ctx)
    ctx.close()
    for budget in (small + (large - small) // 4, (small + large) // 2, large - 4096):
        ctx = _ctx(D, N, p, None, _loads(1), budget, **kw)
        x1 = D.dpg_solve(ctx, rhs=b[:1], nrhs=1, tol=1e-8)[0]
        assert np.array_equal(D.dpg_solve(ctx, rhs=b[:2], nrhs=2, tol=1e-8)[0], x2)
        _refused(D, D.DPG_ENOMEM, D.dpg_solve, ctx, rhs=b, nrhs=32, tol=1e-8)
        assert np.array_equal(D.dpg_solve(ctx, rhs=b[:1], nrhs=1, tol=1e-8)[0], x1)
        assert np.array_equal(D.dpg_solve(ctx, rhs=b[:2], nrhs=2, tol=1e-8)[0], x2)
        _refused(D, D.DPG_ENOMEM, D.dpg_batch_open, ctx, 32)
        _refused(D, D.DPG_ESTATE, D.dpg_batch_step, ctx, 1)
        D.dpg_batch_open(ctx, 2)
        assert D.dpg_batch_add(ctx, b[0], tol=1e-8) == 0
        assert D.dpg_batch_step(ctx, 200) == [0]
        y = D.dpg_batch_take(ctx, 0)[0]
        assert np.linalg.norm(y - x1[0]) <= 1e-6 * np.linalg.norm(x1[0])
        ctx.close()


def test_solves_after_a_load_update_that_failed():
    """Refused loads (a source of no width) leave the loads before in place, with their
    number; loads that do not fit leave none, and the next update goes on as on a context
    on which nothing failed."""
    D = _D()
    N, p = 6, 2
    one, other, more = _loads(1), _loads(3)[2:], _loads(256)
    bad = more[:7] + [dict(amp=0.0, sources=[[0.5, 0.5, 0.5, 0.0, 1.0, 0.0]])]
    ctx = _ctx(D, N, p, None, one)
    x = D.dpg_solve(ctx, tol=1e-8)[0]
    want = D.dpg_load_rhs(ctx, other)
    y = D.dpg_solve(ctx, tol=1e-8)[0]
    small = _resident(D, ctx)
    D.dpg_load_rhs(ctx, more)
    large = _resident(D, ctx)
    ctx.close()
    through = 0
    for budget in (small + 4096, (small + large) // 2, large - 4096):
        ctx = _ctx(D, N, p, None, one, budget)
        _refused(D, D.DPG_EINVAL, D.dpg_load_rhs, ctx, bad)
        _refused(D, D.DPG_EINVAL, D.dpg_solve, ctx, nrhs=8, tol=1e-8)
        assert np.array_equal(D.dpg_solve(ctx, tol=1e-8)[0], x)
        try:
            D.dpg_load_rhs(ctx, other)   # builds the class maps, whose work areas may not fit
        except D.DPGError as e:
            assert e.code == D.DPG_ENOMEM
            ctx.close()
            continue
        _refused(D, D.DPG_ENOMEM, D.dpg_load_rhs, ctx, more)
        for call, kw in ((D.dpg_solve, dict(nrhs=1)), (D.dpg_solve_noalloc, dict(nrhs=1))):
            _refused(D, D.DPG_EINVAL, call, ctx, tol=1e-8, **kw)
        _refused(D, D.DPG_EINVAL, D.dpg_get_fields, ctx, x)
        assert np.array_equal(D.dpg_load_rhs(ctx, other), want)
        assert np.array_equal(D.dpg_solve(ctx, tol=1e-8)[0], y)
        ctx.close()
        through += 1
    assert through >= 1
