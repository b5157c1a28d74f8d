"""A right-hand side beyond FP32 in a mixed-precision batch: its own column ends with a
breakdown, and what it left in the local vectors' padding does not reach the others when
the batch is laid out for another width, nor the next solve.

The others' solutions are those of a batch without it to the rounding bound of mixed
solves at tol 1e-10 (1e-8; the widths differ), iterations +-1."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("medium,nu", [("uniform", (2, 2)), ("varying", (0, 2))])
def test_nonfinite_column_stays_alone(medium, nu):
    from paper_2304_01728_amd import dpgmg as D
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, p = 6, 2
    rng = np.random.default_rng(4)
    c = 1.0 + rng.random(N ** 3) if medium == "varying" else None
    print(f"[nonfinite] N={N} p={p} {medium} nu={nu} mixed", flush=True)
    opt = D.dpg_default_options(nu_pre=nu[0], nu_post=nu[1], precision=D.DPG_MIXED)
    ctx = D.dpg_setup(N, p, 2 * np.pi * N / 5, [dict(dir=[0, 0.6, 0.8], amp=1.0)], c=c, options=opt)
    D.dpg_assemble(ctx)
    D.dpg_build_hierarchy(ctx)
    n = D.dpg_info(ctx).n_trace
    b = rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))

    def batch(columns):
        out = {}
        D.dpg_batch_open(ctx, 4)
        slots = {D.dpg_batch_add(ctx, v, tol=1e-10): k for k, v in columns}
        while slots:
            for s in D.dpg_batch_step(ctx, 1):
                x, it, rr, code = D.dpg_batch_take(ctx, s)
                out[slots.pop(s)] = (x, it, code)
        D.dpg_batch_close(ctx)
        return out

    want = batch([(0, b[0]), (1, b[1])])
    got = batch([(0, b[0]), (1, b[1]), (2, 1e60 * b[2])])
    again = batch([(0, b[0]), (1, b[1])])
    alone = D.dpg_solve(ctx, rhs=b[:2], nrhs=2, tol=1e-10)
    ctx.close()
    assert got[2][2] == D.DPG_EBREAKDOWN
    for k in range(2):
        for x, it, code in (got[k], again[k], (alone[0][k], int(alone[1][k]), alone[3])):
            assert code == D.DPG_OK and abs(it - want[k][1]) <= 1
            assert np.linalg.norm(x - want[k][0]) <= 1e-8 * np.linalg.norm(want[k][0])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_block_solves_after_one_that_failed(precision):
    """A block solve that is refused (NaN) or breaks down leaves no batch open, and the
    next one gives what it gave before, bit for bit."""
    from paper_2304_01728_amd import dpgmg as D
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, p = 4, 2
    print(f"[nonfinite] N={N} p={p} {precision}", flush=True)
    opt = D.dpg_default_options(precision=D.DPG_MIXED if precision == "mixed" else D.DPG_FP64)
    ctx = D.dpg_setup(N, p, 2 * np.pi, [dict(dir=[0, 0.6, 0.8], amp=1.0)], options=opt)
    D.dpg_assemble(ctx)
    D.dpg_build_hierarchy(ctx)
    n = D.dpg_info(ctx).n_trace
    rng = np.random.default_rng(6)
    b = rng.standard_normal((3, n)) + 1j * rng.standard_normal((3, n))
    x = D.dpg_solve(ctx, rhs=b, nrhs=3, tol=1e-8)[0]
    for scale in [np.nan] + [1e60] * (precision == "mixed"):
        bad = b.copy()
        bad[1] *= scale
        with pytest.raises(D.DPGError) as e:
            D.dpg_solve(ctx, rhs=bad, nrhs=3, tol=1e-8)
        assert e.value.code == (D.DPG_EBREAKDOWN if np.isfinite(scale) else D.DPG_EINVAL)
        assert np.array_equal(D.dpg_solve(ctx, rhs=b, nrhs=3, tol=1e-8)[0], x)
    ctx.close()
