"""The error indicator after a load update that changed the number of loads, in a medium
without equal elements (whose elements keep the loads as columns beside B): equal to that
of a context set up with the new load, bit for bit (the same operations on the same
data, whatever was planned before)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first,then", [(3, 1), (1, 3)])
def test_indicator_after_other_number_of_loads(first, then):
    from paper_2304_01728_amd import dpgmg as D
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    N, p = 4, 2
    rng = np.random.default_rng(3)
    c = 1.0 + rng.random(N ** 3)
    dirs = rng.standard_normal((6, 3))
    loads = [dict(dir=d / np.linalg.norm(d), amp=1.0) for d in dirs]
    old, new = loads[:first], loads[3:3 + then]
    print(f"[indicator] N={N} p={p} {first} loads, then {then}", flush=True)

    def context(ld):
        ctx = D.dpg_setup(N, p, 2 * np.pi, ld, c=c, options=D.dpg_default_options())
        D.dpg_assemble(ctx)
        D.dpg_build_hierarchy(ctx)
        return ctx

    ctx, ref = context(old), context(new)
    x = D.dpg_solve(ctx, nrhs=1, tol=1e-10)[0]
    D.dpg_error_indicator(ctx, x)
    D.dpg_load_rhs(ctx, new, want=False)
    y = D.dpg_solve(ref, nrhs=1, tol=1e-10)[0]
    got, want = D.dpg_error_indicator(ctx, y), D.dpg_error_indicator(ref, y)
    ctx.close()
    ref.close()
    assert np.array_equal(got, want)
