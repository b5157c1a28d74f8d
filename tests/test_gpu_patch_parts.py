"""Patch factorisations in one part per level, on alternating streams (little
patch work), against the four parts of a level that a memory budget keeps: the
same arithmetic, so the same bits, on meshes with one to three patch levels,
equal and different patches, and after a second build in the same context."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,p,varying,precision", [
    (4, 1, False, "fp64"), (8, 2, False, "fp64"), (6, 3, True, "fp64"), (16, 1, True, "mixed"),
    (8, 2, True, "mixed")])
def test_parts_of_patch_work(N, p, varying, precision):
    from paper_2304_01728_amd import dpgmg as D
    rng = np.random.default_rng(23)
    c = 1.0 + rng.uniform(0.0, 0.4, N ** 3) if varying else None
    print(f"[parts] N={N} p={p} varying={varying} {precision}", flush=True)
    got = []
    for budget in (0, 200 << 30):
        opt = D.dpg_default_options(nu_pre=2, nu_post=2, hbm_budget=budget,
                                    precision=D.DPG_MIXED if precision == "mixed" else D.DPG_FP64)
        ctx = D.dpg_setup(N, p, 2 * np.pi * N / 5, [dict(dir=[0, 0.6, 0.8], amp=1.0)], c=c,
                          options=opt)
        for _ in range(2):
            D.dpg_assemble(ctx)
            D.dpg_build_hierarchy(ctx)
            got.append(D.dpg_solve(ctx, tol=1e-8)[0])
        ctx.close()
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0
    for x in got[1:]:
        assert np.array_equal(got[0], x)
