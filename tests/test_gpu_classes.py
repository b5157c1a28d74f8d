"""Matrices shared by classes of equal elements, blocks and patches, against
the oracle, which forms every matrix of every level on its own: media in which
few, some and none of the elements are equal, on meshes with even and odd
coarse levels, with Galerkin and stored coarse operators."""
import numpy as np
import pytest

from oracle import dpg, element, multigrid
from paper_2304_01728_amd import workloads
from test_gpu_parity import rel

pytestmark = pytest.mark.gpu


def _speed(medium, N):
    rng = np.random.default_rng(17)
    e = np.arange(N ** 3)
    i, j, k = e % N, e // N % N, e // (N * N)
    if medium == "uniform":
        return np.ones(N ** 3)
    if medium == "halves":              # two half spaces: classes across a plane x = const
        return np.where(i < N // 2, 1.0, 1.75)
    if medium == "layers":              # every coarse element uniform (stored operators too)
        return np.array([1.0, 1.5])[(k // (N // 2)) % 2]
    if medium == "checked":             # two speeds in no regular order
        return rng.choice([1.0, 1.4], N ** 3)
    c = 1.0 + rng.uniform(0.0, 0.5, N ** 3)
    if medium == "pair":                # all different but two
        c[1] = c[2]
    return c


CASES = [(4, 2, "uniform", "fp64", False), (4, 1, "halves", "fp64", False),
         (6, 2, "layers", "fp64", False), (4, 2, "layers", "fp64", True),
         (8, 1, "checked", "fp64", False), (4, 1, "pair", "fp64", False),
         (4, 2, "different", "fp64", False), (8, 1, "layers", "mixed", False)]


@pytest.mark.parametrize("N,p,medium,precision,store", CASES)
def test_class_matrices_and_solutions(N, p, medium, precision, store):
    from paper_2304_01728_amd import dpgmg as D
    import torch
    assert torch.cuda.is_available()
    c = _speed(medium, N)
    omega = 2 * np.pi * c.min() * N / 5
    d = workloads.plane_wave_direction(11)
    loads = [dict(sources=[[0.4, 0.55, 0.6, 0.1, 1.0, 0.5]]), dict(dir=d, amp=1.0)]
    print(f"[classes] N={N} p={p} {medium} {precision} store={store}", flush=True)
    opt = D.dpg_default_options(nu_pre=2, nu_post=2, flags=D.DPG_STORE_COARSE if store else 0,
                                precision=D.DPG_MIXED if precision == "mixed" else D.DPG_FP64)
    ctx = D.dpg_setup(N, p, omega, loads, c=c, options=opt)
    D.dpg_assemble(ctx)
    D.dpg_build_hierarchy(ctx)
    f = dpg.gaussian_sources([[0.4, 0.55, 0.6]], 0.1, [1.0 + 0.5j])

    def u0(X, n):                       # impedance data with Z of the wall element
        e = [np.clip((X[:, a] * N).astype(int), 0, N - 1) for a in range(3)]
        return (1.0 / c[e[0] + N * (e[1] + N * e[2])] - d @ n) * np.exp(-1j * omega * (X @ d))

    pr = dpg.Problem(N, p, omega, [dict(f=f), dict(u0=u0)], kappa=c ** -2, Zel=c)
    S, s, rec = pr.condensed()
    # element matrices: cond(G) times the unit round-off (see test_gpu_parity)
    tol = 1e-12
    for ck in (c.min(), c.max()):
        ev = np.linalg.eigvalsh(element.element_matrices(p, omega, 1.0 / N, kappa=ck ** -2, Z=ck)[0])
        tol = max(tol, ev[-1] / ev[0] * 2.0 ** -53)
    Sg = D.dpg_export(ctx, D.X_ELEM_S).reshape(pr.nel, pr.n_tr, pr.n_tr).transpose(0, 2, 1)
    assert rel(Sg, S) <= tol
    sg = D.dpg_export(ctx, D.X_ELEM_RHS).reshape(2, pr.nel, pr.n_tr)
    for k in range(2):
        assert rel(sg[k], s[:, :, k]) <= tol, k
    def coarse(n):                      # element matrices of a coarser mesh
        r = N // n
        cc = c.reshape(N, N, N)[::r, ::r, ::r].reshape(-1)
        return dpg.Problem(n, p, omega, [], kappa=cc ** -2, Zel=cc).condensed_operator()

    H = multigrid.Hierarchy(N, p, S, nu_pre=2, nu_post=2, coarse=coarse if store else None)
    bound = 1e-11 if precision == "fp64" else 1e-5     # FP32 copies of the inverses
    for lev in range(H.L):
        lv = H.levels[H.L - lev]
        M = D.dpg_export(ctx, D.X_MACRO_M, lev)
        o = 0
        for Mo in lv.Mblocks:
            n = Mo.shape[0]
            assert rel(M[o:o + n * n].reshape(n, n).T, Mo) <= max(1e-12, tol), lev
            o += n * n
        Si = D.dpg_export(ctx, D.X_PATCH_INV, lev)
        o = 0
        for So in lv.Sinv:
            n = So.shape[0]
            assert rel(Si[o:o + n * n].reshape(n, n).T, So) <= max(bound, 10 * tol), lev
            o += n * n
    rhs = dpg.assemble_vector(pr.edofs, s, pr.num.n)
    x, it, rr, code = D.dpg_solve(ctx, nrhs=2, tol=1e-12)
    assert code == D.DPG_OK
    for k in range(2):
        xo, ito, _ = H.solve(rhs[:, k], 1e-12)
        assert np.linalg.norm(x[k] - xo) <= 1e-10 * np.linalg.norm(xo), k
    x1 = D.dpg_solve(ctx, nrhs=1, tol=1e-12)[0]
    assert np.linalg.norm(x1[0] - x[0]) <= 1e-10 * np.linalg.norm(x[0])
    fields = D.dpg_get_fields(ctx, x)
    fo = dpg.recover_fields(rec, pr.edofs, x.T)
    for k in range(2):
        assert rel(fields[k], fo[:, :, k]) <= 1e-10, k
    ref = dpg.error_indicator(pr, x.T, rec)
    for n in (2, 1):                    # also for fewer columns than loads
        eta2 = D.dpg_error_indicator(ctx, x[:n])
        for k in range(n):
            assert np.abs(eta2[k] - ref[:, k]).max() <= 1e-9 * ref[:, k].max(), k
    ctx.close()
