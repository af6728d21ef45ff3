"""Tolerances far below the rounding of the capacitance system: GMRES on a few
coordinates has all of them after as many iterations, and the solution then is
as good as any; such calls end with success, as GMRES on the whole vector does."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def problem(lib, n, ell, nu, dims, **kw):
    h, s = 1.0 / (n + 1), kw.get("bdf_order", 1)
    K = (np.full(n, -nu / h**2), np.full(n, 2 * nu / h**2), np.full(n, -nu / h**2))
    x = np.arange(1, n + 1) * h
    v = np.sin(np.pi * x) + 0.3 * np.sin(2 * np.pi * x) + 0.01 * np.cos(np.arange(n))
    v = np.outer(v, v).ravel() if dims == 2 else v
    u0 = torch.tensor(np.repeat(v[None], s, axis=0) if s > 1 else v, device="cuda:0")
    F = torch.tensor(np.cos(np.arange(ell) / ell)[:, None] * v, device="cuda:0")
    plan = lib.paradiag_plan_create(n, ell, 1.0 / ell, None, K, dims=dims,
                                    stream=torch.cuda.current_stream().cuda_stream, **kw)
    return plan, u0, F


@pytest.mark.parametrize("n,ell,nu,dims,kw", [(63, 32, 1.0, 1, {}), (63, 32, 20.0, 1, {}), (511, 64, 1.0, 1, {}),
                                              (511, 64, 0.3, 1, {}), (300, 64, 1.0, 1, dict(bdf_order=2)),
                                              (63, 32, 1.0, 2, {}), (31, 16, 3.0, 2, {}), (100, 32, 0.5, 2, {})])
def test_solve(lib, n, ell, nu, dims, kw):
    plan, u0, F = problem(lib, n, ell, nu, dims, **kw)
    try:
        ref, U = torch.zeros_like(F), torch.zeros_like(F)
        lib.paradiag_solve(plan, u0, F, ref, 1e-12)
        for tol in (1e-30, 1e-60, 1e-120, 1e-250):
            lib.paradiag_solve(plan, u0, F, U, tol)
            # x differs by what 1e-14 of b leaves, and its rounding
            assert (U - ref).norm() <= 1e-12 * ref.norm(), tol
    finally:
        lib.paradiag_plan_destroy(plan)


def test_batch(lib):
    parts = [problem(lib, n, ell, nu, 1) for n, ell, nu in ((63, 32, 1.0), (511, 64, 1.0), (300, 64, 3.0))]
    try:
        P, u0, F = ([p[i] for p in parts] for i in range(3))
        U, one = [torch.zeros_like(f) for f in F], [torch.zeros_like(f) for f in F]
        lib.paradiag_solve_batch(P, u0, F, U, 1e-100)
        for p, v, f, w, u in zip(P, u0, F, one, U):
            lib.paradiag_solve(p, v, f, w, 1e-100)
            assert torch.equal(u, w)
    finally:
        for p in parts:
            lib.paradiag_plan_destroy(p[0])
