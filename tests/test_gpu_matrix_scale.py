"""Matrices of any scale: M and K times a power of two have the same solution, and
the arithmetic is that of scaled numbers, so the results agree to a few
roundings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def solve(lib, n, ell, M, K, scale, **kw):
    s = kw.get("bdf_order", 1)
    x = np.arange(1, n + 1) / (n + 1)
    u0 = np.sin(np.pi * x) + 0.3 * np.sin(2 * np.pi * x)
    F = np.cos(np.arange(ell) / ell)[:, None] * np.sin(3 * np.pi * x)
    u0 = torch.tensor(np.repeat(u0[None], s, axis=0) if s > 1 else u0, device="cuda:0")
    F = torch.tensor(F, device="cuda:0")
    U = torch.zeros_like(F)
    plan = lib.paradiag_plan_create(n, ell, 1.0 / ell, *(tuple(scale * a for a in A) for A in (M, K)),
                                    stream=torch.cuda.current_stream().cuda_stream, **kw)
    try:
        lib.paradiag_solve(plan, u0, F, U, 1e-10)
        return U.cpu().numpy()
    finally:
        lib.paradiag_plan_destroy(plan)


def fem(n, nu):
    h = 1.0 / (n + 1)
    row = lambda o, d: (np.full(n, o), np.full(n, d), np.full(n, o))
    return row(h / 6, 4 * h / 6), row(-nu / h, 2 * nu / h)


@pytest.mark.parametrize("n,ell,nu,kw", [(300, 64, 1.0, {}), (300, 64, 1e-3, {}), (4095, 32, 1e-3, {}),
                                         (300, 64, 1e-2, dict(alpha=0.1)), (300, 64, 1e-3, dict(bdf_order=2)),
                                         (511, 32, 1e-2, dict(bdf_order=3))])
def test_uniform(lib, n, ell, nu, kw):
    M, K = fem(n, nu)
    ref = solve(lib, n, ell, M, K, 1.0, **kw)
    for e in (-800, -520, -490, 300, 490, 520, 800):
        U = solve(lib, n, ell, M, K, 2.0**e, **kw)
        assert np.linalg.norm(U - ref) <= 8 * 2.0**-53 * np.linalg.norm(ref), e


def graded(n, nu):
    t = np.linspace(0.0, 1.0, n + 2)
    h = np.diff(t - 0.5 * np.sin(2 * np.pi * t) / (2 * np.pi))
    M = (h[:-1] / 6, (h[:-1] + h[1:]) / 3, h[1:] / 6)
    return M, (-nu / h[:-1], nu / h[:-1] + nu / h[1:], -nu / h[1:])


# Scales of the recurrences (2^-290, 2^290) and beyond them, where the partition
# form runs: there the two forms' rounding, at most 40 u times the condition number
# of P_0, about n^2, stands between the results.
@pytest.mark.parametrize("n,ell,nu", [(200, 64, 1.0), (200, 64, 1e-3), (1000, 32, 1.0), (3001, 16, 1e-2)])
def test_general(lib, n, ell, nu):
    M, K = graded(n, nu)
    ref = solve(lib, n, ell, M, K, 1.0)
    for e in (-480, -400, -350, -320, -290, 290, 320, 400, 480):
        U = solve(lib, n, ell, M, K, 2.0**e)
        bound = 8 if abs(e) < 300 else 40 * n * n
        assert np.linalg.norm(U - ref) <= bound * 2.0**-53 * np.linalg.norm(ref), e
