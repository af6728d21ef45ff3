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
