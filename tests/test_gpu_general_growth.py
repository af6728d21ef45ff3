"""General matrices whose factorisation without pivoting grows: transport by
central differences with little diffusion on a graded mesh, whose diagonal is
small against the neighbours.  Every pivot passes against its diagonal entry,
so the recurrences are used; their backward error is the pivots' size against
their rows times a few roundings."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle.spatial import spatial_matrices

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def transport(n, e):
    t = np.linspace(0.0, 1.0, n + 2)
    h = np.diff(t + 0.5 * (t * t - t))
    w = (h[:-1] + h[1:]) / 2
    lo, up = -e / h[:-1] / w - 0.5 / w, -e / h[1:] / w + 0.5 / w
    lo[0] = up[-1] = 0.0
    return lo, e * (1.0 / h[:-1] + 1.0 / h[1:]) / w, up


def pivots(K, tau, lam):
    """Growth of the recurrence: the largest pivot against its row, and the
    smallest against its diagonal entry."""
    a, b, c = tau * K[0], lam + tau * K[1], tau * K[2]
    d, out = b[0], [b[0]]
    for i in range(1, len(b)):
        d = b[i] - a[i] * c[i - 1] / d
        out.append(d)
    out = np.abs(out)
    return (out / np.maximum(np.maximum(np.abs(a), np.abs(b)), np.abs(c))).max(), (out / np.abs(b)).min()


def backward_errors(lib, n, ell, K):
    tau, F2 = 1.0 / ell, ell // 2 + 1
    rng = np.random.default_rng(n)
    H = rng.standard_normal((F2, n)) + 1j * rng.standard_normal((F2, n))
    plan = lib.paradiag_plan_create(n, ell, tau, None, K, stream=torch.cuda.current_stream().cuda_stream)
    try:
        Y = torch.empty((F2, n), dtype=torch.complex128, device="cuda:0")
        lib.paradiag_shifted_solve(plan, torch.tensor(H, device="cuda:0"), None, Y, None)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    _, Ksp = spatial_matrices(None, K, 1)
    Yn, out = Y.cpu().numpy(), []
    for k in range(F2):
        P = sp.csr_matrix((1.0 - np.exp(-2j * np.pi * k / ell)) * sp.eye(n) + tau * Ksp)
        scale = abs(P) @ np.abs(Yn[k]) + np.abs(H[k])
        out.append(np.max(np.abs(P @ Yn[k] - H[k])) / np.max(scale))
    return max(out)


@pytest.mark.parametrize("n,ell,e", [(200, 16, 1e-7), (200, 16, 1e-5), (1000, 16, 1e-7), (1000, 64, 1e-2)])
def test_growth(lib, n, ell, e):
    K = transport(n, e)
    growth, least = pivots(K, 1.0 / ell, 0.0)
    assert least >= 1.0 / 16 and (growth > 16) == (e < 1e-3)
    # a pivot's and its product's rounding, of the pivot's size, beside what every
    # solve has
    assert backward_errors(lib, n, ell, K) < (24 * 8 + 4 * growth) * 2.2e-16
