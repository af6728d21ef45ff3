"""Shifted solves of general tridiagonal M and K in float64 by the two
recurrences: group sizes of 64 to 512 threads, full and ragged last chunks,
several systems to a block, nonsymmetric matrices, and matrices whose pivots
are too small, which keep the partition form."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

from oracle import allatonce, bdf
from oracle.spatial import spatial_matrices

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def graded(n, nu, rng):
    """P1 elements on a mesh of (0, 1) graded towards 0 with jitter."""
    t = np.linspace(0.0, 1.0, n + 2)
    x = t + 0.5 * (t * t - t)
    h = np.diff(x) * rng.uniform(0.7, 1.3, n + 1)
    lo, up = np.r_[0.0, h[1:-1]], np.r_[h[1:-1], 0.0]
    il, iu = np.r_[0.0, 1.0 / h[1:-1]], np.r_[1.0 / h[1:-1], 0.0]
    M = (lo / 6.0, (h[:-1] + h[1:]) / 3.0, up / 6.0)
    return M, (-nu * il, nu * (1.0 / h[:-1] + 1.0 / h[1:]), -nu * iu)


def upwind(n, nu, rng):
    """Variable coefficients with a transport term: nonsymmetric, row sums > 0."""
    a, b = rng.uniform(0.5, 1.5, n) * nu * n, rng.uniform(0.5, 1.5, n) * nu * n
    a[0] = b[-1] = 0.0
    return None, (-a, a + b + rng.uniform(0.1, 1.0, n), -2.0 * b * rng.uniform(0.1, 0.5, n))


def pairs(n, nu, rng):
    """Rows in pairs [[q, q s], [q s, q s^2]]: singular blocks, so that the second
    pivot of a pair is a small part of its diagonal entry at small shifts."""
    q = 1e4 * rng.uniform(0.5, 1.5, n)
    d, lo = np.where(np.arange(n) % 2, 0.0, q), np.zeros(n)
    s = 1.5
    lo[1::2] = s * q[0:-1:2][: lo[1::2].size]
    d[1::2] = s * lo[1::2]
    up = np.r_[lo[1:], 0.0]
    return None, (lo, d, up)


@pytest.mark.parametrize("make,n,ell,alpha", [(graded, 5, 8, 1.0), (upwind, 40, 64, 1.0), (graded, 64, 256, 1.0),
                                              (graded, 100, 64, 1.0), (upwind, 256, 32, 0.1), (graded, 200, 4096, 1.0),
                                              (graded, 257, 16, 1.0), (graded, 511, 32, 1.0), (upwind, 512, 64, 1.0),
                                              (graded, 513, 32, 0.1), (upwind, 1000, 16, 1.0),
                                              (graded, 2049, 32, 1.0), (graded, 4096, 16, 1.0),
                                              (pairs, 600, 16, 0.5), (graded, 700, 2048, 1.0)])
def test_general_solves(lib, make, n, ell, alpha):
    rng = np.random.default_rng(n + ell)
    M, K = make(n, 0.3, rng)
    tau = 1.0 / ell
    Msp, Ksp = spatial_matrices(M, K, 1)
    x = np.linspace(0.0, 1.0, n + 2)[1:-1]
    u0 = np.sin(np.pi * x) + 0.2 * np.sin(5 * np.pi * x)
    F = rng.uniform(-1, 1, (ell, 1)) * np.sin(2 * np.pi * x)
    dev = torch.device("cuda:0")
    F2 = ell // 2 + 1
    H = rng.standard_normal((F2, n)) + 1j * rng.standard_normal((F2, n))
    v = rng.standard_normal(n)
    plan = lib.paradiag_plan_create(n, ell, tau, M, K, alpha=alpha, check_residual=1,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n), dtype=torch.float64, device=dev)
        info = lib.paradiag_solve(plan, torch.tensor(u0, device=dev), torch.tensor(F, device=dev), U, 1e-12)
        Y = torch.empty((F2, n), dtype=torch.complex128, device=dev)
        b = torch.empty(n, dtype=torch.float64, device=dev)
        Jv = torch.empty(n, dtype=torch.float64, device=dev)
        lib.paradiag_shifted_solve(plan, torch.tensor(H, device=dev), torch.tensor(v, device=dev), Y, b)
        lib.paradiag_capacitance_apply(plan, torch.tensor(v, device=dev), Jv)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    Yn, w = Y.cpu().numpy(), alpha ** (1.0 / ell)
    bref, Jref, worst, cond = np.zeros(n), v.copy(), 0.0, 0.0
    for k in range(F2):
        lam = 1.0 - w * np.exp(-2j * np.pi * k / ell)
        P = sp.csc_matrix(lam * Msp + tau * Ksp)
        R = np.stack([Msp @ (H[k] - w * v), Msp @ H[k], Msp @ v.astype(complex)], axis=1)
        lu = spla.splu(P)
        S = lu.solve(R)
        if k in (0, 1, ell // 2):
            inv = spla.LinearOperator((n, n), matvec=lambda z: lu.solve(z.astype(complex)),
                                      rmatvec=lambda z: lu.solve(z.astype(complex), "H"), dtype=complex)
            cond = max(cond, abs(P).sum(axis=0).max() * spla.onenormest(inv))
        # each solver's backward error: eps times a small constant (24 eps here,
        # with pivots down to 1/16 of their diagonal entries)
        y = Yn[k]
        scale = abs(P) @ np.abs(y) + np.abs(R[:, 0])
        worst = max(worst, np.max(np.abs(P @ y - R[:, 0])) / np.max(scale))
        g = (1.0 if k in (0, ell // 2) else 2.0) * np.exp(2j * np.pi * k / ell).conj() / ell
        bref += (g * S[:, 1]).real
        Jref += w * (g * S[:, 2]).real
    assert worst < 24 * 2.2e-16 * 8
    # two backward stable solvers: 2 backward errors times the condition number
    tol = 48 * 2.2e-16 * cond
    assert np.linalg.norm(b.cpu().numpy() - bref) < tol * np.linalg.norm(bref)
    assert np.linalg.norm(Jv.cpu().numpy() - Jref) < tol * np.linalg.norm(Jref)
    ref = allatonce.step_1d(M, K, tau, u0, F)
    assert allatonce.rel_err(U.cpu().numpy(), ref) < 1e-9
    assert 0 <= info.rel_residual < 1e-9


def test_general_bdf(lib):
    n, ell, s = 900, 32, 3
    rng = np.random.default_rng(3)
    M, K = graded(n, 0.3, rng)
    tau = 1.0 / ell
    Msp, Ksp = spatial_matrices(M, K, 1)
    x = np.linspace(0.0, 1.0, n + 2)[1:-1]
    U0 = np.stack([(1 + 0.1 * j) * np.sin(np.pi * x) for j in range(s)])
    F = rng.uniform(-1, 1, (ell, 1)) * np.sin(2 * np.pi * x)
    dev = torch.device("cuda:0")
    plan = lib.paradiag_plan_create(n, ell, tau, M, K, bdf_order=s,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n), dtype=torch.float64, device=dev)
        lib.paradiag_solve(plan, torch.tensor(U0, device=dev), torch.tensor(F, device=dev), U, 1e-11)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    assert allatonce.rel_err(U.cpu().numpy(), bdf.step_bdf(Msp, Ksp, tau, s, list(U0), F)) < 4e-9
