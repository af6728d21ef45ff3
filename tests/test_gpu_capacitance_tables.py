"""J on a slow mode, to rounding: J x = b for b a sine vector, so that x is
b / (1 + D), against D summed over the frequencies in extended precision from the
matrices' entries as plan creation rounds them.  The solution multiplies an
error of D by D again."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

L = np.longdouble
PI = L("3.14159265358979323846264338327950288")


def toeplitz(o, d, n):
    lo, up = np.full(n, o), np.full(n, o)
    lo[0] = up[-1] = 0.0
    return lo, np.full(n, d), up


def exact_d(M, tk, n, ell, j, line):
    """D of mode j; line: None, or the eigenvalue of the line along x (2D)."""
    s2 = np.sin(j * PI / (2 * L(n + 1))) ** 2
    eig = lambda o, d: (L(d) + 2 * L(o)) - 4 * L(o) * s2
    m = L(1) if line is not None else eig(*M)
    D = L(0)
    for k in range(ell // 2 + 1):
        a = 2 * np.pi * k / ell
        lr, li, w = 1 - np.cos(a), np.sin(a), 1 if k in (0, ell // 2) else 2
        if line is not None:
            re, im = eig(tk[0], lr + line + tk[1]), L(li)
        else:
            re, im = eig(lr * M[0] + tk[0], lr * M[1] + tk[1]), eig(li * M[0], li * M[1])
        D += m * L(w) / ell * (L(np.cos(a)) * re - L(np.sin(a)) * im) / (re * re + im * im)
    return D


@pytest.mark.parametrize("kind,n,ell,nu", [("fem", 300, 512, 3e-3), ("fd", 300, 64, 1e-2), ("fd", 511, 256, 3e-3),
                                           ("fem", 1000, 64, 1.5e-3), ("fd", 257, 256, 1.5e-3), ("fd", 4097, 32, 1e-2),
                                           ("fd2", 63, 32, 0.1), ("fd2", 255, 64, 0.1), ("fd2", 200, 128, 0.04)])
def test_slow_modes(lib, kind, n, ell, nu):
    h, dims = 1.0 / (n + 1), 2 if kind == "fd2" else 1
    M, K = ((h / 6.0, 4.0 * h / 6.0), (-nu / h, 2.0 * nu / h)) if kind == "fem" else \
        ((0.0, 1.0), (-nu / h**2, 2.0 * nu / h**2))
    tau = (0.1 if dims == 2 else 1.0) / ell
    tk = (tau * K[0], tau * K[1])
    line = tk[1] + 2.0 * tk[0] * np.cos(np.pi / (n + 1)) if dims == 2 else None
    plan = lib.paradiag_plan_create(n, ell, tau, toeplitz(*M, n) if kind == "fem" else None, toeplitz(*K, n),
                                    dims=dims, stream=torch.cuda.current_stream().cuda_stream)
    try:
        for j in (1, 2):
            i = np.arange(1, n + 1)
            s = (np.sqrt(2 / L(n + 1)) * np.sin(PI * ((i * j) % (2 * (n + 1))) / (n + 1))).astype(float)
            b = np.zeros((n, n)) if dims == 2 else s.copy()
            if dims == 2:
                b[:, 0] = s          # the line m = 1 of the DST-x domain
            bd = torch.tensor(b.ravel(), device="cuda:0")
            x = torch.zeros_like(bd)
            lib.paradiag_capacitance_solve(plan, bd, x, 1e-15, allow_notconv=True)
            ref = b.ravel() / float(1 + exact_d(M, tk, n, ell, j, line))
            # the projection, 1 + D, the quotient and the iteration's scalings: a
            # rounding each
            assert np.linalg.norm(x.cpu().numpy() - ref) <= 6 * 2.0**-53 * np.linalg.norm(ref)
    finally:
        lib.paradiag_plan_destroy(plan)
