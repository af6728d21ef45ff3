"""The rows' DST of sine-basis plans, n + 1 a power of two: one to many rows per
block, rows of less and more than a wave's threads, in place, and an unsorted
magnitude in the first time row (u0)."""
import numpy as np
import pytest

from oracle import allatonce
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,ell", [(15, 8), (31, 64), (127, 4), (511, 32), (1023, 16), (2047, 64), (4095, 8), (8191, 4)])
def test_rows(lib, n, ell):
    rng = np.random.default_rng(n)
    p = wl.heat_1d("fem1", n, ell, 1.0, 0.1, rng, True)
    x = rng.standard_normal((ell, n))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, shifted_solver=lib.PD_SHIFTED_SINE,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        same, out = dev(x), torch.empty((ell, n), dtype=torch.float64, device="cuda:0")
        lib.paradiag_sine_transform(plan, same, out)
        lib.paradiag_sine_transform(plan, same, same)
        U = torch.empty((ell, n), dtype=torch.float64, device="cuda:0")
        lib.paradiag_solve(plan, dev(p.u0), dev(p.F), U, 1e-12)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    # the odd extension's FFT in extended precision
    ext = np.zeros((ell, 2 * (n + 1)), dtype=np.longdouble)
    ext[:, 1:n + 1], ext[:, n + 2:] = x, -x[:, ::-1]
    import scipy.fft
    ref = (-scipy.fft.fft(ext, axis=1).imag[:, 1:n + 1] / np.sqrt(2 * np.longdouble(n + 1))).astype(np.float64)
    err = np.linalg.norm(out.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    # prefix sums of n / 2 terms, each with the error of log2(n) stages
    assert err.max() < 1.2e-16 * 2 * np.sqrt(n / 2) * np.log2(n + 1)
    assert torch.equal(out, same)
    assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9
