"""DST rows of lengths off 2^m - 1 around the number of rows where the product takes
over from the chirp-z form, against an extended-precision DST."""
import numpy as np
import pytest
import scipy.fft

from oracle import allatonce
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# rows of the product: any for n <= 144, 6 n for n <= 316, 10 n above
@pytest.mark.parametrize("n,ell", [(144, 2), (145, 512), (145, 1024), (160, 1024), (200, 2048), (256, 2048), (300, 2048),
                                   (316, 1024), (316, 2048), (317, 2048), (317, 4096), (400, 4096), (385, 4096)])
def test_rows(lib, n, ell):
    rng = np.random.default_rng(n)
    p = wl.heat_1d("fem1", n, ell, 1.0, 0.1, rng, False)
    x = rng.standard_normal((ell, n))
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, shifted_solver=lib.PD_SHIFTED_SINE,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        same = torch.tensor(x, device="cuda:0")
        out = torch.empty_like(same)
        lib.paradiag_sine_transform(plan, same, out)
        lib.paradiag_sine_transform(plan, same, same)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    ref = scipy.fft.dst(x.astype(np.longdouble), 1, norm="ortho").astype(np.float64)
    err = np.linalg.norm(out.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    # n / 2 products and sums per output (the chirp-z form: two FFTs of 1024)
    assert err.max() < (n / 2 + 3) * 1.2e-16
    assert torch.equal(out, same)


# 2D: n ell rows; u0 in the first time row, accumulating inverse in the mixed form
@pytest.mark.parametrize("n,ell,prec", [(150, 4, 0), (150, 8, 1), (200, 4, 1), (317, 8, 0), (317, 16, 1)])
def test_2d(lib, n, ell, prec):
    p = wl.heat_2d(n, ell, 1.0, 0.1, np.random.default_rng(n))
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, precision=prec, check_residual=1,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        F = torch.tensor(p.F, device="cuda:0")
        U = torch.empty_like(F)
        info = lib.paradiag_solve(plan, torch.tensor(p.u0, device="cuda:0"), F, U, 1e-11)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9
    assert 0 <= info.rel_residual < 1e-9
