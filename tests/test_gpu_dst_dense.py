"""The DST along x as a product on the matrix cores: tile and chunk edges, odd
and even n + 1, powers of two, rows that do not fill a block, the first
time row's u0, in place and accumulating use."""
import numpy as np
import pytest
import scipy.fft

from oracle import allatonce, bdf
from oracle.spatial import spatial_matrices
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda:0")


@pytest.mark.parametrize("n,ell", [(16, 4), (17, 64), (33, 32), (64, 16), (100, 128), (161, 8),
                                   (256, 64), (300, 32), (321, 16), (385, 64), (439, 8), (440, 32)])
def test_rows(lib, n, ell):
    rng = np.random.default_rng(n)
    p = wl.heat_1d("fem1", n, ell, 1.0, 0.1, rng, True)
    x = rng.standard_normal((ell, n))
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, shifted_solver=lib.PD_SHIFTED_SINE,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        out = torch.empty((ell, n), dtype=torch.float64, device="cuda:0")
        same = dev(x)
        lib.paradiag_sine_transform(plan, same, out)
        lib.paradiag_sine_transform(plan, same, same)
        U = torch.empty((ell, n), dtype=torch.float64, device="cuda:0")
        lib.paradiag_solve(plan, dev(p.u0), dev(p.F), U, 1e-12)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    ref = scipy.fft.dst(x.astype(np.longdouble), 1, norm="ortho").astype(np.float64)
    err = np.linalg.norm(out.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    # n / 2 products and sums per output (the chirp-z form: two FFTs of 2048)
    assert err.max() < (n / 2 + 3) * 1.2e-16
    assert torch.equal(out, same)
    assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9


@pytest.mark.parametrize("n,ell", [(16, 4), (31, 8), (45, 16), (63, 4), (101, 4)])
def test_solve_2d(lib, n, ell):
    rng = np.random.default_rng(n)
    p = wl.heat_2d(n, ell, 1.0, 0.1, rng)
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, check_residual=1,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n * n), dtype=torch.float64, device="cuda:0")
        info = lib.paradiag_solve(plan, dev(p.u0), dev(p.F), U, 1e-12)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9
    assert 0 <= info.rel_residual < 1e-9


def test_bdf_2d(lib):
    n, ell, s = 40, 16, 2
    rng = np.random.default_rng(n)
    p = wl.heat_2d(n, ell, 1.0, 0.1, rng)
    U0 = np.stack([p.u0 * (1 + 0.1 * j) for j in range(s)])
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, bdf_order=s,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n * n), dtype=torch.float64, device="cuda:0")
        lib.paradiag_solve(plan, dev(U0), dev(p.F), U, 1e-11)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    Msp, Ksp = spatial_matrices(p.M, p.K, 2)
    assert allatonce.rel_err(U.cpu().numpy(), bdf.step_bdf(Msp, Ksp, p.tau, s, list(U0), p.F)) < 4e-9
