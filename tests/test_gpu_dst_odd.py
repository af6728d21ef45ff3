"""The DST along x of 2D plans with n + 1 a power of two: pairs of rows that do
not fill a block, an odd number of rows, the sizes around the block's pair count,
the accumulating form (BDF) and the smaller sizes, which keep the full FFT."""
import numpy as np
import pytest

from oracle import allatonce, bdf
from oracle.spatial import spatial_matrices
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda:0")


@pytest.mark.parametrize("n,ell,s", [(15, 8, 1), (31, 4, 1), (63, 2, 1), (127, 8, 1), (255, 4, 1), (31, 16, 3),
                                     (63, 8, 2)])
def test_solve(lib, n, ell, s):
    rng = np.random.default_rng(n + ell)
    p = wl.heat_2d(n, ell, 1.0, 0.1, rng)
    U0 = np.stack([p.u0 * (1 + 0.1 * j) for j in range(s)]) if s > 1 else p.u0
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, bdf_order=s,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n * n), dtype=torch.float64, device="cuda:0")
        lib.paradiag_solve(plan, dev(U0), dev(p.F), U, 1e-12)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    if s == 1:
        assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9
    else:
        Msp, Ksp = spatial_matrices(p.M, p.K, 2)
        assert allatonce.rel_err(U.cpu().numpy(), bdf.step_bdf(Msp, Ksp, p.tau, s, list(U0), p.F)) < 4e-9


@pytest.mark.parametrize("n,ell", [(31, 2), (255, 2), (511, 2), (1023, 2)])
def test_forward_transform(lib, n, ell):
    """Hhat_0 and Hhat_1 of two time steps: sum and difference of the rows'
    sine transforms."""
    rng = np.random.default_rng(n)
    K = wl.fd_laplacian(n, 1.0)
    F, u0 = rng.standard_normal((ell, n * n)), rng.standard_normal(n * n)
    plan = lib.paradiag_plan_create(n, ell, 0.5, None, K, dims=2, stream=torch.cuda.current_stream().cuda_stream)
    try:
        H = torch.empty((2, n * n), dtype=torch.complex128, device="cuda:0")
        lib.paradiag_forward_transform(plan, dev(u0), dev(F), H)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    j = np.arange(1, n + 1)
    S = np.sqrt(2.0 / (n + 1)) * np.sin(np.pi * (np.outer(j, j) % (2 * (n + 1))) / (n + 1))
    h = 0.5 * F
    h[0] += u0
    h = (h.reshape(ell, n, n) @ S).reshape(ell, -1)
    H = H.cpu().numpy()
    for got, ref in ((H[0], h[0] + h[1]), (H[1], h[0] - h[1])):
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        # the reference's dot products of n terms, and log2(2n) FFT stages
        assert err < 1.2e-16 * (np.sqrt(n) + 4 * np.log2(2 * n))
