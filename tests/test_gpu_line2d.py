"""2D line solves in the recurrence form: lines of 1 to 64 lanes with 4 and 8
rows each, full and ragged, columns that do not fill the last block, one and
several frequencies to a block, complex128 and complex64 right-hand sides."""
import numpy as np
import pytest

from oracle import allatonce
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n,ell", [(5, 8), (20, 64), (32, 8), (33, 512), (64, 16), (65, 4), (113, 128), (128, 8),
                                   (129, 4), (200, 16), (256, 4), (257, 8), (300, 4), (512, 4)])
def test_lines(lib, n, ell, mixed):
    rng = np.random.default_rng(n + ell)
    p = wl.heat_2d(n, ell, 0.5, 0.05, rng)
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, check_residual=1,
                                    precision=lib.PD_MIXED if mixed else lib.PD_FP64,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        dev = lambda a: torch.tensor(np.ascontiguousarray(a), device="cuda:0")
        U = torch.empty((ell, n * n), dtype=torch.float64, device="cuda:0")
        info = lib.paradiag_solve(plan, dev(p.u0), dev(p.F), U, 1e-11)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    # the residual of a backward stable solve, amplified by at most the two
    # transforms and the time steps' sum
    assert 0 <= info.rel_residual < 1e-10
    if n <= 130:
        assert allatonce.rel_err(U.cpu().numpy(), allatonce.step(p)) < 1e-9
