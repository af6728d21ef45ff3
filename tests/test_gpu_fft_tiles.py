"""Time transforms with the wider tiles of launches of many tiles: a ragged last
tile in 2D, and a batch whose problems alone take the narrower ones."""
import numpy as np
import pytest

from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda:0")


def test_ragged_2d(lib):
    n, ell = 340, 256   # 115600 columns: 3612.5 tiles of 32
    p = wl.heat_2d(n, ell, 0.5, 0.05, np.random.default_rng(1))
    plan = lib.paradiag_plan_create(n, ell, p.tau, p.M, p.K, dims=2, check_residual=1,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        U = torch.empty((ell, n * n), dtype=torch.float64, device="cuda:0")
        info = lib.paradiag_solve(plan, dev(p.u0), dev(p.F), U, 1e-11)
        torch.cuda.synchronize()
    finally:
        lib.paradiag_plan_destroy(plan)
    assert 0 <= info.rel_residual < 1e-10


def test_batch_equals_alone(lib):
    rng = np.random.default_rng(2)
    stream = torch.cuda.current_stream().cuda_stream
    probs = [wl.heat_1d("fd1", 4000 - 7 * i, 256 << (i % 3), 1.0, 0.1, rng, True) for i in range(20)]
    plans = [lib.paradiag_plan_create(p.n, p.ell, p.tau, p.M, p.K, stream=stream) for p in probs]
    try:
        u0, F = [dev(p.u0) for p in probs], [dev(p.F) for p in probs]
        U = [torch.empty_like(f) for f in F]
        lib.paradiag_solve_batch(plans, u0, F, U, 1e-11)
        for plan, a, f, u in zip(plans, u0, F, U):
            alone = torch.empty_like(f)
            lib.paradiag_solve(plan, a, f, alone, 1e-11)
            torch.cuda.synchronize()
            assert torch.equal(alone, u)
    finally:
        for plan in plans:
            lib.paradiag_plan_destroy(plan)
