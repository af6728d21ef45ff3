"""The residual pass at the edges of its walks: 62 columns to a wave, 32 rows
to an item, general (non-constant) and constant diagonals, against the
oracle's residual of the same U."""
import numpy as np
import pytest

from oracle import allatonce
from oracle.spatial import problem_matrices
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind,n,ell", [("fem1", 2, 2), ("fd1", 62, 32), ("fem1", 63, 64), ("graded", 125, 128),
                                        ("fd1", 61, 4), ("fd2", 2, 2), ("fd2", 33, 8), ("fd2", 62, 4), ("fd2", 63, 2),
                                        ("fd2", 64, 16)])
def test_residual_of_random_iterate(lib, kind, n, ell):
    rng = np.random.default_rng(n + ell)
    if kind == "fd2":
        p = wl.heat_2d(n, ell, 0.1, 1.0, rng)
        p.F = rng.standard_normal(p.F.shape)
    else:
        p = wl.heat_1d("fem1" if kind == "graded" else kind, n, ell, 1.0, 0.1, rng, True)
        if kind == "graded":
            s = rng.uniform(0.5, 1.5, n)
            p.K = (p.K[0] * s, p.K[1] * (1 + s), p.K[2] * s[::-1])
            p.M = (p.M[0] * s, p.M[1] * (1 + s), p.M[2] * s[::-1])
    U = rng.standard_normal((ell, p.nbar))
    dev = torch.device("cuda:0")
    plan = lib.paradiag_plan_create(p.n, ell, p.tau, p.M, p.K, dims=p.dims,
                                    stream=torch.cuda.current_stream().cuda_stream)
    try:
        got = [f(plan, torch.tensor(p.u0, device=dev), torch.tensor(p.F, device=dev), torch.tensor(U, device=dev))
               for f in (lib.paradiag_residual, lib.paradiag_residual_noalloc)]
    finally:
        lib.paradiag_plan_destroy(plan)
    Msp, Ksp = problem_matrices(p)
    ref = allatonce.residual(Msp, Ksp, p.tau, p.u0, p.F, U)[1]
    # sums of up to 2^14 positive squares of values formed with a few roundings
    assert abs(got[0] - ref) <= 1e-12 * ref and abs(got[1] - ref) <= 1e-12 * ref
