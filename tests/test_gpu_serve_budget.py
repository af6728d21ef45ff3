"""Requests whose budget holds a plan without the fast forms' tables only: they run
with such a plan, and the accounting keeps to the budget."""
import numpy as np
import pytest

from oracle import allatonce, modal
from paper_2304_12597_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MB = 1 << 20


# room: what the plan may take; its estimate with all tables is more
@pytest.mark.parametrize("dims,n,ell,prec,room", [(1, 4095, 8, 0, 4 * MB), (1, 8191, 16, 0, 9 * MB),
                                                  (1, 8191, 16, 1, 8 * MB), (1, 1023, 16, 1, MB),
                                                  (2, 127, 4, 0, 11100000)])
def test_small_budget(lib, dims, n, ell, prec, room):
    rng = np.random.default_rng(n)
    p = wl.heat_2d(n, ell, 0.1, 0.5, rng) if dims == 2 else wl.heat_1d("fd1", n, ell, 1.0, 0.5, rng, False)
    dev = torch.device("cuda:0")
    arrays = (2 * ell + 1) * p.nbar * 8
    assert lib.paradiag_plan_bytes(n, ell, dims=dims, precision=prec) > room
    u0, F = torch.tensor(p.u0, device=dev), torch.tensor(p.F, device=dev)
    Us = [torch.empty_like(F) for _ in range(3)]
    torch.cuda.synchronize()
    srv = lib.pd_server_create(2, int(arrays + room))
    try:
        tickets = [lib.pd_server_submit(srv, n, ell, p.tau, p.M, p.K, u0, F, U, 1e-9, dims=dims, precision=prec)
                   for U in Us]
        for t in tickets:
            done, st, _ = lib.pd_server_wait(srv, t, -1)
            assert done and st == 0
        stats = lib.pd_server_stats(srv)
        assert stats["peak_bytes"] <= arrays + room and stats["cache_hits"] == 2
        with pytest.raises(lib.PDError) as e:
            lib.pd_server_submit(srv, n, 64 * ell, p.tau, p.M, p.K, u0, F, Us[0], 1e-9, dims=dims, precision=prec)
        assert e.value.status == lib.PD_EBUDGET
    finally:
        lib.pd_server_destroy(srv)
    ref = modal.modal_solution(p)
    for U in Us:
        assert allatonce.rel_err(U.cpu().numpy(), ref) < 1e-8
