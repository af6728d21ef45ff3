"""paradiag_plan_bytes counts the sine-basis capacitance tables, and those of the DST
as a product, only for plans that may use them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MB = 1 << 20


@pytest.mark.parametrize("kw", [dict(autotune=1), dict(krylov=1)])
def test_no_tables(lib, kw):
    n, ell = 8191, 8
    tables = 192 * 8192 * 8   # of the plan with GMRES and no autotuning
    h = 1.0 / (n + 1)
    K = (np.full(n, -1 / h**2), np.full(n, 2 / h**2), np.full(n, -1 / h**2))
    plan = lib.paradiag_plan_create(n, ell, 1.0 / ell, None, K,
                                    stream=torch.cuda.current_stream().cuda_stream, **kw)
    lib.paradiag_plan_destroy(plan)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    plan = lib.paradiag_plan_create(n, ell, 1.0 / ell, None, K,
                                    stream=torch.cuda.current_stream().cuda_stream, **kw)
    used = free - torch.cuda.mem_get_info()[0]
    lib.paradiag_plan_destroy(plan)
    est = lib.paradiag_plan_bytes(n, ell, **kw)
    print("estimate %d, used %d" % (est, used))
    assert est < used + tables // 2


# 441 points never take the product; fewer points that do not for these numbers of
# rows need no more memory than those
@pytest.mark.parametrize("n,ell", [(300, 128), (400, 64), (400, 512), (440, 2), (440, 2048)])
def test_no_product_tables(lib, n, ell):
    assert lib.paradiag_plan_bytes(n, ell, shifted_solver=1) <= lib.paradiag_plan_bytes(441, ell, shifted_solver=1)
