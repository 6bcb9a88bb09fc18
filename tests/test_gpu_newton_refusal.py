"""A Jacobian call that is refused (k(T) not positive) has finished with the
caller's buffers when it returns, and has not touched its output."""
import pytest

from paper_2606_21410_amd import workloads as W
from tests.gpu_util import log, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(193, 193, 193), (9, 300, 7)])
def test_refused_jacobian_leaves_nothing_running(n):
    require_gpu()
    import torch
    from paper_2606_21410_amd import _lib as L
    from paper_2606_21410_amd.api import Plan
    log(f"refused jacobian {n}")
    plan = Plan(n, bc=W.MIXED_X_BC)
    K, v = (torch.ones(n, device="cuda", dtype=torch.float64) for _ in range(2))
    T = torch.full_like(K, -3.0)  # 1 + 0.5 T < 0
    y = torch.full_like(K, 7.0)
    torch.cuda.synchronize()
    for _ in range(2):
        with pytest.raises(L.ChebError) as e:
            plan.newton_jacobian(K, T, v, 0.5, y)
        assert torch.cuda.current_stream().query()
        assert e.value.code == L.CHEB_ERR_BAD_INPUT
    assert bool((y == 7.0).all())
    # the same plan goes on
    assert torch.isfinite(plan.newton_jacobian(K, T + 3.0, v, 0.5, y)).all()
