"""x and y axes whose row-block counts differ by one: applies read tables of one block
more for the shorter axis where x and y share a launch, derivatives its own.  Every
mode against the oracle on both sides of the rule, the same bits with three launches.
Bars as for every apply: relative L2 error to the oracle <= 1e-12 in FP64 and <= 1e-5
in FP32."""
import ctypes

import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)


@pytest.mark.parametrize("prec", ["f64", "f32", "mixed"])
@pytest.mark.parametrize("n", [
    (33, 49, 12), (49, 33, 12),          # one and two blocks, a lone middle row in the one
    (64, 97, 9), (129, 97, 40),          # two and three, three and four
    (129, 131, 9), (150, 100, 12),       # four and five, few tasks
    (131, 128, 75),                      # four and five, 1163 tasks: FP64 takes three launches
    (161, 193, 7), (257, 225, 5), (65, 97, 300),
])
def test_axes_a_block_apart(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd import _lib as L
    from paper_2606_21410_amd.api import Plan
    bc, robin = BC_SETS["NDNNDN"], (0.5, 0.0, 0.25, 1.0, 0.0, 2.0)
    log(f"axes a block apart {n} {prec}")
    G = O.Grid3(n, LO, HI, bc, robin)
    dt, tol = (torch.float32, 1e-5) if prec == "f32" else (torch.float64, 1e-12)
    cast = (lambda a: a.astype(np.float32).astype(np.float64)) if prec == "f32" else (lambda a: a)
    u, K = cast(W.random_field(n, 1)), cast(W.random_conductivity(n, 2, 0.5))
    plan = Plan(n, LO, HI, bc, prec, robin=robin)
    Kd, ud = to_dev(K, dt), to_dev(u, dt)
    side = torch.cuda.Stream()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    for mode, flags, ref in (("reduced", 1, O.apply_reduced(G, K, u)),
                             ("transpose", 3, O.apply_reduced_transpose(G, K, u)),
                             ("full", 0, O.apply_full(G, K, u))):
        y = torch.full(n, float("nan"), device="cuda", dtype=dt)
        plan.apply(Kd, ud, y, mode=mode)
        assert rel_l2(to_host(y), ref) <= tol, mode
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            z = torch.full_like(y, float("nan"))
            plan._sync_stream()
            L.check(plan.lib.cheb_apply(plan.handle, p(Kd), p(ud), p(z), flags))
        torch.cuda.synchronize()
        assert torch.equal(y, z), mode
    for a in range(3):
        assert rel_l2(to_host(plan.derivative(ud, a)), O.deriv(G.D[a], u, a)) <= tol
    if prec != "f32":
        T = 0.3 * np.tanh(W.random_field(n, 3))
        y_o = O.newton_jacobian(G, K, 0.5, T, u)
        y = to_host(plan.newton_jacobian(Kd, to_dev(T, dt), ud, 0.5))
        assert np.max(np.abs(y - y_o)) <= 1e-12 * np.max(np.abs(y_o))
