"""Matrix-core passes of few tasks: axes of three and four row blocks on both sides
of one task per CU, every mode and axis, against the oracle, and the same bits
whether the x and y passes share a launch or not.  Bars as for every apply:
relative L2 error to the oracle <= 1e-12 in FP64 and <= 1e-5 in FP32."""
import ctypes

import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [
    (66, 5, 7), (5, 97, 6), (7, 6, 129),             # a task or two; the rows' remainders
    (67, 12, 30), (30, 98, 12), (12, 30, 100),
    (129, 128, 18), (97, 96, 20),                    # x and y together just below 256 tasks
    (129, 129, 20), (97, 97, 30),                    # and above it
    (64, 64, 66), (66, 66, 70),                      # z: 241 tasks, 256 (FULL: 273)
])
def test_few_tasks(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd import _lib as L
    from paper_2606_21410_amd.api import Plan
    bc, robin = BC_SETS["NDNNDN"], (0.5, 0.0, 0.25, 1.0, 0.0, 2.0)
    log(f"few tasks {n} {prec}")
    G = O.Grid3(n, LO, HI, bc, robin)
    dt, tol = (torch.float64, 1e-12) if prec == "f64" else (torch.float32, 1e-5)
    cast = (lambda a: a) if prec == "f64" else (lambda a: a.astype(np.float32).astype(np.float64))
    u, K = cast(W.random_field(n, 1)), cast(W.random_conductivity(n, 2, 0.5))
    ub = u.copy()
    ub[~G.interior] = np.nan  # the reduced forms ignore boundary values
    plan = Plan(n, LO, HI, bc, prec, robin=robin)
    Kd, ud, ubd = to_dev(K, dt), to_dev(u, dt), to_dev(ub, dt)
    side = torch.cuda.Stream()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    for mode, flags, x, ref in (("reduced", 1, ubd, O.apply_reduced(G, K, u)),
                                ("transpose", 3, ubd, O.apply_reduced_transpose(G, K, u)),
                                ("full", 0, ud, O.apply_full(G, K, u))):
        y = torch.full(n, float("nan"), device="cuda", dtype=dt)
        plan.apply(Kd, x, y, mode=mode)
        assert rel_l2(to_host(y), ref) <= tol, mode
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            z = torch.full_like(y, float("nan"))
            plan._sync_stream()
            L.check(plan.lib.cheb_apply(plan.handle, p(Kd), p(x), p(z), flags))  # three launches
        torch.cuda.synchronize()
        if n[2] in (33, 65, 97, 129):  # a lone middle row along z: added in another order
            mid = n[2] // 2
            assert float((y - z).abs().max()) <= 4 * torch.finfo(dt).eps * float(y.abs().max())
            y[:, :, mid] = z[:, :, mid] = 0
        assert torch.equal(y, z), mode
    for a in range(3):
        assert rel_l2(to_host(plan.derivative(ud, a)), O.deriv(G.D[a], u, a)) <= tol
    if prec == "f64":
        T = 0.3 * np.tanh(W.random_field(n, 3))
        y_o = O.newton_jacobian(G, K, 0.5, T, u)
        y = to_host(plan.newton_jacobian(Kd, to_dev(T, dt), ubd, 0.5))
        assert np.max(np.abs(y - y_o)) <= 1e-12 * np.max(np.abs(y_o))
