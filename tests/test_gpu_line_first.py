"""Unit-stride passes that open an apply, and strided ones that add to it, on axes of
more than four row blocks: grids whose x and y cannot share a launch.  Bars as for
every apply."""
import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [(9, 66, 140), (66, 9, 161), (7, 70, 193), (70, 7, 200), (9, 97, 225), (66, 5, 257),
                               (140, 9, 66), (9, 161, 70), (193, 70, 7), (70, 225, 5), (257, 66, 6), (6, 250, 140)])
def test_three_launch_applies(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    bc, robin = BC_SETS["NDNNDN"], (0.5, 0.0, 0.25, 1.0, 0.0, 2.0)
    log(f"three launches {n} {prec}")
    G = O.Grid3(n, LO, HI, bc, robin)
    dt, tol = (torch.float64, 1e-12) if prec == "f64" else (torch.float32, 1e-5)
    cast = (lambda a: a) if prec == "f64" else (lambda a: a.astype(np.float32).astype(np.float64))
    u, K = cast(W.random_field(n, 1)), cast(W.random_conductivity(n, 2, 0.5))
    ub = u.copy()
    ub[~G.interior] = np.nan
    plan = Plan(n, LO, HI, bc, prec, robin=robin)
    Kd, ud, ubd = to_dev(K, dt), to_dev(u, dt), to_dev(ub, dt)
    for mode, x, ref in (("reduced", ubd, O.apply_reduced(G, K, u)), ("full", ud, O.apply_full(G, K, u)),
                         ("transpose", ubd, O.apply_reduced_transpose(G, K, u))):
        y = torch.full(n, float("nan"), device="cuda", dtype=dt)
        assert rel_l2(to_host(plan.apply(Kd, x, y, mode=mode)), ref) <= tol, mode
    if prec == "f64":
        T = 0.3 * np.tanh(W.random_field(n, 3))
        y_o = O.newton_jacobian(G, K, 0.5, T, u)
        y = to_host(plan.newton_jacobian(Kd, to_dev(T, dt), ubd, 0.5))
        assert np.max(np.abs(y - y_o)) <= 1e-12 * np.max(np.abs(y_o))
