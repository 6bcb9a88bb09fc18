"""Plans and batches with an axis past the matrix-core route (N > 256) beside shorter
ones: Newton's per-axis passes, and a batch whose boxes take different routes."""
import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)


@pytest.mark.parametrize("prec", ["f64", "mixed"])
@pytest.mark.parametrize("n", [(258, 9, 7), (7, 258, 9), (9, 7, 258), (260, 259, 5), (5, 35, 300)])
def test_newton_of_mixed_axes(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    d = lambda a: to_dev(a, torch.float64)
    log(f"newton mixed axes {n} {prec}")
    bc = BC_SETS["NDNNDN"]
    G = O.Grid3(n, LO, HI, bc)
    T, K0 = 0.4 * np.tanh(W.random_field(n, 31)), W.random_conductivity(n, 32)
    f, v = W.random_field(n, 33), W.random_field(n, 34)
    plan = Plan(n, LO, HI, bc, prec)
    r = to_host(plan.newton_residual(d(K0), d(T), d(f), 0.5))
    y = to_host(plan.newton_jacobian(d(K0), d(T), d(v), 0.5))
    for got, ref in ((r, O.newton_residual(G, K0, 0.5, T, f)), (y, O.newton_jacobian(G, K0, 0.5, T, v))):
        assert np.max(np.abs(got - ref)) <= 1e-12 * np.max(np.abs(ref))
        assert np.all(got[~G.interior] == 0.0)


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_batch_of_both_routes(prec):
    """A box with an axis of 259 nodes (a pass per system), one of 9x12x10 (batched
    passes), three load cases each, on the side streams together."""
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Batch, SolveOptions
    d = lambda a: to_dev(a, torch.float64)
    lo, hi = (0.0,) * 3, (1.0,) * 3
    grids, Ks, fs, gs, refs = [], [], [], [], []
    for n in ((259, 6, 5), (9, 12, 10), (5, 6, 261)):
        for a in range(3):
            bc = W.load_case_bc(a)
            K = W.random_conductivity(n, 7 + a, 0.3)
            g = W.random_faces(W.Grid(n, lo, hi, bc), 9)
            grids.append((n, lo, hi, bc))
            Ks.append(d(K)), fs.append(d(np.zeros(n))), gs.append(d(g))
            refs.append((O.Grid3(n, lo, hi, bc), K, g))
    log(f"batch of both routes {prec}")
    us, infos = Batch(grids, prec).solve(Ks, fs, gs, opts=SolveOptions(rtol=1e-10, maxiter=4000, precond=True))
    for u, info, (G, K, g) in zip(us, infos, refs):
        assert info["status"] == 0
        e = rel_l2(to_host(u), O.solve_dense(G, K, np.zeros(G.n), g))
        log(f"  {G.n}: {info['matvecs']} matvecs, err {e:.1e}")
        # the condition, about N^4 of the long axis (4e9), times FP64 rounding
        assert e <= 1e-5
