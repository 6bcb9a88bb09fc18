"""GPU parity of the matrix-core axis passes at the edges of their row blocks.

An axis of N = n - 1 takes R = N // 2 + 1 row pairs in 16-row blocks; the sizes
are the smallest, both sides of every kind of block boundary (an even N with
N % 32 == 0 has a lone middle row, an odd N none), the change from one-wave
tasks (up to four blocks) to row-block workgroups, and the largest (N = 256);
each on each axis, the other two short.  Bars, as for every apply: relative L2
error to the oracle <= 1e-12 in FP64 and <= 1e-5 in FP32; the Jacobian <= 1e-12
of its largest entry.
"""
import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)
N_NODES = [3, 16, 31, 32, 33, 34, 64, 65, 67, 98, 128, 129, 130, 160, 161, 193, 226, 256, 257]


def _grid(n, axis):
    g = [7, 7, 7]
    g[axis], g[(axis + 1) % 3] = n, 20  # 18 interior pencils across: a ragged tail of the 16-pencil tile
    return tuple(g)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("n", N_NODES)
def test_line_pass_sizes(n, axis, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    g = _grid(n, axis)
    bc = BC_SETS["NDNNDN"]
    robin = (0.5, 0.0, 0.25, 1.0, 0.0, 2.0)
    log(f"line passes n={g} {prec}")
    G = O.Grid3(g, LO, HI, bc, robin)
    dt, tol = (torch.float64, 1e-12) if prec == "f64" else (torch.float32, 1e-5)
    cast = (lambda a: a) if prec == "f64" else (lambda a: a.astype(np.float32).astype(np.float64))
    u, K = cast(W.random_field(g, 1)), cast(W.random_conductivity(g, 2, 0.5))
    ub = u.copy()
    ub[~G.interior] = np.nan  # the reduced forms ignore boundary values
    plan = Plan(g, LO, HI, bc, prec, robin=robin)
    Kd, ud, ubd = to_dev(K, dt), to_dev(u, dt), to_dev(ub, dt)
    for shape in (0, 1):
        plan.set_tile_shape(shape, prec)
        y = torch.full(g, float("nan"), device="cuda", dtype=dt)
        yr = to_host(plan.apply(Kd, ubd, y, mode="reduced"))
        assert rel_l2(yr, O.apply_reduced(G, K, u)) <= tol
        assert np.all(yr[~G.interior] == 0.0)
        y = torch.full(g, float("nan"), device="cuda", dtype=dt)
        yt = to_host(plan.apply(Kd, ubd, y, mode="transpose"))
        assert rel_l2(yt, O.apply_reduced_transpose(G, K, u)) <= tol
        assert np.all(yt[~G.interior] == 0.0)
    y = torch.full(g, float("nan"), device="cuda", dtype=dt)
    assert rel_l2(to_host(plan.apply(Kd, ud, y, mode="full")), O.apply_full(G, K, u)) <= tol
    for a in range(3):
        assert rel_l2(to_host(plan.derivative(ud, a)), O.deriv(G.D[a], u, a)) <= tol
    if prec == "f64":
        T = 0.3 * np.tanh(W.random_field(g, 3))
        y_o = O.newton_jacobian(G, K, 0.5, T, u)
        y = to_host(plan.newton_jacobian(Kd, to_dev(T, dt), ubd, 0.5))
        assert np.max(np.abs(y - y_o)) <= 1e-12 * np.max(np.abs(y_o))


@pytest.mark.parametrize("n", [(20, 34, 27), (131, 9, 12)])
def test_batch_ragged_sizes_vs_oracle(n):
    """Batched passes on axes of different block counts: preconditioned solves
    to the oracle's solutions within 1e-8 (as the other batched solves)."""
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Batch, SolveOptions, load_case
    d = lambda a: to_dev(a, torch.float64)
    grids, Ks, fs, gs, refs = [], [], [], [], []
    for a in range(3):
        bc, gf = load_case(n, a, "cpu")
        K = W.random_conductivity(n, 7, 0.3)
        grids.append((n, (0.0,) * 3, (1.0,) * 3, bc))
        Ks.append(d(K)), fs.append(d(np.zeros(n))), gs.append(d(gf.numpy()))
        refs.append(O.solve(O.Grid3(n, (0, 0, 0), (1, 1, 1), bc), K, np.zeros(n), gf.numpy(), tol=1e-14))
    us, infos = Batch(grids, "f64").solve(Ks, fs, gs, opts=SolveOptions(rtol=1e-11, maxiter=4000, precond=True))
    for u, info, ref in zip(us, infos, refs):
        assert info["status"] == 0
        assert rel_l2(to_host(u), ref) <= 1e-8
