"""The FFT route by name, at every compiled transform size and at sizes without one.
(The default route takes the matrix cores for N <= 256.)  Bars as for every apply:
relative L2 error to the oracle <= 1e-12 in FP64 and <= 1e-5 in FP32."""
import numpy as np
import pytest

from oracle import cheb_oracle as O
from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, rel_l2, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -1.0, 0.5), (1.0, 1.0, 2.0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", [
    (9, 13, 17), (25, 9, 7), (9, 25, 7), (7, 9, 25), (33, 49, 65), (97, 7, 9), (9, 129, 7), (7, 9, 97),
    (193, 9, 9), (9, 193, 7), (6, 5, 193), (257, 5, 7), (5, 257, 6), (6, 7, 257), (385, 5, 6), (5, 6, 385),
    (24, 35, 10),  # no compiled transform
])
def test_fft_route(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    bc, robin = BC_SETS["NDNNDN"], (0.5, 0.0, 0.25, 1.0, 0.0, 2.0)
    log(f"fft route {n} {prec}")
    G = O.Grid3(n, LO, HI, bc, robin)
    dt, tol = (torch.float64, 1e-12) if prec == "f64" else (torch.float32, 1e-5)
    cast = (lambda a: a) if prec == "f64" else (lambda a: a.astype(np.float32).astype(np.float64))
    u, K = cast(W.random_field(n, 1)), cast(W.random_conductivity(n, 2, 0.5))
    plan = Plan(n, LO, HI, bc, prec, robin=robin, route="fft")
    Kd, ud = to_dev(K, dt), to_dev(u, dt)
    for mode, ref in (("reduced", O.apply_reduced(G, K, u)), ("transpose", O.apply_reduced_transpose(G, K, u)),
                      ("full", O.apply_full(G, K, u))):
        y = to_host(plan.apply(Kd, ud, mode=mode))
        assert rel_l2(y, ref) <= tol, mode
        if mode != "full":
            assert np.all(y[~G.interior] == 0.0)
    for a in range(3):
        assert rel_l2(to_host(plan.derivative(ud, a)), O.deriv(G.D[a], u, a)) <= tol
    if prec == "f64":
        T = 0.3 * np.tanh(W.random_field(n, 3))
        y_o = O.newton_jacobian(G, K, 0.5, T, u)
        y = to_host(plan.newton_jacobian(Kd, to_dev(T, dt), ud, 0.5))
        assert np.max(np.abs(y - y_o)) <= 1e-12 * np.max(np.abs(y_o))


def test_adjoint_gradient_on_the_fft_route():
    """The transposed derivatives of the gradient, against the matrix-core route's."""
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan, SolveOptions
    n = (33, 25, 20)
    d = lambda a: to_dev(a, torch.float64)
    K, f, w = W.random_conductivity(n, 1, 0.3), W.random_field(n, 2), W.random_field(n, 3)
    g = W.random_faces(W.Grid(n, (0, 0, 0), (1, 1, 1), W.MIXED_X_BC), 4)
    grads = []
    for route in ("fft", "matrix"):
        plan = Plan(n, bc=W.MIXED_X_BC, route=route)
        opts = SolveOptions(rtol=1e-13, precond=True)
        u, _ = plan.solve(d(K), d(f), d(g), opts=opts)
        _, grad, info = plan.adjoint(d(K), u, d(w), opts)
        assert info["status"] == 0
        grads.append(to_host(grad))
    # two solves to 1e-13 of systems whose condition is below 1e4
    assert rel_l2(grads[0], grads[1]) <= 1e-8
