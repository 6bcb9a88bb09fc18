"""One plan's applies on several streams at once: they share no memory, whatever
stream the plan was created on, and give the same results on every stream and from a
replayed graph."""
import ctypes

import pytest

from paper_2606_21410_amd import workloads as W
from tests.gpu_util import BC_SETS, log, require_gpu, to_dev

pytestmark = pytest.mark.gpu

MODES = ("reduced", "transpose", "full")
# equal and different row-block counts along x and y, a lone middle row (N % 32 == 0)
# along x, along z and along neither, more than four row blocks
SIZES = [(33, 33, 33), (25, 20, 49), (100, 100, 100), (65, 34, 129), (140, 9, 161)]


def _fields(n, prec, count):
    import torch
    dt = torch.float32 if prec == "f32" else torch.float64
    K = to_dev(W.random_conductivity(n, 2, 0.5), dt)
    return K, [to_dev(W.random_field(n, 10 + i), dt) for i in range(count)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", SIZES)
def test_same_bits_on_every_stream(n, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd import _lib as L
    from paper_2606_21410_amd.api import Plan
    plan = Plan(n, bc=BC_SETS["NDNNDN"], precision=prec)
    K, (u,) = _fields(n, prec, 1)
    side = torch.cuda.Stream()
    T = 0.3 * torch.tanh(u) if prec == "f64" else None
    calls = [lambda m=m: plan.apply(K, u, mode=m) for m in MODES]

    def no_scratch():
        # the C entry on whatever stream is current: three launches off the creation stream
        y = torch.empty_like(u)
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        plan._sync_stream()
        L.check(plan.lib.cheb_apply(plan.handle, p(K), p(u), p(y), 3))
        return y

    calls.append(no_scratch)
    if prec == "f64":
        calls.append(lambda: plan.newton_jacobian(K, T, u, 0.5))
    for i, call in enumerate(calls):
        log(f"streams {n} {prec} call {i}")
        home = call()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            other = call()
        torch.cuda.synchronize()
        if call is no_scratch and n[2] in (33, 65, 97, 129):
            # a lone middle row along z: three launches add its terms in another order
            eps = torch.finfo(home.dtype).eps
            assert float((home - other).abs().max()) <= 4 * eps * float(home.abs().max())
            mid = n[2] // 2
            home[:, :, mid] = other[:, :, mid] = 0
        assert torch.equal(home, other)


@pytest.mark.parametrize("n", [(33, 33, 33), (100, 100, 100), (129, 129, 129)])
@pytest.mark.parametrize("mode", MODES)
def test_concurrent_applies(n, mode):
    """Applies on the creation stream, on two others and from a graph in flight
    together, each with its own input, against the same calls one at a time."""
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    log(f"concurrent {mode} {n}")
    plan = Plan(n, bc=BC_SETS["DDNNNN"])
    K, us = _fields(n, "f64", 4)
    refs = [plan.apply(K, u, mode=mode) for u in us]
    torch.cuda.synchronize()
    streams = [torch.cuda.current_stream()] + [torch.cuda.Stream() for _ in range(3)]
    ys = [[torch.full_like(u, float("nan")) for _ in range(12)] for u in us]
    graph = plan.capture_applies(K, [us[3]] * 12, ys[3], mode)
    for y in ys[3]:
        y.fill_(float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[3]):
        graph.replay()
    for k in range(12):
        for i in range(3):
            with torch.cuda.stream(streams[i]):
                plan.apply(K, us[i], ys[i][k], mode)
    torch.cuda.synchronize()
    for i, ref in enumerate(refs):
        for k in range(12):
            assert torch.equal(ys[i][k], ref), (i, k)


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_solve_beside_applies(prec):
    """A solve on one stream while applies of the same plan are pending on its
    creation stream: both as when they run alone."""
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan, SolveOptions
    n = (65, 50, 65)
    log(f"solve beside applies {prec}")
    plan = Plan(n, bc=W.MIXED_X_BC, precision=prec)
    K, (u, f) = _fields(n, "f64", 2)
    g = to_dev(W.random_faces(W.Grid(n, (0, 0, 0), (1, 1, 1), W.MIXED_X_BC), 5), torch.float64)
    opts = SolveOptions(precond=True, rtol=1e-10)
    ref, x_ref = plan.apply(K, u, mode="reduced"), plan.solve(K, f, g, opts=opts)[0]
    torch.cuda.synchronize()
    ys = [torch.empty_like(u) for _ in range(40)]
    side = torch.cuda.Stream()
    for y in ys:
        plan.apply(K, u, y, "reduced")
    with torch.cuda.stream(side):
        x = plan.solve(K, f, g, opts=opts)[0]
    torch.cuda.synchronize()
    assert torch.equal(x, x_ref)
    for y in ys:
        assert torch.equal(y, ref)


def test_apply_scratch_arguments():
    require_gpu()
    import torch
    from paper_2606_21410_amd import _lib as L
    from paper_2606_21410_amd.api import Plan
    n = (9, 9, 9)
    plan = Plan(n, bc=W.MIXED_X_BC)
    K, u, y = (torch.ones(n, device="cuda", dtype=torch.float64) for _ in range(3))
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    for bad in (None, p(K), p(u), p(y)):
        assert plan.lib.cheb_apply_scratch(plan.handle, p(K), p(u), p(y), 1, bad) == L.CHEB_ERR_INVALID_ARG
