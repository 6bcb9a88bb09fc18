"""The preconditioner at the interior sizes where its contractions' padding can go
wrong, against the Kronecker inverse of the 1-D operators, within a bound that stays
small on axes with Neumann faces at both ends.  (Such an axis' operator alone is
singular; what is inverted is the sum of the three axes' eigenvalues.)

The bound: the rounding of the six contractions, a dot product of m terms each, in the
type's tables; and that of the decomposition, whose eigenvalues are off by the
rounding of the largest one, on both sides of the comparison, against the smallest
sum that is divided by."""
import numpy as np
import pytest

from oracle import cheb_oracle as O
from tests.gpu_util import log, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu

KC = 1.7
EDGE = (1.0, 2.0, 1.5)


def along(M, x, axis):
    return np.moveaxis(np.tensordot(M, x, (1, axis)), 0, axis)


@pytest.mark.parametrize("shape,bc", [
    ((3, 4, 5), (0, 0, 1, 1, 0, 0)),
    ((33, 34, 35), (0, 0, 1, 1, 0, 0)),
    ((20, 67, 100), (0, 0, 0, 0, 1, 1)),
    ((12, 100, 66), (0, 0, 0, 1, 1, 1)),
    ((9, 70, 99), (1, 1, 1, 1, 0, 1)),
    ((10, 66, 52), (0, 1, 1, 0, 0, 1)),
    ((5, 130, 130), (0, 0, 0, 0, 0, 0)),
    ((6, 129, 122), (0, 0, 1, 1, 0, 0)),
    # past 128 interior nodes: halves that are not whole 16-row blocks or chunks, on
    # every axis, beside a plain long axis
    ((5, 143, 131), (0, 0, 1, 1, 0, 0)),
    ((163, 6, 140), (1, 1, 0, 0, 0, 1)),
    ((195, 4, 258), (0, 0, 0, 0, 1, 1)),
    ((7, 132, 5), (0, 0, 1, 1, 0, 1)),
    ((134, 5, 7), (0, 1, 1, 1, 0, 0)),
])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_precond_within_its_rounding(shape, bc, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan
    dt, nt, eps = (torch.float64, np.float64, 2.0 ** -53) if prec == "f64" else (torch.float32, np.float32, 2.0 ** -24)
    plan = Plan(shape, (0.0, 0.0, 0.0), EDGE, bc, prec)
    r = np.random.default_rng(sum(shape)).standard_normal(shape).astype(nt)
    A = [O.reduced_1d(O.diff_matrix(shape[a] - 1, 0.0, EDGE[a]), bc[2 * a], bc[2 * a + 1]) for a in range(3)]
    lam, V = zip(*(np.linalg.eig(M) for M in A))
    lam, V = [x.real for x in lam], [x.real for x in V]
    Vi = [np.linalg.inv(x) for x in V]
    den = lam[0][:, None, None] + lam[1][None, :, None] + lam[2][None, None, :]
    tol = eps * sum(len(x) * np.linalg.cond(x) for x in V) + 8 * 2.0 ** -53 * np.abs(den).max() / np.abs(den).min()
    assert tol < (1e-6 if prec == "f64" else 1e-3)
    for tr in (False, True):
        got = to_host(plan.precond(to_dev(r, dt), KC, transpose=tr))
        x = r[1:-1, 1:-1, 1:-1].astype(np.float64)
        for a in range(3):
            x = along(V[a].T if tr else Vi[a], x, a)
        x = x / (KC * den)
        for a in range(3):
            x = along(Vi[a].T if tr else V[a], x, a)
        e = np.linalg.norm(got[1:-1, 1:-1, 1:-1] - x) / np.linalg.norm(x)
        log(f"precond {prec} {shape} {bc} transpose={tr}: {e:.1e} of {tol:.1e}")
        assert e <= tol
        got[1:-1, 1:-1, 1:-1] = 0
        assert not got.any()
