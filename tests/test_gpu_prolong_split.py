"""The even-odd prolongation at the sizes where its tiling can go wrong: the
mirrored middle node (even and odd degrees, coarse and fine), remainders of a
contraction step, of its load group and of a 16-row block, one and several row
groups, a last task of few pencils, and the launch with three row blocks."""
import numpy as np
import pytest

from tests.gpu_util import log, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu


def matrix(Nc, Nf):
    """Coarse coefficients, then the fine cosine sum, in long double."""
    L = np.longdouble
    pi = L("3.14159265358979323846264338327950288")
    k = np.arange(Nc + 1)
    c = np.cos((np.outer(k, k) % (2 * Nc)).astype(L) * pi / L(Nc)) * 2 / L(Nc)
    c[:, 0] /= 2
    c[:, -1] /= 2
    c[0] /= 2
    c[-1] /= 2
    return np.cos((np.outer(np.arange(Nf + 1), k) % (2 * Nf)).astype(L) * pi / L(Nf)) @ c


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("nc,nf", [
    ((5, 6, 7), (5, 7, 11)), ((8, 9, 10), (31, 32, 33)), ((17, 18, 16), (34, 63, 64)),
    ((64, 65, 3), (65, 66, 130)), ((3, 66, 67), (97, 129, 68)), ((4, 134, 5), (4, 140, 193)),
    ((260, 190, 20), (260, 190, 70))])
def test_prolong_tiles(nc, nf, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Plan, prolong
    dt = torch.float64 if prec == "f64" else torch.float32
    log(f"prolong {prec} {nc} -> {nf}")
    u = np.random.default_rng(sum(nc)).standard_normal(nc)
    u = u.astype(np.float64 if prec == "f64" else np.float32)
    box = ((0.0, 0.0, 0.0), (1.0, 1.0, 1.0))
    pc, pf = (Plan(n, *box, precision=prec) for n in (nc, nf))
    uf = to_host(prolong(pc, pf, to_dev(u, dt))[0])
    ref = u.astype(np.longdouble)
    for a in (2, 1, 0):
        if nc[a] != nf[a]:
            ref = np.moveaxis(np.tensordot(matrix(nc[a] - 1, nf[a] - 1), ref, (1, a)), 0, a)
    # the rounding of a dot product of the pairs, per axis, on values that the
    # axes' Lebesgue constants bound; plus, in f32, that of three stored fields
    leb = np.prod([1 + 2 / np.pi * np.log(m) for m in nc])
    tol = (2.0 ** -53 * sum(m / 2 + 16 for m in nc) + (3 * 2.0 ** -24 if prec == "f32" else 0)) * leb
    assert np.max(np.abs(uf - ref)) <= tol * np.max(np.abs(u))
