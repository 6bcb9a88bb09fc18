"""The long axes' contraction kernel as a plain GEMM at the edges of its 64 x 64
tiles and 16-wide chunks."""
import numpy as np
import pytest

from tests.gpu_util import log, require_gpu, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 15, 65), (64, 16, 64), (65, 17, 63), (129, 200, 130)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_gemm_tiles(shape, prec):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import debug_gemm
    I, K, C = shape
    log(f"gemm {shape} {prec}")
    r = np.random.default_rng(I + K + C)
    dt, nt, eps = (torch.float64, np.float64, 2.0 ** -53) if prec == "f64" else (torch.float32, np.float32, 2.0 ** -24)
    A, B = r.standard_normal((I, K)).astype(nt), r.standard_normal((K, C)).astype(nt)
    D = to_host(debug_gemm(to_dev(A, dt), to_dev(B, dt)))
    ref = A.astype(np.longdouble) @ B.astype(np.longdouble)
    # K roundings per dot product, against the sums of magnitudes
    assert np.all(np.abs(D - ref) <= (K + 1) * eps * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)))
