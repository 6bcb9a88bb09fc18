"""What a batch holds on the device besides its workspace: tables per box, not a
field per system."""
import pytest

from tests.gpu_util import log, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bc", [((129, 129, 129), (0, 0, 1, 1, 1, 1)), ((100, 120, 140), (0, 1, 1, 1, 0, 0))])
def test_batch_holds_no_field_per_system(n, bc):
    require_gpu()
    import torch
    from paper_2606_21410_amd.api import Batch
    count = 24
    field = n[0] * n[1] * n[2] * 8
    grid = (n, (0.0,) * 3, (1.0,) * 3, bc)
    Batch([grid], "mixed")  # first use of the library and the device
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    batch = Batch([grid] * count, "mixed")
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    log(f"{count} systems of {n}: {held / 2**20:.1f} MiB, a field is {field / 2**20:.1f} MiB")
    assert held < count * field / 4
    del batch
