"""Upload and download of a device state: element reordering in 16-byte words where
both addresses allow it, in 8-byte words otherwise; numbers of values around the
2,048 (1,024) of a block.  Bytes have to come back unchanged."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import uniform_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [3, 4])
@pytest.mark.parametrize("nx,ny", [(1, 1), (3, 5), (16, 1), (41, 1), (13, 5), (64, 3)])
def test_device_round_trip(N, nx, ny):
    import torch
    import paper_2607_06045_amd as P
    s = P.Solver(N)
    s.set_mesh(*uniform_mesh(nx, ny).args())
    x, y = s.node_coords()
    u = states.random_admissible(x, nx)
    s.upload(u)
    assert np.array_equal(s.download(), u)
    for shift in (0, 1):  # 16-byte aligned, 8-byte aligned
        buf = torch.zeros(u.size + 2, dtype=torch.float64, device="cuda")
        v = buf[shift:shift + u.size].view(u.shape)
        v.copy_(torch.from_numpy(u))
        assert v.data_ptr() % 16 == 8 * shift
        s.upload(2.0 * u)
        s.upload(v)
        assert np.array_equal(s.download(), u)
        assert torch.equal(s.download(device=True).cpu(), torch.from_numpy(u))
