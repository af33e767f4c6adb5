"""A step of the local limiting modes on a mesh of at least 16,384 element batches (of 4 at
N = 3, of 5 at N = 4), whose dt is reduced by a kernel of its own, and of one batch fewer:
the same bits as a step with the dt that the host reduces, since both divide the CFL number
by the same maximum."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import uniform_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limiter", ["combined", "local", "lowsol"])
@pytest.mark.parametrize("N,nx,ny", [(3, 256, 256), (3, 276, 237), (4, 320, 256), (4, 315, 260)])
def test_step_with_reduced_dt(N, nx, ny, limiter):
    import paper_2607_06045_amd as P
    kw = {"combined": dict(limiter=P.LIMIT_COMBINED), "local": dict(limiter=P.LIMIT_LOCAL),
          "lowsol": dict(limiter=P.LIMIT_LOCAL_LOWORDER, dt_mode=P.DT_LOWORDER)}[limiter]
    s = P.Solver(N, **kw)
    s.set_mesh(*uniform_mesh(nx, ny, -1.0, -1.0, 2.0, 2.0).args())
    x, y = s.node_coords()
    u = states.sedov_tophat(x, y, r0=0.3, p0=0.01)
    s.upload(u)
    st = s.step(0.4)
    a = s.download()
    s.upload(u)
    dt = s.max_dt(0.4)
    s.step_dt(dt)
    b = s.download()
    s.upload(u)
    s.step(0.4, stats=False)
    print(f"N={N} {nx}x{ny} {limiter} dt {st['dt']!r} {dt!r} difference {np.abs(a - b).max():.1e}", flush=True)
    assert st["dt"] == dt
    assert np.array_equal(a, b) and np.array_equal(s.download(), a)
    assert not np.array_equal(a, u)
