"""Adaptation of a mesh whose arrays, some 70 bytes a leaf, are more than the 32 MiB that go
to the device through page-locked memory in one copy, and of one with less: the next step
is bit for bit that of a solver which is given the new leaves and the new state."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import MeshSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 720])
def test_step_after_adaptation(n):
    import paper_2607_06045_amd as P
    iy, ix = (a.ravel().astype(np.int32) for a in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    spec = MeshSpec(np.zeros(n * n, np.int8), ix, iy, 0.0, 0.0, 1.0, 1.0, n, n)
    s = P.Solver(3)
    s.set_mesh(*spec.args())
    s.upload(states.density_wave(*s.node_coords()))
    s.step(0.5)
    box = (abs(ix - n // 2) < 20) & (abs(iy - n // 3) < 20)
    st = s.refine_coarsen(box.astype(np.int8))
    assert st["n_refined"] == box.sum() and s.E == n * n + 3 * box.sum()
    u = s.download()
    t = P.Solver(3)
    t.set_mesh(*s.mesh(), 0.0, 0.0, 1.0, 1.0, n, n)
    t.upload(u)
    a, b = s.step(0.5), t.step(0.5)
    print(f"{n}x{n} E={s.E} M={s.M} dt {a['dt']!r} {b['dt']!r}", flush=True)
    assert s.M == t.M > 0 and a["dt"] == b["dt"]
    assert np.array_equal(s.download(), t.download())
    # and back again
    level = s.mesh()[0]
    st = s.refine_coarsen(np.where(level == 1, -1, 0).astype(np.int8))
    assert st["n_coarsened"] > 0 and s.E == n * n
