"""A stage of two launches, the second of which starts with the corrections of the
first one's mortars (from 16,384 element batches of 4 at N = 3 and of 5 at N = 4, with at
most an eighth of them holding a mortar): one refined element, whose 4 mortars fill
a fraction of one block, and a refined box with a batch of mortars per wave.  One
step with statistics against the oracle, one without against the first.  Smooth data;
tolerance 1e-12 per DOF and 1e-13 on dt, as in the other parity tests (both sides are
FP64 and differ in the order of operations)."""
import numpy as np
import pytest

from parity import state_err
from workloads import states
from workloads.meshes import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nx,ny,box", [(3, 257, 256, 1), (3, 264, 258, 33), (4, 321, 256, 1), (4, 330, 256, 33)])
def test_step_of_two_launches(oracle, N, nx, ny, box):
    import paper_2607_06045_amd as P
    cx, cy = (nx // 2 + 0.5) / nx, (ny // 2 + 0.5) / ny  # an element's centre
    h, k = 0.5 * box / nx, 0.5 * box / ny
    spec = build((0.0, 0.0, 1.0, 1.0, nx, ny), lambda x, y, l: abs(x - cx) < h and abs(y - cy) < k, 1)
    s = P.Solver(N)
    s.set_mesh(*spec.args())
    assert s.M >= 4 * box
    M = oracle.Mesh(N, *spec.args())
    x, y, _ = M.geometry()
    u = states.density_wave(x, y)
    s.upload(u)
    st = s.step(0.5)
    a = s.download()
    ref, sref = M.ssprk3(u, 0.5)
    err = state_err(a, ref)
    print(f"{nx}x{ny} N={N} E={s.E} M={s.M} err={err:.2e} dt={st['dt']!r}", flush=True)
    assert abs(st["dt"] - sref["dt"]) <= 1e-13 * sref["dt"]
    assert st["violations"] == 0 and st["fv_inadmissible"] == 0
    assert err < 1e-12
    s.upload(u)
    s.step(0.5, stats=False)
    assert np.array_equal(s.download(), a)
