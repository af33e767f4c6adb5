"""The time step on either side of the size from which its kernel takes rows and
columns of nodes per lane (40,960 elements), against the oracle: periodic and mixed
boundaries, mortars, both estimates, numbers of elements that leave the last wave
and the last block ragged.  One element at a time is given 40 times its energy, so
that the maximum lies at many places.  Tolerance 1e-13, as in the other parity tests
(both sides are FP64 and differ in the order of operations)."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import build

pytestmark = pytest.mark.gpu

G = 1.4


@pytest.mark.parametrize("nx,ny", [(195, 201), (203, 202), (211, 203)])
@pytest.mark.parametrize("bc", [[0, 0, 0, 0], [2, 3, 1, 1]])
@pytest.mark.parametrize("N", [3, 4])
def test_dt_by_size(oracle, N, bc, nx, ny):
    import paper_2607_06045_amd as P
    spec = build((0.0, 0.0, 1.0, 1.0, nx, ny), lambda x, y, l: (x - 0.4) ** 2 + (y - 0.6) ** 2 < 4e-3, 1)
    ext = np.tile(states.conservative(*[np.array([q]) for q in (1.2, 0.7, -0.4, 0.9)], G)[0], (4, 1))
    M = oracle.Mesh(N, *spec.args(), bc=bc, ext=ext)
    x, y, _ = M.geometry()
    u = states.conservative(1.0 + 0.3 * np.sin(6 * x) * np.cos(5 * y), 1.3 * np.sin(4 * y), -1.1 * np.cos(7 * x),
                            1.0 + 0.2 * np.cos(9 * x * y), G)
    rng = np.random.default_rng(nx)
    # places: the first and last elements, the refined ones and their neighbours, the rest
    fine = np.flatnonzero(spec.level == 1)
    at = np.concatenate([[0, 1, 47, 48, 63, 64, M.E - 2, M.E - 1], rng.choice(fine, 4), rng.choice(M.E, 6)])
    for mode, omode in ((P.DT_IDP, oracle.DT_IDP), (P.DT_LOWORDER, oracle.DT_LOWORDER)):
        s = P.Solver(N, bc=bc, ext=ext, dt_mode=mode)
        s.set_mesh(*spec.args())
        assert s.E == M.E
        for e in at:
            w = u.copy()
            w[e, 3] *= 40.0
            s.upload(w)
            dg, dc = s.max_dt(0.9), M.max_dt(w, 0.9, mode=omode)
            assert abs(dg - dc) <= 1e-13 * dc, (N, bc, nx, ny, mode, int(e), dg, dc)
