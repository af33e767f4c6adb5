"""Statistics of a stage of two launches, whose mortars are corrected by the first blocks of
the second: a blast with its edge on the border of a refined box, so that volume and mortar
factors below 1 are among those counted.  Against the oracle: equal counts, the smallest
factors and the mean low-order fractions to 1e-10, dt to 1e-13 and the state to 1e-12 per
DOF, the tolerances of the tests of small meshes (a mean of these sums, a few thousand
numbers other than zero, adds less than 1e-12)."""
import numpy as np
import pytest

from parity import state_err
from workloads import states
from workloads.meshes import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nx,ny", [(3, 264, 258), (4, 330, 256)])
def test_statistics_of_two_launches(oracle, N, nx, ny):
    import paper_2607_06045_amd as P
    h = 16.5 / ny  # the box: 33 x 33 elements, 2 * 33 on the finer level
    spec = build((-0.5 * nx / ny, -0.5, nx / ny, 1.0, nx, ny), lambda x, y, l: abs(x) < h and abs(y) < h, 1)
    s = P.Solver(N)
    s.set_mesh(*spec.args())
    assert s.M >= 100
    M = oracle.Mesh(N, *spec.args())
    x, y, _ = M.geometry()
    u = states.sedov_tophat(x, y, r0=1.02 * h)
    s.upload(u)
    st = s.step(0.9)
    ref, sref = M.ssprk3(u, 0.9)
    err = state_err(s.download(), ref)
    print(f"N={N} E={s.E} M={s.M} err={err:.2e} gpu={st} oracle={sref}", flush=True)
    assert abs(st["dt"] - sref["dt"]) <= 1e-13 * sref["dt"]
    assert st["violations"] == sref["violations"] == 0 and st["fv_inadmissible"] == sref["fv_inadmissible"]
    for key in ("theta_vol_min", "theta_mort_min", "alpha_vol_mean", "alpha_mort_mean"):
        assert abs(st[key] - sref[key]) < 1e-10, key
    assert st["theta_vol_min"] < 1.0 and st["theta_mort_min"] < 1.0
    assert st["alpha_vol_mean"] > 0.0 and st["alpha_mort_mean"] > 0.0
    assert err < 1e-12
