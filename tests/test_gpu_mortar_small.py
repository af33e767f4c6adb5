"""Mortar factors where a node's density increment is next to nothing: a gas of constant
density and pressure with momenta of `scale`, so that every increment is a rounding
error of the constant state (below 1e-15 of it) or a number of the momenta's size,
down to subnormal ones.  Against floors of a tenth of the state each admits the full
step, so every factor is exactly 1 and the oracle's as well."""
import numpy as np
import pytest

from workloads.meshes import build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1e-300, 1e-306, 1e-309, 1e-312, 1e-315])
@pytest.mark.parametrize("N", [3, 4])
def test_full_step_for_a_tiny_density_increment(oracle, N, scale):
    import paper_2607_06045_amd as P
    spec = build((0.0, 0.0, 1.0, 1.0, 6, 6), lambda x, y, l: abs(x - 0.42) < 0.05 and abs(y - 0.42) < 0.05, 1)
    s = P.Solver(N)
    s.set_mesh(*spec.args())
    assert s.M == 4
    x, y = s.node_coords()
    one = np.ones_like(x)
    u = np.stack([one, scale * np.sin(7 * x + 3 * y), scale * np.cos(5 * x - 2 * y), 2.5 * one], axis=1)
    s.upload(u)
    dt = s.max_dt(0.5)
    st = s.limit(dt)
    theta = oracle.Mesh(N, *spec.args()).fe_step_detail(u, dt)[4]
    print(f"N={N} scale={scale:g} {st} oracle {theta}", flush=True)
    assert np.all(theta == 1.0)
    assert st["theta_mort_min"] == 1.0 and st["alpha_mort_mean"] == 0.0
    assert st["theta_vol_min"] == 1.0 and st["violations"] == 0
