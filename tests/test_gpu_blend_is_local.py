"""The blend of positivity and local factors with weight 1 in every element is local
limiting: theta = (1 - w) theta_pos + w theta_local.  In a gas of constant density whose
pressure jumps inside every element the shock indicator is 1 to the last bit (its
exponent is below -100), and the bounds have no width in many places, so a node's factor
is a quotient of rounding errors: the two modes agree only if they do the same operations
in the same order.  They do, so one limited forward-Euler step has to give equal states and
smallest factors."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import random_mesh, uniform_mesh

pytestmark = pytest.mark.gpu

MESHES = {"uniform": lambda: uniform_mesh(24, 20, 0.0, 0.0, 1.0, 1.0),
          "random, mortars": lambda: random_mesh(7, 16, 2, 0.4, L=1.0, x0=0.0, y0=0.0)}


def state(x, y, shear, pattern):
    one = np.ones_like(x)
    j, e = np.arange(x.shape[1])[None, :, None] * one, np.arange(len(x))[:, None, None] * one
    p = np.where(j < x.shape[1] / 2, 1.0, 0.1) if pattern == "layers" else np.where((j + e) % 3 == 0, 1.0, 0.2)
    v1 = 0.3 * np.sin(2 * np.pi * y) if shear else 0.3 * one
    return states.conservative(one, v1, 0.1 * np.sin(2 * np.pi * x), p, 1.4)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("pattern", ["layers", "thirds"])
@pytest.mark.parametrize("shear", [False, True])
@pytest.mark.parametrize("name", list(MESHES))
@pytest.mark.parametrize("N", [3, 4])
def test_blend_of_weight_one_is_local_limiting(N, name, shear, pattern, precision):
    import paper_2607_06045_amd as P
    got = []
    for limiter in (P.LIMIT_LOCAL, P.LIMIT_COMBINED):
        s = P.Solver(N, limiter=limiter, precision=P.MIXED if precision == "mixed" else P.FP64)
        s.set_mesh(*MESHES[name]().args())
        s.upload(state(*s.node_coords(), shear, pattern))
        st = s.limit(s.max_dt(0.5))
        got.append((s.download(), st))
    (a, sa), (b, sb) = got
    print(f"N={N} {name} shear={shear} {pattern} {precision} difference {np.abs(a - b).max():.1e} {sa} {sb}", flush=True)
    assert np.array_equal(a, b)
    assert sa["theta_vol_min"] == sb["theta_vol_min"] < 1.0
    assert sa["dt"] == sb["dt"]
