"""Statistics of a limited step against the oracle, on meshes with fewer, as many
and more blocks than the statistics accumulators they are spread over (64).

The counts are equal; the smallest factors and the mean low-order fractions agree
to 1e-10, the tolerance of the other statistics tests (the factors themselves are
compared at 1e-12 through the state, and a mean adds at most the rounding of its
sum, below 1e-12 at these sizes).  With local bounds the means are left out: in
the constant surroundings a factor is 1 where an increment is exactly zero and 0
where it is a rounding error, so they count roundings.  A second call gives the
same values: the accumulators start from zero each time."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import random_mesh, uniform_mesh

pytestmark = pytest.mark.gpu

MESHES = {"9 elements": lambda: uniform_mesh(3, 3, -2.0, -2.0, 4.0, 4.0),
          "256 elements": lambda: uniform_mesh(16, 16, -2.0, -2.0, 4.0, 4.0),
          "random, mortars": lambda: random_mesh(21, 16, 2, 0.4, L=4.0, x0=-2.0, y0=-2.0)}


@pytest.mark.parametrize("N", [3, 4])
@pytest.mark.parametrize("limiter", ["positivity", "local", "combined"])
@pytest.mark.parametrize("name", list(MESHES))
def test_statistics_match_the_oracle(oracle, name, limiter, N):
    import paper_2607_06045_amd as P
    spec = MESHES[name]()
    lim = {"positivity": (P.LIMIT_POSITIVITY, oracle.LIM_POSITIVITY), "local": (P.LIMIT_LOCAL, oracle.LIM_LOCAL),
           "combined": (P.LIMIT_COMBINED, oracle.LIM_COMBINED)}[limiter]
    M = oracle.Mesh(N, *spec.args())
    x, y, _ = M.geometry()
    u = states.sedov_tophat(x, y, r0=0.9)
    s = P.Solver(N, limiter=lim[0])
    s.set_mesh(*spec.args())
    _, ref = M.ssprk3(u, 0.9, limiter=lim[1])
    for _ in range(2):
        s.upload(u)
        st = s.step(0.9)
        print(f"stats {name} {limiter} N={N} gpu={st} oracle={ref}", flush=True)
        assert st["violations"] == ref["violations"] == 0
        assert st["fv_inadmissible"] == ref["fv_inadmissible"]
        assert abs(st["dt"] - ref["dt"]) <= 1e-13 * ref["dt"]
        means = ("alpha_vol_mean", "alpha_mort_mean") if limiter == "positivity" else ()
        for key in ("theta_vol_min", "theta_mort_min") + means:
            assert abs(st[key] - ref[key]) < 1e-10, key
    assert np.isfinite(ref["alpha_vol_mean"]) and ref["alpha_vol_mean"] > 0.0
