"""The two-point volume fluxes in every form of the logarithmic means, through the
high-order residual and one limited step against the oracle.

A wave takes the series where all its pairs have |f| < 1e-2, f = (x - y) / (x + y),
the polynomials where they have |f| < 0.171, and logarithms beyond.  The amplitudes
put all pairs of random states on the series (1e-4), around its edge, so that most
waves hold both kinds (1e-2, 2e-2), on the polynomials (0.08), around their edge
(0.17) and mostly beyond (0.6); the scales shift the logarithms' range
(a density and a pressure in other units).  Element counts of 1, 5 and 24 leave
the last block partly filled (blocks of 4 elements at N = 3, 5 at N = 4).
Tolerance 1e-12 in the metrics of parity.py, the bound of every other parity
test: both sides are FP64 and differ in the order of operations."""
import numpy as np
import pytest

from parity import rate_err, state_err
from workloads import states
from workloads.meshes import random_mesh, uniform_mesh
from workloads.rng import uniform

pytestmark = pytest.mark.gpu
TOL = 1e-12


def noisy(x, amp, rs, ps):
    k = np.arange(4 * x.size, dtype=np.uint64)
    U = 2.0 * uniform(31, k).reshape((4,) + x.shape) - 1.0
    c = np.sqrt(ps / rs)
    return states.conservative(rs * (1 + amp * U[0]), 0.3 * c * (1 + amp * U[2]), -0.2 * c * (1 + amp * U[3]),
                               ps * (1 + amp * U[1]), 1.4)


@pytest.mark.parametrize("N", [3, 4])
@pytest.mark.parametrize("flux", ["ranocha", "chandrashekar"])
@pytest.mark.parametrize("amp", [1e-4, 1e-2, 2e-2, 0.08, 0.17, 0.6])
@pytest.mark.parametrize("rs,ps", [(1.0, 1.0), (1e-9, 3e4), (7e8, 2e-7)])
def test_pair_flux_forms(oracle, rs, ps, amp, flux, N):
    import paper_2607_06045_amd as P
    for spec in (uniform_mesh(1, 1), uniform_mesh(5, 1, Lx=5.0), uniform_mesh(6, 4, Lx=1.5), random_mesh(9, 4, 2, 0.4)):
        M = oracle.Mesh(N, *spec.args(), volume_flux=flux)
        s = P.Solver(N, volume_flux=P.FLUX_CHANDRASHEKAR if flux == "chandrashekar" else P.FLUX_RANOCHA)
        s.set_mesh(*spec.args())
        x, y, _ = M.geometry()
        u = noisy(x, amp, rs, ps)
        s.upload(u)
        w0 = 2.0 / (N * (N + 1))
        err = rate_err(s.rhs(P.RHS_HIGH), M.rhs(u), u, x, y, w0)
        assert err < TOL, (spec.E, err)
        st = s.step(0.5)
        ref, _ = M.ssprk3(u, 0.5)
        es = state_err(s.download(), ref)
        print(f"pairs E={spec.E} N={N} {flux} amp={amp} rho {rs} p {ps}: rhs {err:.1e} step {es:.1e}", flush=True)
        assert es < TOL and st["violations"] == 0
