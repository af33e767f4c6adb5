"""The scheme has no units: density times 2^i and pressure times 2^j (velocities times
2^((j - i) / 2)) give the same flow in powers of two, so a step is the plain one's, scaled, up
to where a number of the scheme leaves the range of doubles.  The pairs reach rho^2 / p of
2^-1680 and 2^1680 and its neighbourhood of 2^-1022 and 2^1024, with p / rho (the squared
sound speed) between 2^-960 and 2^960 and rho E, whose square the pressure factor needs,
between 2^-480 and 2^360.  Tolerance 1e-12 as in the other
parity tests: where a product would leave the range other forms of the same means are taken,
which differ by rounding."""
import numpy as np
import pytest

from workloads import states
from workloads.meshes import random_mesh

pytestmark = pytest.mark.gpu

PAIRS = [(-720, 240), (-600, 360), (-480, 480), (-360, 480), (-341, 341), (-341, 343), (-340, 340), (-340, 346), (-240, 600),
         (240, -600), (340, -340), (340, -342), (341, -341), (342, -340), (360, -480), (480, -480), (600, -360), (720, -240)]


@pytest.mark.parametrize("flux", ["ranocha", "chandrashekar"])
@pytest.mark.parametrize("limiter", ["positivity", "none"])
@pytest.mark.parametrize("N", [3, 4])
def test_a_step_in_other_units(N, limiter, flux):
    import paper_2607_06045_amd as P
    s = P.Solver(N, limiter=P.LIMIT_POSITIVITY if limiter == "positivity" else P.LIMIT_NONE,
                 volume_flux=P.FLUX_RANOCHA if flux == "ranocha" else P.FLUX_CHANDRASHEKAR)
    s.set_mesh(*random_mesh(7, 8, 1, 0.4, L=1.0, x0=0.0, y0=0.0).args())
    x, y = s.node_coords()
    one = np.ones_like(x)
    top = 1.0 if limiter == "positivity" else 0.1  # (smooth enough without limiting)
    p = 0.01 + top * ((x - 0.5) ** 2 + (y - 0.5) ** 2 < 0.05) if limiter == "positivity" else 1.0 + 0.5 * np.sin(2 * np.pi * y)
    u = states.conservative(1.0 + 0.3 * np.sin(2 * np.pi * x), 0.3 * np.sin(2 * np.pi * y), 0.2 * one, p * one, 1.4)
    s.upload(u)
    dt = s.step(0.5)["dt"]
    ref = s.download()
    scale = np.abs(ref).max(axis=(0, 2, 3))[None, :, None, None]
    for i, j in PAIRS:
        i, j = i, j + (i + j) % 2  # (an even sum: momenta by a power of two)
        unit = np.array([2.0 ** i, 2.0 ** ((i + j) // 2), 2.0 ** ((i + j) // 2), 2.0 ** j])[None, :, None, None]
        s.upload(u * unit)
        st = s.step(0.5)
        err = np.max(np.abs(s.download() / unit - ref) / scale)
        print(f"N={N} {limiter} {flux} rho 2^{i} p 2^{j} rho^2/p 2^{2 * i - j}: err {err:.1e}", flush=True)
        assert err < 1e-12
        assert abs(st["dt"] / (dt * 2.0 ** ((i - j) // 2)) - 1.0) < 1e-13 and st["violations"] == 0
