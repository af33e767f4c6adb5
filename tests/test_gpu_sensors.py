"""GPU modal indicator, features and learned indicator on element counts at the
edges of their split: a wave takes 16 elements at N = 3 and 12 at N = 4 (the
learned indicator twice as many), a block four waves.  Against the oracle;
outputs are FP32, computed in FP64 and rounded once: 2^-24 relative plus FP64
round-off (the indicator is at most 0.5; its cut at 1e-3 is compared only away
from it).  The learned indicator equals the stand-alone network on the
stand-alone features bit for bit."""
import numpy as np
import pytest

from oracle import indicator as IND
from oracle import mlp as MLP
from workloads import states
from workloads.meshes import uniform_mesh

pytestmark = pytest.mark.gpu

SIZES = {3: [(5, 3), (4, 4), (17, 1), (11, 3), (9, 7), (13, 5), (43, 3)],
         4: [(11, 1), (4, 3), (13, 1), (5, 5), (7, 7), (19, 5), (97, 1)]}


@pytest.mark.parametrize("N,nx,ny", [(N, nx, ny) for N in SIZES for nx, ny in SIZES[N]])
def test_sensors_at_tile_edges(N, nx, ny):
    import paper_2607_06045_amd as P
    s = P.Solver(N)
    s.set_mesh(*uniform_mesh(nx, ny).args())
    x, y = s.node_coords()
    u = states.random_admissible(x, nx + ny)
    s.upload(u)
    T = IND.threshold(N)
    raw = 1.0 / (1.0 + np.exp(-(np.log(9999.0) / T) * (IND.hennemann_energy(u, N) - T)))
    away = np.abs(raw - IND.ALPHA_MIN) > 1e-9
    a = s.indicator(P.IND_HENNEMANN)
    assert a.shape == (nx * ny,)
    assert np.abs(a - IND.hennemann(u, N))[away].max(initial=0.0) <= 2.0 ** -24 * 0.5 + 1e-12
    f = s.features()
    assert np.abs(f - IND.features(u, N)).max() <= 2.0 ** -24 + 1e-12
    w = MLP.init(7)
    s.mlp_set_weights(w)
    assert np.array_equal(s.indicator(P.IND_MLP), s.mlp_forward(f))
