"""Analysis of a mixed-form plan on either side of the rule that sends its
smooth rings to the size classes (up to 2048 pixels; from 7 maps on, or below
1200 rings over all maps): it is FP64 on every plan, so it agrees with an FP64
plan's to the bound of the ring tests, 1e-13 log2 n of the largest mode."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1010_1260_amd as P
    return P


# rings over all maps 1199 and 1596; 7 maps; rings of 2048 and 2052 pixels
@pytest.mark.parametrize("nside,nmaps", [(300, 1), (200, 2), (200, 7), (512, 7), (513, 1)])
def test_analysis_of_a_mixed_plan(P, nside, nmaps):
    print("[case] mixed analysis", nside, nmaps, flush=True)
    sys.stdout.flush()
    g, lmax = W.healpix_geometry(nside), nside // 2
    m = np.random.default_rng(nside).standard_normal((nmaps, g.npix))
    m = torch.from_numpy(m).to("cuda:0")
    w = 1.0 + np.arange(g.nrings) / g.nrings
    a = P.Plan(lmax, g, nmaps=nmaps, precision="fp32_mfma")
    b = P.Plan(lmax, g, nmaps=nmaps)
    tol = 1e-13 * np.log2(4 * nside + 1)
    for x, y in ((a.map2delta_adjoint(m), b.map2delta_adjoint(m)),
                 (a.alm2map_adjoint(m), b.alm2map_adjoint(m)),
                 (a.map2alm(m, w), b.map2alm(m, w))):
        assert (x - y).abs().max().item() < tol * y.abs().max().item()
