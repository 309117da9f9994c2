"""sht_delta2map of a Delta larger than the last cache (256 MB a map), where the
ring kernel paces its loads: against the whole transform, whose Delta lies in
blocks of rings.  Bound of the other ring tests, 1e-13 log2 n of the largest
pixel: the same modes through transforms of log2 n levels."""
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


@pytest.mark.parametrize("gap", [False, True], ids=["all m", "a gap"])
def test_delta_past_the_cache(P, gap):
    print("[case] delta past the cache", gap, flush=True)
    sys.stdout.flush()
    lmax, nside = 4200, 2048
    mval = np.arange(lmax + 1, dtype=np.int32)
    if gap:
        mval = np.delete(mval, [3, 4, 1700])
    plan = P.Plan(lmax, W.healpix_geometry(nside), mval=mval)
    assert plan.nm * plan.nrings * 16 > 256 << 20
    gen = torch.Generator(device="cuda:0").manual_seed(841)
    a = torch.randn((1, plan.nalm, 2), dtype=torch.float64, device="cuda:0", generator=gen)
    a = torch.view_as_complex(a)
    whole = plan.alm2map(a)
    stage = plan.delta2map(plan.alm2delta(a))
    err = (whole - stage).abs().max().item()
    assert err < 1e-13 * np.log2(4 * nside + 1) * whole.abs().max().item()
