"""Mixed forms' Legendre waves four to a workgroup (where a launch has about one
wave per SIMD: more than 768 and up to 1152 of them on 256 CUs) and one each: a
wave's arithmetic does not depend on the waves beside it, so a map comes out the
same to the bit."""
import sys

import numpy as np
import pytest

import workloads as W
from oracle import ref

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1010_1260_amd as P
    return P


# 7 blocks of ring pairs (nside 200) x m-pairs: 112 784 waves, 128 896, 146 1022, 160
# (odd m count) 1120 for 16 maps; 33 maps have two groups of 16 in one launch, twice
# as many waves, and one map more
@pytest.mark.parametrize("prec", ["fp32_mfma", "bf16x3_mfma", "f16x2_mfma"])
@pytest.mark.parametrize("nm", [223, 256, 292, 319])
def test_waves_four_to_a_workgroup(P, prec, nm):
    print("[case] waves per workgroup", prec, nm, flush=True)
    sys.stdout.flush()
    lmax, g = 320, W.healpix_geometry(200)
    mval = np.arange(nm, dtype=np.int32)
    a = np.stack([W.random_alm(lmax, [861, i], mval=mval) for i in range(33)])
    alm = torch.from_numpy(a).to("cuda:0")
    few = P.Plan(lmax, g, mval=mval, nmaps=16, precision=prec).alm2delta(alm[:16].contiguous())
    many = P.Plan(lmax, g, mval=mval, nmaps=33, precision=prec).alm2delta(alm)
    assert torch.equal(few, many[:16])
    e = ref.delta(lmax, mval, g.cth, g.sth, a[15]).T
    assert np.linalg.norm(few[15].cpu().numpy() - e) <= 1e-6 * np.linalg.norm(e)
