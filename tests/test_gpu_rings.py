"""Even rings of FP64 plans on the register-held paths, in both directions:
half lengths h = 2 len with a len that has a prime factor above 7, at the
edges of the convolution classes (h - 1 <= 1024, 2048, 4096) and of the direct
DFT (h <= 64), and 7-smooth ones that the fast path refuses.

The synthesis is taken through the whole transform, whose own Delta goes
through these kernels, and compared with the oracle's ring sum of the plan's
Delta. Tolerance, of the largest output (which is no less than their rms): a
convolution is three transforms of at most log2(n) + 1 butterfly levels, each
of which adds a few units of 2^-53 to the rms error, and the largest of 8000
errors lies within 5 rms: below 300 units per log2(n) of both sides together,
1e-13 for short."""
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


def _dev():
    return torch.device("cuda", 0)


HALVES = [22, 62, 74, 2 * 509, 2 * 513, 2 * 1021, 2 * 1025, 2 * 2039, 2 * 2051,
          686, 2058, 3430, 3750]
MSETS = [np.arange(301), np.r_[0, 3, 4, 150:290:7, 300]]


@pytest.mark.parametrize("mval", MSETS, ids=["all m", "some m"])
@pytest.mark.parametrize("half", HALVES)
def test_even_rings_both_directions(P, half, mval):
    print("[case] even ring", half, len(mval), flush=True)
    sys.stdout.flush()
    n, lmax, nr, nmaps = 2 * half, 300, 5, 3
    cth = np.array([0.92, 0.6, 0.0, -0.6, -0.92])
    geo = W.Geometry(cth, np.sqrt(1 - cth ** 2),
                     np.array([0.37, 0.0, np.pi / n, 0.0, 1.1]),
                     np.full(nr, n, np.int64), np.arange(nr) * n, nr * n)
    mval = mval.astype(np.int32)
    plan = P.Plan(lmax, geo, mval=mval, nmaps=nmaps)
    a = np.stack([W.random_alm(lmax, [811, half, i], mval=mval) for i in range(nmaps)])
    alm = torch.from_numpy(a).to(_dev())
    got = plan.alm2map(alm).cpu().numpy()
    d = plan.alm2delta(alm).cpu().numpy()                  # [map][m][ring]
    tol = 1e-13 * np.log2(n + 1)
    for i in range(nmaps):
        e = ref.map_from_delta(mval, geo, d[i].T)
        assert np.max(np.abs(got[i] - e)) < tol * np.max(np.abs(e))
    g = np.random.default_rng(half).standard_normal((nmaps, nr * n))
    dt = plan.map2delta_adjoint(torch.from_numpy(g).to(_dev())).cpu().numpy()
    for i in range(nmaps):
        for r in range(nr):
            e = ref.ring_analysis(g[i, r * n:(r + 1) * n], mval, geo.phi0[r])
            assert np.max(np.abs(dt[i, :, r] - e)) < tol * np.max(np.abs(e))
