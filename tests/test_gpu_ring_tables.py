"""Rings of one Bluestein length on different paths keep kernel spectra of
their own: n = L and 2 L (odd L with a prime factor above 7) run by size class
and n = 4 L on the two-convolution path, all three with chirps of length L but
not always with the same convolution length.

Bound of the other ring tests: 1e-13 log2 n of the largest output in FP64
(three transforms of log2 n levels).  The mixed forms' passes are complex64
with FP64 folds: the same count of roundings at 2^-24, 1e-13 * 2^29."""
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


# convolution lengths by size class / two-convolution FP64 / mixed: 401 840 /
# 896 / 840, 479 960 / 1024 / 960, 131 the same everywhere
@pytest.mark.parametrize("order", [1, -1])
@pytest.mark.parametrize("prec", ["fp64", "f16x2_mfma"])
@pytest.mark.parametrize("L", [131, 401, 479])
def test_one_bluestein_length_on_every_path(P, L, prec, order):
    print("[case] spectra", L, prec, order, flush=True)
    sys.stdout.flush()
    n = np.array([L, 2 * L, 4 * L], np.int64)[::order]
    lmax, nr = 100, len(n)
    cth = np.array([0.6, 0.3, 0.1])
    start = np.concatenate([[0], np.cumsum(n)[:-1]])
    geo = W.Geometry(cth, np.sqrt(1 - cth ** 2), np.array([0.25, 0.0, 0.5]), n, start, int(n.sum()))
    mval = np.arange(lmax + 1)
    plan = P.Plan(lmax, geo, nmaps=2, precision=prec)
    a = np.stack([W.random_alm(lmax, [831, L, i]) for i in range(2)])
    alm = torch.from_numpy(a).to("cuda:0")
    got = plan.alm2map(alm).cpu().numpy()
    d = plan.alm2delta(alm)
    stage = plan.delta2map(d).cpu().numpy()          # FP64 on every plan
    g = np.random.default_rng(L).standard_normal((2, geo.npix))
    dt = plan.map2delta_adjoint(torch.from_numpy(g).to("cuda:0")).cpu().numpy()
    unit = 1e-13 * np.log2(n.max() + 1)
    for i in range(2):
        e = ref.map_from_delta(mval, geo, d.cpu().numpy()[i].T)
        for r in range(nr):
            p = slice(int(start[r]), int(start[r] + n[r]))
            top = np.max(np.abs(e[p]))
            assert np.max(np.abs(got[i, p] - e[p])) < unit * top * (1 if prec == "fp64" else 2 ** 29)
            assert np.max(np.abs(stage[i, p] - e[p])) < unit * top
            x = ref.ring_analysis(g[i, p], mval, geo.phi0[r])
            assert np.max(np.abs(dt[i, :, r] - x)) < unit * np.max(np.abs(x))
