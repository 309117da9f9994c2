"""Infinite and NaN inputs reach what a sum over all terms would give them to,
also past the terms that the start table leaves out: a coefficient every pixel
of its map (and every ring of its Delta_m), a pixel every coefficient of its
map; and nothing else."""
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


def _say(*a):
    print("[case] non-finite", *a, flush=True)
    sys.stdout.flush()


LMAX = 700      # sin(theta)^700 of the first rings is far below 2^-960
MSETS = {"all": None, "gaps": np.r_[3, 7, 300, 650:701].astype(np.int32)}


def _bad(x):
    return ~np.isfinite(x)


def _geo():
    """The ten rings next to either pole, some between, and the equator."""
    g = W.healpix_geometry(350)
    R = g.nrings
    i = np.r_[0:10, 200, 349, 500, R // 2, R - 501, R - 10:R]
    n = g.nphi[i].copy()
    start = np.concatenate([[0], np.cumsum(n)[:-1]]).astype(np.int64)
    return W.Geometry(g.cth[i].copy(), g.sth[i].copy(), g.phi0[i].copy(), n, start, int(n.sum()))


def _places(mval):
    """(index in the set, l): the first and last of an m, the first m, dead ones."""
    n = len(mval)
    return [(0, mval[0]), (0, LMAX), (n // 2, mval[n // 2]), (n - 1, LMAX), (n - 2, LMAX)]


def _off(mval, i, l):
    return int(np.sum(LMAX + 1 - mval[:i])) + l - int(mval[i])


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("mset", list(MSETS))
@pytest.mark.parametrize("nmaps", [1, 12])
def test_coefficient(P, nmaps, mset, value):
    _say("coefficient", nmaps, mset, value)
    mval = MSETS[mset] if MSETS[mset] is not None else np.arange(LMAX + 1, dtype=np.int32)
    plan = P.Plan(LMAX, _geo(), mval=mval, nmaps=nmaps)
    a = np.stack([W.random_alm(LMAX, [851, i], mval=mval) for i in range(nmaps)])
    clean = torch.from_numpy(a).to("cuda:0")
    m0, d0 = plan.alm2map(clean).cpu().numpy(), plan.alm2delta(clean).cpu().numpy()
    assert np.all(np.isfinite(m0)) and np.all(np.isfinite(d0))
    for k, (i, l) in enumerate(_places(mval)):
        b = k % nmaps
        x = a.copy()
        x[b, _off(mval, i, l)] = value
        alm = torch.from_numpy(x).to("cuda:0")
        m, d = plan.alm2map(alm).cpu().numpy(), plan.alm2delta(alm).cpu().numpy()
        rest = np.arange(nmaps) != b
        assert np.all(_bad(m[b])), (i, l)
        assert np.array_equal(m[rest], m0[rest])
        assert np.all(_bad(d[b, i])), (i, l)
        d[b, i] = d0[b, i]
        assert np.array_equal(d, d0)
    if mval[0] == 0:        # the imaginary part of a_l0 is ignored
        x = a.copy()
        x[0, 5] = complex(x[0, 5].real, value)
        assert np.array_equal(plan.alm2map(torch.from_numpy(x).to("cuda:0")).cpu().numpy(), m0)


def test_batch(P):
    _say("batch")
    plans = [P.Plan(LMAX, _geo()), P.Plan(64, W.healpix_geometry(32)), P.Plan(LMAX, _geo())]
    batch = P.Batch(plans)
    a = [W.random_alm(p.lmax, [852, i]) for i, p in enumerate(plans)]
    dev = [torch.from_numpy(x).to("cuda:0") for x in a]
    clean = [o.cpu().numpy().copy() for o in batch.alm2map(dev, batch.new_maps())]
    a[2][-1] = np.nan
    dev[2] = torch.from_numpy(a[2]).to("cuda:0")
    got = [o.cpu().numpy() for o in batch.alm2map(dev, batch.new_maps())]
    assert np.array_equal(got[0], clean[0]) and np.array_equal(got[1], clean[1])
    assert np.all(_bad(got[2]))


@pytest.mark.parametrize("prec", ["fp64", "f16x2_mfma"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("mset", list(MSETS))
def test_pixel(P, mset, value, prec):
    _say("pixel", mset, value, prec)
    mval = MSETS[mset] if MSETS[mset] is not None else np.arange(LMAX + 1, dtype=np.int32)
    g, nmaps = _geo(), 3
    plan = P.Plan(LMAX, g, mval=mval, nmaps=nmaps, precision=prec)
    s = np.random.default_rng(853).standard_normal((nmaps, g.npix))
    a0 = plan.alm2map_adjoint(torch.from_numpy(s).to("cuda:0")).cpu().numpy()
    dt0 = plan.map2delta_adjoint(torch.from_numpy(s).to("cuda:0")).cpu().numpy()
    c0 = plan.delta2alm_adjoint(torch.from_numpy(dt0).to("cuda:0")).cpu().numpy()
    for k, r in enumerate([0, 12, g.nrings - 1]):
        b = k % nmaps
        rest = np.arange(nmaps) != b
        x = s.copy()
        x[b, int(g.ringstart[r]) + 1] = value
        got = plan.alm2map_adjoint(torch.from_numpy(x).to("cuda:0")).cpu().numpy()
        assert np.all(_bad(got[b].real)), r
        assert np.array_equal(got[rest], a0[rest])
        w = np.ones(g.nrings)
        got = plan.map2alm(torch.from_numpy(x).to("cuda:0"), w).cpu().numpy()
        assert np.all(_bad(got[b].real)) and np.all(np.isfinite(got[rest])), r
        # the stage: one entry of a caller's Delta~
        i = len(mval) - 1 - k
        d = dt0.copy()
        d[b, i, r] = value
        got = plan.delta2alm_adjoint(torch.from_numpy(d).to("cuda:0")).cpu().numpy()
        p = slice(_off(mval, i, int(mval[i])), _off(mval, i, LMAX) + 1)
        assert np.all(_bad(got[b, p].real)), (i, r)
        got[b, p] = c0[b, p]
        assert np.array_equal(got, c0)
