"""Start table of the recurrence: the terms it leaves out are below the
rounding of every m's own sum, also where a plan sees an m only deep in its
growing range (rings near a pole), and the ring stage that skips the dead
modes agrees with the one that reads a whole Delta."""
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


def _say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


# rings from the pole only (every m small there), around the poles and the
# equator, one ring, the pole itself (sin = 0), and whole grids; row counts
# around multiples of 8, ring-pair counts around 64 and 128, gaps in the m-set
CASES = [
    ("cap", 512, np.arange(0, 24), 256, None),
    ("cap pairs", 1000, np.r_[0:40, 1983:2023], 506, None),
    ("mixed", 301, np.r_[0:10, 120:330], 128, np.r_[0, 1, 7, 8, 9, 150:290:3, 301]),
    ("one", 257, np.array([3]), 64, None),
    ("whole", 135, None, 65, None),
    ("whole few m", 519, None, 33, np.array([2, 500, 518])),
]


def _geom(rings, nside):
    g = W.healpix_geometry(nside)
    return g if rings is None else g.subset(rings)


@pytest.mark.parametrize("lmax,rings,nside", [(512, np.arange(0, 24), 256),
                                              (1000, np.r_[0:40, 1983:2023], 506)])
def test_m_that_only_grow_keep_their_relative_accuracy(P, lmax, rings, nside):
    """Rings around the poles only: the m above 2 l_max sin(theta_max) never
    leave their growing range there, where all errors are relative (seed
    sin^m: m roundings, then at most 3 per step; both sides), although their
    Delta lies down to 2^-250 below the other m's."""
    _say("growing m", lmax, nside)
    g = _geom(rings, nside)
    a = W.random_alm(lmax, [803, lmax], spectrum="flat")
    plan = P.Plan(lmax, g)
    d = plan.alm2delta(torch.from_numpy(a).to(_dev()).reshape(1, -1)).cpu().numpy()[0]   # [m][ring]
    # |a_lm| P_lm in place of a_lm P_lm: the scale of each m's rounding errors
    e = ref.delta(lmax, None, g.cth, g.sth, a).T
    t = ref.delta(lmax, None, np.abs(g.cth), g.sth, np.abs(a) + 0j).T
    m0 = int(2 * lmax * g.sth.max()) + 1
    ms = np.arange(m0, lmax + 1)
    top = np.abs(t).max(axis=1)[m0:]
    err = np.abs(d - e).max(axis=1)[m0:]
    seen = top > 2.0 ** -250
    assert seen.sum() > 20
    assert np.all(err[seen] <= (8 * (lmax + ms[seen]) * 2.0 ** -53) * top[seen])


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("f16x2_mfma", 1e-6)])
@pytest.mark.parametrize("name,lmax,rings,nside,mval", CASES, ids=[c[0] for c in CASES])
def test_whole_and_stagewise_agree(P, prec, tol, name, lmax, rings, nside, mval):
    """alm2map (dead modes left out) against delta2map of the whole Delta,
    on buffers that hold NaN beforehand."""
    _say("whole vs stagewise", prec, name)
    g = _geom(rings, nside)
    a = torch.from_numpy(np.stack([W.random_alm(lmax, [802, i], mval=mval) for i in range(3)]))
    plan = P.Plan(lmax, g, mval=mval, nmaps=3, precision=prec)
    plan.workspace().view(torch.float64)[: plan.workspace_bytes // 8].fill_(float("nan"))
    out = torch.zeros((3, plan.npix), dtype=torch.float64, device=_dev())
    m1 = plan.alm2map(a.to(_dev()), out=out).cpu().numpy()
    d = plan.alm2delta(a.to(_dev()))
    m2 = plan.delta2map(d).cpu().numpy()
    assert np.all(np.isfinite(m1))
    assert np.linalg.norm(m1 - m2) <= tol * np.linalg.norm(m2)


# waves per CU (256 CUs) of 16 ring blocks x 151 m-pairs per map: 7 maps go in
# pairs and one alone, 11 in 4 + 4 + 3, 13 in 4 + 4 + 4 + 1, 5 one by one
@pytest.mark.parametrize("nmaps", [5, 7, 11, 13])
def test_maps_together_equal_maps_alone(P, nmaps):
    """A wave that takes several maps does each map's arithmetic unchanged."""
    _say("maps per wave", nmaps)
    lmax = 301
    g = W.ecp_geometry(1999, 8)
    alms = np.stack([W.random_alm(lmax, [804, i]) for i in range(nmaps)])
    a = torch.from_numpy(alms).to(_dev())
    many = P.Plan(lmax, g, nmaps=nmaps)
    one = P.Plan(lmax, g)
    got, d = many.alm2map(a).cpu(), many.alm2delta(a).cpu()
    for i in range(nmaps):
        assert torch.equal(got[i], one.alm2map(a[i]).cpu()[0]), i
        assert torch.equal(d[i], one.alm2delta(a[i]).cpu()[0]), i
    e = ref.alm2map(lmax, g, alms[-1])
    assert np.linalg.norm(got[-1].numpy() - e) <= 1e-12 * np.linalg.norm(e)


# launches of 1, 2 and 8 ring pairs per lane (waves per CU at one pair per lane
# below 4, up to 48, above), row counts around multiples of the 16-row tile, m
# dead on whole ring blocks, an odd and a single m
@pytest.mark.parametrize("lmax,nside,rings,mval,nmaps", [
    (15, 8, None, None, 1),
    (16, 130, np.r_[0:5, 40:200], np.array([0, 3, 16]), 2),
    (257, 128, None, np.array([5]), 3),
    (399, 256, None, None, 2),
    (303, 512, None, None, 13),
])
def test_adjoint_shapes(P, lmax, nside, rings, mval, nmaps):
    _say("adjoint", lmax, nside, nmaps)
    g = _geom(rings, nside)
    maps = np.random.default_rng(805).standard_normal((nmaps, g.npix))
    plan = P.Plan(lmax, g, mval=mval, nmaps=nmaps)
    plan.workspace().view(torch.float64)[: plan.workspace_bytes // 8].fill_(float("nan"))
    got = plan.alm2map_adjoint(torch.from_numpy(maps).to(_dev())).cpu().numpy()
    for i in (0, nmaps - 1):
        e = ref.alm2map_adjoint(lmax, g, maps[i], mval=mval)
        assert np.linalg.norm(got[i] - e) <= 1e-12 * np.linalg.norm(e), i


# FP32 operands: 1..8 map pairs per wave, a last pair of one map, groups of 16
# and a rest; row counts around the 16-row block
@pytest.mark.parametrize("nmaps", [2, 3, 5, 8, 9, 11, 14, 16, 17, 21])
@pytest.mark.parametrize("lmax,nside", [(31, 40), (144, 72)])
def test_fp32_maps_equal_maps_alone(P, lmax, nside, nmaps):
    """Every product adds one term in the order of l, so a map's result does
    not depend on the maps beside it."""
    _say("fp32 maps", lmax, nside, nmaps)
    g = W.healpix_geometry(nside)
    alms = np.stack([W.random_alm(lmax, [806, i]) for i in range(nmaps)])
    a = torch.from_numpy(alms).to(_dev())
    got = P.Plan(lmax, g, nmaps=nmaps, precision="fp32_mfma").alm2delta(a).cpu()
    one = P.Plan(lmax, g, precision="fp32_mfma")
    for i in range(nmaps):
        assert torch.equal(got[i], one.alm2delta(a[i]).cpu()[0]), i
    e = ref.delta(lmax, None, g.cth, g.sth, alms[-1]).T
    assert np.linalg.norm(got[-1].numpy() - e) <= 1e-6 * np.linalg.norm(e)
