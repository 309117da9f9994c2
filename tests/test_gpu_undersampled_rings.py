"""FP64 plans on rings with far fewer pixels than modes (l_max up to 8191 on
44 to 8188 pixels), whose live modes a Bluestein workgroup's LDS cannot hold
beside its convolutions: both directions, the refined analysis and a batch in
which one such plan sits beside an ordinary one.

The Fourier stage is looked at by itself: the whole transforms against the
oracle's ring sums around the same plan's Legendre stage. Bound of the other
ring tests, 1e-13 log2 n of the largest output: three transforms of log2 n
levels; a phase is at most 64 products of 2^-53 each. phi0 has few bits, so
that m phi0 and the oracle's phases are exact also at m = 16383."""
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


def _geo(ns, cths):
    """One ring of every length in ns at every cos(theta) in cths."""
    x = np.repeat(cths, len(ns))
    n = np.tile(np.array(ns, np.int64), len(cths))
    start = np.concatenate([[0], np.cumsum(n)[:-1]])
    return W.Geometry(x, np.sqrt(1 - x ** 2), (1 + np.arange(len(n)) % 5) / 16.0, n, start,
                      int(n.sum()))


# len = n / 4 with a prime factor above 7: 11, 263, 1021 and 2047; at
# cos(theta) = 0.9999 (sin 0.014) a ring keeps few of its modes and stays on
# the Bluestein path beside the others
NS = [44, 1052, 4084, 8188]
CTHS = [0.05, -0.05, 0.9999]
# kFastMaxModes is 4352
CASES = [("few m", 8191, np.r_[0:6, 100, 4351, 4352, 5000, 8190, 8191]),
         ("all m", 4800, np.arange(4801)),
         ("largest", 16383, np.r_[0, 1, 7, 9000, 16383])]


@pytest.mark.parametrize("name,lmax,mval", CASES, ids=[c[0] for c in CASES])
def test_both_directions(P, name, lmax, mval):
    print("[case] undersampled", name, flush=True)
    sys.stdout.flush()
    mval = mval.astype(np.int32)
    geo = _geo(NS, CTHS)
    plan = P.Plan(lmax, geo, mval=mval)
    a = W.random_alm(lmax, [821, lmax], mval=mval)
    tol = 1e-13 * np.log2(max(NS) + 1)

    def close(x, e):
        assert np.max(np.abs(x - e)) < tol * np.max(np.abs(e))

    alm = torch.from_numpy(a).to("cuda:0").reshape(1, -1)
    d = plan.alm2delta(alm)
    exp = ref.map_from_delta(mval, geo, d.cpu().numpy()[0].T)
    close(plan.alm2map(alm).cpu().numpy()[0], exp)
    close(plan.delta2map(d).cpu().numpy()[0], exp)

    g = np.random.default_rng(lmax).standard_normal(geo.npix)
    g_dev = torch.from_numpy(g).to("cuda:0").reshape(1, -1)
    dt = np.stack([ref.ring_analysis(g[s:s + n], mval, p) for s, n, p in
                   zip(geo.ringstart, geo.nphi, geo.phi0)], axis=1)
    close(plan.map2delta_adjoint(g_dev).cpu().numpy()[0], dt)
    exp = plan.delta2alm_adjoint(torch.from_numpy(dt[None].copy()).to("cuda:0"))
    close(plan.alm2map_adjoint(g_dev).cpu().numpy(), exp.cpu().numpy())
    w = 1.0 + np.arange(geo.nrings) / 7.0
    dt = dt * w / np.where(mval == 0, 1.0, 2.0)[:, None]
    exp = plan.delta2alm_adjoint(torch.from_numpy(dt[None].copy()).to("cuda:0"))
    close(plan.map2alm(g_dev, w).cpu().numpy(), exp.cpu().numpy())


def test_batch_beside_an_ordinary_plan(P):
    print("[case] undersampled batch", flush=True)
    name, lmax, mval = CASES[0]
    mval = mval.astype(np.int32)
    geo, small = _geo(NS, CTHS), W.healpix_geometry(74)
    plans = [P.Plan(lmax, geo, mval=mval), P.Plan(148, small), P.Plan(300, _geo(NS, CTHS))]
    batch = P.Batch(plans)
    alms = [W.random_alm(lmax, [822, 0], mval=mval), W.random_alm(148, [822, 1]),
            W.random_alm(300, [822, 2])]
    dev = [torch.from_numpy(a).to("cuda:0") for a in alms]
    outs = batch.alm2map(dev, batch.new_maps())
    for p, a, o in zip(plans, dev, outs):
        assert torch.equal(o.reshape(-1), p.alm2map(a.reshape(1, -1)).reshape(-1))
