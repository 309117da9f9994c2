"""Phases of the mixed forms' two-map ring kernel: those of the FP64 plans'
one-map kernel, rounding for rounding.

A ring of n = 4 m pixels with the mode m alone and real Delta_m = D has
F_m = e^{i m phi0} D; at k = m = n / 4 the half-length construction takes F to
Z = 2 conj(F), without a rounding when m is a multiple of 64 (the table's
products have a factor 1 and every other entry is 0), and the pixels are
alternately +-2 Re F and +-2 Im F.  With m phi0 an odd multiple of pi / 2 the
even ones show Re e^{i m phi0}, which is nothing but the rounding errors of
the phase (around 1e-16), to FP32's relative precision."""
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


@pytest.mark.parametrize("prec", ["f16x2_mfma", "fp32_mfma"])
@pytest.mark.parametrize("nmaps", [1, 2, 3])
@pytest.mark.parametrize("m", [64, 640, 768, 1280, 1920])
def test_phases_are_those_of_the_one_map_fold(P, prec, nmaps, m):
    print("[case] fold phases", prec, nmaps, m, flush=True)
    sys.stdout.flush()
    odd = np.array([1, 3, 5, 7, 9, 11, 13, 15])
    nr, n, lmax = len(odd), 4 * m, m + 3
    cth = np.linspace(0.05, 0.01, nr)
    geo = W.Geometry(cth, np.sqrt(1 - cth ** 2), odd * (np.pi / 2) / m,
                     np.full(nr, n, np.int64), np.arange(nr) * n, nr * n)
    plan = P.Plan(lmax, geo, nmaps=nmaps, precision=prec)
    ref = P.Plan(lmax, geo, nmaps=nmaps)
    a = np.zeros((nmaps, plan.nalm), np.complex128)
    off = sum(lmax + 1 - k for k in range(m))
    a[:, off:off + lmax + 1 - m] = np.random.default_rng(m).standard_normal((nmaps, lmax + 1 - m))
    a = torch.from_numpy(a).to("cuda:0")
    got = plan.alm2map(a).cpu().numpy().reshape(nmaps, nr, n)
    exp = ref.delta2map(plan.alm2delta(a)).cpu().numpy().reshape(nmaps, nr, n)
    assert np.abs(exp[:, :, 0::2]).max() < 1e-12 * np.abs(exp).max()
    # to FP32: F, the table's entry and the sum that gives Z
    assert np.all(np.abs(got - exp) <= 3 * 2.0 ** -24 * np.abs(exp))
