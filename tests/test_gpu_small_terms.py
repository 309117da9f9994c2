"""Terms far below an m's largest: Delta, coefficients and maps that consist of
nothing else keep their relative accuracy down to 2^-950.

Expected values in 80-bit arithmetic (15 exponent bits: no scaling, errors of
2^-64).  The rings lie at sin(theta) where every P_lm with l <= l_max still grows
and is positive, so errors are relative: sin^m has up to m roundings, a step of
the recurrence at most 3 on either addend, a sum one per term, and the same on
the weights: below 8 (l_max + m) 2^-53."""
import sys

import numpy as np
import pytest

import workloads as W
from oracle import ref

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
LD = np.longdouble


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1010_1260_amd as P
    return P


def _say(*a):
    print("[case] small terms", *a, flush=True)
    sys.stdout.flush()


LMAX = 190
SIN = np.array([0.02, 0.03, 0.1, 0.2])   # 190 sin(theta) stays below the m used
MS = [40, 90, 150, 161]


def _geo():
    s = SIN.copy()
    c = np.sqrt(1 - s * s)
    s = np.sqrt(1 - c * c)
    n = np.full(len(s), 64, np.int64)
    return W.Geometry(c, s, np.array([0.25, 0.5, 0.0, 1.0]), n, np.arange(len(s)) * 64, 64 * len(s))


def _plm(m, c, s):
    """P_lm, l = m..LMAX, of every ring, in 80 bits: [l][ring]."""
    c, s = c.astype(LD), s.astype(LD)
    mu = np.sqrt(1 / (4 * LD(np.pi)))
    for k in range(1, m + 1):
        mu *= np.sqrt(1 + 1 / LD(2 * k))
    p = [mu * s ** m]
    if m < LMAX:
        p.append(np.sqrt(LD(2 * m + 3)) * c * p[0])
    beta = lambda l: np.sqrt((4 * LD(l) * l - 1) / (LD(l) * l - LD(m) * m))
    for l in range(m + 2, LMAX + 1):
        p.append(beta(l) * (c * p[-1] - p[-2] / beta(l - 1)))
    return np.array(p)


# 80-bit pi of the constant above: numpy's is a double
_PI = LD(3) + LD("0.14159265358979323846264338327950288")


def _tol(m):
    return 8 * (LMAX + m) * 2.0 ** -53


def _weights(kind, m):
    n = LMAX + 1 - m
    if kind == "l = m":
        w = np.zeros(n)
        w[0] = 1.25
    else:                       # a wide beam: 2^-20 per step
        w = 1.5 * 2.0 ** (-20.0 * np.arange(n))
    return w


def _off(m):
    return sum(LMAX + 1 - k for k in range(m))


@pytest.mark.parametrize("kind", ["l = m", "steep"])
@pytest.mark.parametrize("nmaps", [1, 4])
def test_synthesis(P, kind, nmaps):
    _say("synthesis", kind, nmaps)
    g = _geo()
    plan = P.Plan(LMAX, g, nmaps=nmaps)
    one = np.sqrt(LD(np.pi) / _PI)
    for m in MS:
        a = np.zeros(plan.nalm, np.complex128)
        w = _weights(kind, m)
        a[_off(m):_off(m) + len(w)] = w * (1 - 0.5j)
        alm = torch.from_numpy(np.stack([a * (b + 1) for b in range(nmaps)])).to("cuda:0")
        e = (w.astype(LD)[:, None] * _plm(m, g.cth, g.sth) * one).sum(axis=0)
        seen = np.abs(e) > 2.0 ** -950
        assert seen.sum() >= 3
        d = plan.alm2delta(alm).cpu().numpy()
        mp = plan.alm2map(alm).cpu().numpy()
        for b in range(nmaps):
            x = d[b, m] / (b + 1)
            assert np.all(np.abs(x.real - e)[seen] <= _tol(m) * e[seen]), m
            assert np.all(np.abs(x.imag + e / 2)[seen] <= _tol(m) * e[seen]), m
            for r in np.nonzero(seen)[0]:
                if e[r] < 2.0 ** -900:      # products of the ring transform
                    continue
                s = ref.ring_synthesis(np.array([complex(float(e[r])) * (1 - 0.5j) * 2.0 ** 800]),
                                       np.array([m]), g.phi0[r], 64)
                y = mp[b, r * 64:(r + 1) * 64] / (b + 1) * 2.0 ** 800
                # and log2 n levels of the transform
                assert np.max(np.abs(y - s)) <= 2 * (_tol(m) + 1e-14) * np.max(np.abs(s)), (m, r)


@pytest.mark.parametrize("prec", ["fp64", "f16x2_mfma"])
def test_adjoint(P, prec):
    _say("adjoint", prec)
    g = _geo()
    plan = P.Plan(LMAX, g, precision=prec)
    one = np.sqrt(LD(np.pi) / _PI)
    dt = np.zeros((1, LMAX + 1, g.nrings), np.complex128)
    for r in range(g.nrings):
        dt[:] = 0
        dt[:, MS, r] = 1.5 - 0.75j
        got = plan.delta2alm_adjoint(torch.from_numpy(dt).to("cuda:0")).cpu().numpy()[0]
        for m in MS:
            e = _plm(m, g.cth[r:r + 1], g.sth[r:r + 1])[:, 0] * one
            x = got[_off(m):_off(m) + len(e)]
            seen = e > 2.0 ** -950
            assert np.all(np.abs(x.real - 1.5 * e)[seen] <= _tol(m) * 1.5 * e[seen]), (m, r)
            assert np.all(np.abs(x.imag + 0.75 * e)[seen] <= _tol(m) * 1.5 * e[seen]), (m, r)
