"""Timed cases of the transform: what programs call it for, over the sizes they use.

Every case goes through the public Python entry points (``Plan``, ``Batch``,
``alm2map``) with its inputs and its plan in hand, as in a program that
transforms many maps on one geometry.  Kinds:

* ``synth``    alm2map of ``nmaps`` maps (FP64 or one of the mixed forms);
* ``adjoint``  alm2map_adjoint of ``nmaps`` maps (a gradient);
* ``grad``     differentiable alm2map, the loss 0.5 |map - d|^2 and its
               backward pass: the map and the coefficient gradient;
* ``map2alm``  quadrature-weighted analysis with ``niter`` Jacobi steps;
* ``batch``    a batch of FP64 maps of uneven band limits in one call.

Grids: ``healpix`` (any nside, also odd), ``gl`` (Gauss-Legendre, odd or even
ring lengths) and ``ecp`` (equidistant).  ``mmax`` below ``lmax`` leaves the
upper m out.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1010_1260_amd import Batch, Plan, alm2map

BATCH_LMAX = (256, 512, 1024, 2048)


# --------------------------------------------------------------------- cases
def _case(name, kind, grid, lmax, nmaps=1, precision="fp64", mmax=None, niter=0, nside=0,
          nrings=0, nphi=0, pick=0):
    c = dict(kind=kind, grid=grid, lmax=lmax, mmax=lmax if mmax is None else mmax, nmaps=nmaps,
             precision=precision, niter=niter, nside=nside, nrings=nrings, nphi=nphi, pick=pick)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest useful map: a call in a sampler's inner loop, all latency
        _case("synth_l64_n32", "synth", "healpix", 64, nside=32),
        # an ordinary single map in full precision
        _case("synth_l1024_n512", "synth", "healpix", 1024, nside=512),
        # the full-size single map in full precision
        _case("synth_l4096_n2048", "synth", "healpix", 4096, nside=2048),
        # a few maps on a Gauss-Legendre grid with odd ring lengths and a band
        # of m left out (a simulation at reduced azimuthal resolution)
        _case("synth_gl_l500_x3", "synth", "gl", 500, nmaps=3, mmax=450, nrings=501, nphi=1001),
        # full-size batch of simulations in the fastest mixed form
        _case("f16x2_l4096_n2048_x16", "synth", "healpix", 4096, nmaps=16,
              precision="f16x2_mfma", nside=2048),
        # a medium batch of simulations, split BF16
        _case("bf16x3_l1024_n512_x16", "synth", "healpix", 1024, nmaps=16,
              precision="bf16x3_mfma", nside=512),
        # an odd number of maps at odd sizes on FP32 matrix operands
        _case("fp32_l1999_n999_x5", "synth", "healpix", 1999, nmaps=5, precision="fp32_mfma",
              nside=999),
        # the gradient of one map
        _case("adjoint_l2048_n1024", "adjoint", "healpix", 2048, nside=1024),
        # a step of a gradient-based reconstruction: forward, loss, backward
        _case("grad_l1024_n512_x8", "grad", "healpix", 1024, nmaps=8, nside=512),
        # the full-size analysis of one map
        _case("map2alm_l4096_n2048", "map2alm", "healpix", 4096, nside=2048),
        # a refined analysis of a small map
        _case("map2alm_l512_n256_it3", "map2alm", "healpix", 512, niter=3, nside=256),
        # 64 maps of four band limits drawn at random, one batched call
        _case("batch_uneven_x64", "batch", "healpix", 2048, nmaps=64, pick=4),
    ]


def _cost(c):
    """Rough relative cost of a pass (1 = one full-size FP64 synthesis)."""
    unit = (c["lmax"] / 4096.0) ** 2 * max(c["nside"] / 2048.0, c["nrings"] / 8192.0)
    n = c["nmaps"]
    if c["kind"] == "batch":
        return n * (c["lmax"] / 4096.0) ** 3 * 0.5
    if c["kind"] == "synth":
        # the mixed forms take 16 maps at a time
        return unit * (n if c["precision"] == "fp64" else 3.0 * math.ceil(n / 16))
    if c["kind"] == "adjoint":
        return 2.0 * unit * n
    if c["kind"] == "grad":
        return 3.0 * unit * n
    return unit * n * (2.0 + 3.0 * c["niter"])


def draw(rng):
    while True:
        kind = rng.choice(["synth", "synth", "synth", "mixed", "mixed", "adjoint", "grad",
                           "map2alm", "batch"])
        lmax = int(round(math.exp(rng.uniform(math.log(48), math.log(4096)))))
        if kind == "batch":
            c = _case(None, "batch", "healpix", rng.choice([256, 512, 1024, 2048]),
                      nmaps=rng.randint(2, 64), pick=rng.randint(0, 1 << 20))
        else:
            prec = rng.choice(["f16x2_mfma", "f16x2_mfma", "bf16x3_mfma", "fp32_mfma"]) \
                if kind == "mixed" else "fp64"
            nmaps = rng.choice([1, 1, 2, 3, 4, 5, 8, 13, 16]) if kind != "mixed" else \
                rng.choice([1, 4, 7, 8, 15, 16])
            niter = rng.randint(0, 3) if kind == "map2alm" else 0
            grid = "healpix" if lmax > 1500 or kind == "map2alm" else \
                rng.choice(["healpix", "healpix", "gl", "ecp"])
            mmax = lmax if rng.random() < 0.8 else rng.randint(lmax // 2, lmax)
            kind = "synth" if kind == "mixed" else kind
            if grid == "healpix":
                c = _case(None, kind, grid, lmax, nmaps, prec, mmax, niter,
                          nside=max(16, lmax // 2))
            elif grid == "gl":
                c = _case(None, kind, grid, lmax, nmaps, prec, mmax, niter, nrings=lmax + 1,
                          nphi=2 * lmax + rng.choice([1, 2]))
            else:
                c = _case(None, kind, grid, lmax, nmaps, prec, mmax, niter, nrings=2 * lmax,
                          nphi=2 * lmax + 2 * rng.randint(0, 8))
        if _cost(c) <= 2.0:
            return c


# ------------------------------------------------------------------ geometry
def _healpix(n):
    """HEALPix rings of nside n, north to south (Gorski et al. 2005)."""
    i = np.arange(1, 2 * n + 1, dtype=np.float64)
    cap = i < n
    omz = i * i / (3.0 * n * n)
    zb = 2.0 * (2 * n - i) / (3.0 * n)
    z = np.where(cap, 1.0 - omz, zb)
    s = np.sqrt(np.where(cap, omz * (1.0 + z), (1.0 - zb) * (1.0 + zb)))
    m = np.where(cap, 4 * i, 4 * n).astype(np.int64)
    p0 = np.where(cap, math.pi / (4.0 * i),
                  np.where((i.astype(np.int64) - n) % 2 == 0, math.pi / (4.0 * n), 0.0))
    z[-1], s[-1] = 0.0, 1.0
    cth = np.concatenate([z, -z[-2::-1]])
    nphi = np.concatenate([m, m[-2::-1]])
    start = np.concatenate([[0], np.cumsum(nphi)[:-1]])
    return SimpleNamespace(cth=cth, sth=np.concatenate([s, s[-2::-1]]), nphi=nphi,
                           phi0=np.concatenate([p0, p0[-2::-1]]), ringstart=start,
                           npix=12 * n * n, weight=np.full(len(cth), math.pi / (3.0 * n * n)))


def _rows(x, s, nphi, weight):
    n = len(x)
    return SimpleNamespace(cth=x, sth=s, nphi=np.full(n, nphi, dtype=np.int64),
                           phi0=np.zeros(n), ringstart=np.arange(n, dtype=np.int64) * nphi,
                           npix=n * nphi, weight=weight * (2.0 * math.pi / nphi))


def _geometry(c):
    if c["grid"] == "healpix":
        return _healpix(c["nside"])
    n, nphi = c["nrings"], c["nphi"]
    if c["grid"] == "gl":
        x, w = np.polynomial.legendre.leggauss(n)
        x, w = x[::-1].copy(), w[::-1].copy()
        x = 0.5 * (x - x[::-1])
        return _rows(x, np.sqrt((1.0 - x) * (1.0 + x)), nphi, w)
    th = math.pi * (np.arange(n) + 0.5) / n
    x, s = np.cos(th), np.sin(th)
    h = n // 2
    x[n - h:], s[n - h:] = -x[:h][::-1], s[:h][::-1]
    if n % 2:
        x[h], s[h] = 0.0, 1.0
    return _rows(x, s, nphi, s * (math.pi / n))


# -------------------------------------------------------------------- inputs
def _lm(lmax, mmax, dev):
    """l and m of every packed coefficient (for each m: l = m..lmax)."""
    off = np.concatenate([[0], np.cumsum(lmax + 1 - np.arange(mmax + 1))])
    off = torch.from_numpy(off).to(dev)
    i = torch.arange(int(off[-1]), device=dev)
    m = torch.searchsorted(off, i, right=True) - 1
    return i - off[m] + m, m


def _alm(c, lmax, mmax, nmaps, gen, dev):
    """Gaussian coefficients with the spectrum 1 / (l (l + 1)), l >= 2."""
    l, m = _lm(lmax, mmax, dev)
    ll = l.to(torch.float64)
    sd = torch.where(l >= 2, (0.5 / (ll * (ll + 1.0)).clamp(min=1.0)).sqrt(), torch.zeros_like(ll))
    a = torch.empty((nmaps, l.numel()), dtype=torch.complex128, device=dev)
    for b in range(nmaps):
        z = torch.randn((l.numel(), 2), dtype=torch.float64, device=dev, generator=gen)
        z *= sd[:, None]
        z[m == 0, 0] *= math.sqrt(2.0)
        z[m == 0, 1] = 0.0
        a[b] = torch.view_as_complex(z)
    return a


def _batch_lmax(c):
    rng = np.random.default_rng([4, c["pick"]])
    top = [v for v in BATCH_LMAX if v <= c["lmax"]]
    return [int(top[k]) for k in rng.integers(0, len(top), size=c["nmaps"])]


def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed))


def _inputs(c, seed, dev):
    """The seeded tensors of a case: coefficients, maps, data."""
    gen = _gen(seed, dev)
    if c["kind"] == "batch":
        return dict(alm=[_alm(c, v, v, 1, gen, dev)[0] for v in _batch_lmax(c)])
    npix = _geometry(c).npix
    d = {}
    if c["kind"] in ("synth", "grad"):
        d["alm"] = _alm(c, c["lmax"], c["mmax"], c["nmaps"], gen, dev)
    if c["kind"] in ("adjoint", "grad", "map2alm"):
        d["map"] = torch.randn((c["nmaps"], npix), dtype=torch.float64, device=dev, generator=gen)
    return d


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    st = dict(kind=case["kind"], niter=case["niter"], **_inputs(case, seed, dev))
    if case["kind"] == "batch":
        # maps of one band limit share a plan
        lmaxes = _batch_lmax(case)
        plans = {v: Plan(v, _healpix(v // 2), device=dev) for v in sorted(set(lmaxes))}
        st["batch"] = Batch([plans[v] for v in lmaxes])
        st["out"] = st["batch"].new_maps()
        return st
    geom = _geometry(case)
    st["plan"] = Plan(case["lmax"], geom, mval=np.arange(case["mmax"] + 1, dtype=np.int32),
                      nmaps=case["nmaps"], device=dev, precision=case["precision"])
    if case["kind"] == "map2alm":
        st["weight"] = torch.from_numpy(geom.weight).to(dev)
    return st


# ----------------------------------------------------------------------- run
def run(state):
    kind = state["kind"]
    if kind == "synth":
        return state["plan"].alm2map(state["alm"])
    if kind == "adjoint":
        return state["plan"].alm2map_adjoint(state["map"])
    if kind == "map2alm":
        return state["plan"].map2alm(state["map"], state["weight"], niter=state["niter"])
    if kind == "batch":
        return state["batch"].alm2map(state["alm"], state["out"])
    a = state["alm"].detach().requires_grad_(True)
    m = alm2map(a, state["plan"])
    loss = 0.5 * (m - state["map"]).square().sum()
    (g,) = torch.autograd.grad(loss, a)
    return {"map": m.detach(), "grad": g}


# ---------------------------------------------------------------------- work
def _one(lmax, mmax, npairs, npix, nmaps):
    """(bytes, flops) of one transform: the coefficients and the maps once;
    per (ring pair, l, m) one recurrence step (3 flops) shared by all maps and
    one complex accumulation (4 flops) per map; 2.5 n log2 n per ring's FFT."""
    nalm = (mmax + 1) * (lmax + 1) - mmax * (mmax + 1) // 2
    fl = npairs * nalm * (3.0 + 4.0 * nmaps)
    fl += nmaps * 2.5 * npix * math.log2(max(2, 2 * lmax))
    return nmaps * (16.0 * nalm + 8.0 * npix), fl


def work(case):
    if case["kind"] == "batch":
        b = f = 0.0
        for v in _batch_lmax(case):
            x, y = _one(v, v, v, 3 * v * v, 1)
            b, f = b + x, f + y
        return {"bytes": b, "flops": f}
    if case["grid"] == "healpix":
        npairs, npix = 2 * case["nside"], 12 * case["nside"] ** 2
    else:
        npairs, npix = (case["nrings"] + 1) // 2, case["nrings"] * case["nphi"]
    b, f = _one(case["lmax"], case["mmax"], npairs, npix, case["nmaps"])
    if case["kind"] == "grad":   # forward and backward; the data map once more
        return {"bytes": 2 * b + 8.0 * npix * case["nmaps"], "flops": 2 * f}
    if case["kind"] == "map2alm":
        n = 1 + 2 * case["niter"]
        return {"bytes": n * b, "flops": n * f}
    return {"bytes": b, "flops": f}


# --------------------------------------------------------------------- exact
class _Exact:
    """The transform in plain FP64 tensor operations: the recurrence for all
    (m, ring) of one hemisphere at a time, batched products over blocks of l,
    per-ring FFTs of the full length."""

    LB = 32   # rows of l per block

    def __init__(self, lmax, mmax, geom, dev):
        self.lmax, self.mmax, self.geom, self.dev = lmax, mmax, geom, dev
        n = len(geom.cth)
        self.nrings, self.np = n, (n + 1) // 2
        # every grid here is symmetric about the equator, north to south
        self.north = torch.arange(self.np, device=dev)
        self.south = n - 1 - self.north
        self.x = torch.from_numpy(geom.cth[:self.np].copy()).to(dev)
        self.s = torch.from_numpy(geom.sth[:self.np].copy()).to(dev)
        self.off = np.concatenate([[0], np.cumsum(lmax + 1 - np.arange(mmax + 1))])

    def _legendre(self, m0, m1, use):
        """use(l0, P): P[l - l0, i, pair] = P_lm of m = m0 + i (zero for l < m)."""
        dev, lmax, np_ = self.dev, self.lmax, self.np
        k = torch.arange(1, m1 + 1, dtype=torch.float64, device=dev)
        lmu = torch.zeros(m1 + 1, dtype=torch.float64, device=dev)
        lmu[1:] = torch.cumsum(0.5 * torch.log2((2 * k + 1) / (2 * k)), 0)
        lmu += 0.5 * math.log2(1.0 / (4.0 * math.pi))
        m = torch.arange(m0, m1, dtype=torch.float64, device=dev)[:, None]
        # sin^m as mantissa and exponent by repeated squaring of (mantissa, exponent)
        man, ex = torch.frexp(self.s)
        r = torch.ones((m1 - m0, np_), dtype=torch.float64, device=dev)
        re = torch.zeros((m1 - m0, np_), dtype=torch.float64, device=dev)
        b, be = man.clone(), ex.to(torch.float64)
        mi = torch.arange(m0, m1, device=dev)
        for bit in range(15):
            on = ((mi >> bit) & 1).bool()[:, None]
            r = torch.where(on, r * b, r)
            re = torch.where(on, re + be, re)
            r, e = torch.frexp(r)
            re += e
            b, e = torch.frexp(b * b)
            be = 2 * be + e
        fl = torch.floor(lmu[m0:m1])[:, None]
        seed = r * torch.exp2(lmu[m0:m1, None] - fl)
        se = re + fl
        u0 = torch.zeros((m1 - m0, np_), dtype=torch.float64, device=dev)
        u1 = torch.zeros_like(u0)      # u1 2^e = P_{l-1}, u0 2^e = P_{l-2}
        e = torch.zeros_like(u0)
        x = self.x[None, :]
        bp = torch.ones_like(m)
        for l0 in range(m0, lmax + 1, self.LB):
            l1 = min(l0 + self.LB, lmax + 1)
            P = torch.zeros((l1 - l0, m1 - m0, np_), dtype=torch.float64, device=dev)
            for l in range(l0, l1):
                bl = torch.sqrt((4.0 * l * l - 1.0) / (l * l - m * m).clamp(min=1.0))
                u = bl * (x * u1 - u0 / bp)
                if l < m1 and l >= m0:     # this row's seed
                    i = l - m0
                    u[i:] = 0.0
                    u[i] = seed[i]
                    e[i] = se[i]
                    bl[i:] = 1.0
                u0, u1, bp = u1, u, bl
                P[l - l0] = u * torch.exp2(e.clamp(min=-1000.0))
            big = torch.maximum(u0.abs(), u1.abs())
            sh = torch.frexp(big)[1].to(torch.float64)
            sh = torch.where((big > 0) & (e < 0), torch.minimum(sh, -e), torch.zeros_like(sh))
            f = torch.exp2(-sh)
            u0, u1, e = u0 * f, u1 * f, e + sh
            use(l0, P)

    def _chunks(self, nmaps):
        step = max(1, int(2e9 / (8 * self.np * (self.LB + 4 * nmaps + 12))))
        return [(m, min(m + step, self.mmax + 1)) for m in range(0, self.mmax + 1, step)]

    def synth(self, alm):
        nb, dev = alm.shape[0], self.dev
        delta = torch.zeros((nb, self.mmax + 1, self.nrings), dtype=torch.complex128, device=dev)
        for m0, m1 in self._chunks(nb):
            nm = m1 - m0
            sums = [torch.zeros((nm, 2 * nb, self.np), dtype=torch.float64, device=dev)
                    for _ in range(2)]   # l even, l odd
            # dense [l][m][map, re/im] of this chunk
            A = torch.zeros((self.lmax + 1, nm, 2 * nb), dtype=torch.float64, device=dev)
            for m in range(m0, m1):
                v = torch.view_as_real(alm[:, self.off[m]:self.off[m + 1]].contiguous())
                A[m:, m - m0] = v.permute(1, 0, 2).reshape(-1, 2 * nb)
            if m0 == 0:
                A[:, 0, 1::2] = 0.0

            def use(l0, P):
                a = A[l0:l0 + P.shape[0]]
                for p in (0, 1):
                    rows = slice((p - l0) % 2, None, 2)
                    if P[rows].shape[0]:
                        sums[p] += torch.bmm(a[rows].permute(1, 2, 0).contiguous(),
                                             P[rows].permute(1, 0, 2).contiguous())

            self._legendre(m0, m1, use)
            for i in range(nm):
                m = m0 + i
                e, o = (torch.complex(q[i, 0::2], q[i, 1::2])
                        for q in (sums[m % 2], sums[1 - m % 2]))
                delta[:, m, self.south] = e - o
                delta[:, m, self.north] = e + o
        return self._rings(delta)

    def _lengths(self):
        g = {}
        for r, n in enumerate(self.geom.nphi):
            g.setdefault(int(n), []).append(r)
        return g

    def _phase(self, rings, sign):
        p0 = torch.from_numpy(self.geom.phi0[rings]).to(self.dev)
        m = torch.arange(self.mmax + 1, dtype=torch.float64, device=self.dev)
        t = m[:, None] * p0[None, :]
        return torch.complex(torch.cos(t), sign * torch.sin(t))

    def _fft(self, f, inverse):
        """Along the last axis; ring lengths that come once or twice on the host."""
        where = f.device if f.shape[-2] > 2 else torch.device("cpu")
        g = f.to(where)
        return (torch.fft.ifft(g) * g.shape[-1] if inverse else torch.fft.fft(g)).to(self.dev)

    def _rings(self, delta):
        nb = delta.shape[0]
        out = torch.zeros((nb, self.geom.npix), dtype=torch.float64, device=self.dev)
        for n, rings in self._lengths().items():
            d = delta[:, :, rings] * self._phase(rings, 1.0)
            d = d.transpose(1, 2).contiguous()
            pad = -d.shape[-1] % n
            f = torch.nn.functional.pad(torch.view_as_real(d), (0, 0, 0, pad))
            f = torch.view_as_complex(f.reshape(nb, len(rings), -1, n, 2).sum(2).contiguous())
            s = 2.0 * self._fft(f, True).real - d[:, :, :1].real
            at = torch.from_numpy(self.geom.ringstart[rings]).to(self.dev)[:, None] + \
                torch.arange(n, device=self.dev)
            out[:, at.reshape(-1)] = s.reshape(nb, -1)
        return out

    def analyse(self, maps, weight=None, cm=2.0):
        """sum over pixels of (weight) map e^{-i m phi} P_lm, times cm for m > 0."""
        nb, dev = maps.shape[0], self.dev
        dt = torch.zeros((nb, self.mmax + 1, self.nrings), dtype=torch.complex128, device=dev)
        for n, rings in self._lengths().items():
            at = torch.from_numpy(self.geom.ringstart[rings]).to(dev)[:, None] + \
                torch.arange(n, device=dev)
            f = maps[:, at.reshape(-1)].reshape(nb, len(rings), n).to(torch.complex128)
            g = self._fft(f, False)
            g = g[:, :, torch.arange(self.mmax + 1, device=dev) % n].transpose(1, 2)
            dt[:, :, rings] = g * self._phase(rings, -1.0)
        dt[:, 1:] *= cm
        dt[:, 0].imag.zero_()
        if weight is not None:
            dt *= weight
        out = torch.zeros((nb, int(self.off[-1])), dtype=torch.complex128, device=dev)
        for m0, m1 in self._chunks(nb):
            n = dt[:, m0:m1][:, :, self.north]
            s = dt[:, m0:m1][:, :, self.south]
            s = torch.where(self.north == self.south, torch.zeros_like(s), s)
            odd = (torch.arange(m0, m1, device=dev) % 2 == 1)[None, :, None]
            we, wo = torch.where(odd, n - s, n + s), torch.where(odd, n + s, n - s)
            w = [torch.view_as_real(v.permute(1, 2, 0).contiguous()).reshape(m1 - m0, self.np, -1)
                 for v in (we, wo)]     # l even, l odd
            A = torch.zeros((self.lmax + 1, m1 - m0, 2 * nb), dtype=torch.float64, device=dev)

            def use(l0, P):
                for p in (0, 1):
                    rows = slice((p - l0) % 2, None, 2)
                    if P[rows].shape[0]:
                        r = torch.bmm(P[rows].permute(1, 0, 2).contiguous(), w[p])
                        A[l0:l0 + P.shape[0]][rows] = r.permute(1, 0, 2)

            self._legendre(m0, m1, use)
            for m in range(m0, m1):
                v = A[m:, m - m0].reshape(-1, nb, 2).permute(1, 0, 2).contiguous()
                out[:, self.off[m]:self.off[m + 1]] = torch.view_as_complex(v)
        return out


def exact(case, seed):
    # a dozen full-size maps take longer than a check is worth
    if case["kind"] != "batch" and case["nmaps"] * case["lmax"] ** 2 > 2.5 * 4096 ** 2:
        return None
    dev = torch.device("cuda", torch.cuda.current_device())
    d = _inputs(case, seed, dev)
    if case["kind"] == "batch":
        # the first two maps of each band limit
        lmaxes = _batch_lmax(case)
        out = [None] * len(lmaxes)
        for v in sorted(set(lmaxes)):
            at = [i for i, x in enumerate(lmaxes) if x == v][:2]
            s = _Exact(v, v, _healpix(v // 2), dev).synth(torch.stack([d["alm"][i] for i in at]))
            for i, m in zip(at, s):
                out[i] = m
        return out
    geom = _geometry(case)
    e = _Exact(case["lmax"], case["mmax"], geom, dev)
    if case["kind"] == "synth":
        return e.synth(d["alm"])
    if case["kind"] == "adjoint":
        return e.analyse(d["map"])
    if case["kind"] == "map2alm":
        w = torch.from_numpy(geom.weight).to(dev)
        a = e.analyse(d["map"], w, 1.0)
        for _ in range(case["niter"]):
            a = a + e.analyse(d["map"] - e.synth(a), w, 1.0)
        return a
    m = e.synth(d["alm"])
    return {"map": m, "grad": e.analyse(m - d["map"])}
