"""Crossing times of the shrinking lightcone sphere (paper Sec. 3) over drifts in which its radius
falls by a few parts in a hundred up to a factor of 60, tens of thousands of crossings each, some
within 1e-8 of either end: every record against a bisection in 80-bit floats on the series the
call was given.

Bound, before the first run: the computed F = |d0 + p D|^2 - chi^2 carries the rounding of the
squares and sums (at most 6 units of 2^-52 r^2, r the offset's length) and of the two series
(Clenshaw in FP64: at most 4 units of 2^-52 of the coefficients' sum in chi, twice chi of it in F),
so its zero lies within that over dF/dt of the true one; t and a = a0 + (t + 1)(a1 - a0) / 2 are
rounded to 2^-52 each; the offset d moves by |p| dD/dt of the error in t.
"""
import math

import numpy as np
import pytest

import dzs_ics

pytestmark = pytest.mark.gpu

N = 60000
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def dz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_05328_amd as dz
    return dz


def _cheb(c, t):
    b1 = np.zeros_like(t)
    b2 = np.zeros_like(t)
    for v in c[:0:-1]:
        b1, b2 = 2 * t * b1 - b2 + v, b1
    return t * b1 - b2 + c[0]


@pytest.mark.parametrize("vel", [300.0, 3000.0])
@pytest.mark.parametrize("a0,a1", [(0.50, 0.52), (0.90, 0.91), (0.95, 0.9505), (0.95, 0.99),
                                   (0.99, 0.9995), (0.997, 0.99995)])
def test_crossing_times_to_the_rounding_of_f(dz, a0, a1, vel):
    lc = dz.step_factors(a0, a1, 0.3).lc
    chi0, chi1 = math.sqrt(lc.chi2_0), math.sqrt(lc.chi2_1)
    L = 3.0 * chi0
    g = dzs_ics.rng(17)
    u = g.standard_normal((3, N))
    u /= np.sqrt((u ** 2).sum(0))
    near = 10.0 ** (-8 * g.random(N))
    w = np.choose(np.arange(N) % 4, [near, 1 - near, g.random(N), g.random(N)])
    ps = dzs_ics.uniform_random(N, L, seed=5)
    ps.x, ps.y, ps.z = 0.5 * L + (chi1 + (chi0 - chi1) * w) * u
    ps.px, ps.py, ps.pz = g.standard_normal((3, N)) * vel
    ps.id = np.arange(N, dtype=np.uint32)
    for d in range(3):
        lc.x_obs[d] = 0.5 * L
    ctx = dz.Context(N, 0)
    ring = dz.LCRing(N)
    ring.reset()
    ctx.lightcone_emit(dz.make_box(L, 1.0, 1.0), dz.State.from_host(ps), lc, ring)
    rec = ring.records()
    ctx.close()
    assert rec["overflow"] == 0 and rec["count"] > 0.7 * N

    i = rec["id"].astype(np.int64)
    # (offsets as the call forms them, then 80 bits)
    d0 = np.stack([v[i] - 0.5 * L for v in (ps.x, ps.y, ps.z)]).astype(np.longdouble)
    p = np.stack([v[i] for v in (ps.px, ps.py, ps.pz)]).astype(np.longdouble)
    cc = np.array(lc.cheb_chi[:lc.n_cheb], np.longdouble)
    cd = np.array(lc.cheb_drift[:lc.n_cheb], np.longdouble)

    def F(t):
        return ((d0 + p * _cheb(cd, t)) ** 2).sum(0) - _cheb(cc, t) ** 2

    one = np.ones(len(i), np.longdouble)
    ok = (F(-one) < 0) & (F(one) > 0)   # (the last sign may differ from the FP64 test's)
    assert ok.mean() > 0.999
    lo, hi = -one, one.copy()
    for _ in range(66):
        mid = 0.5 * (lo + hi)
        neg = F(mid) < 0
        lo, hi = np.where(neg, mid, lo), np.where(neg, hi, mid)
    t = 0.5 * (lo + hi)
    chi, D = _cheb(cc, t), _cheb(cd, t)
    h = np.longdouble(1e-6)
    slope = (F(t + h) - F(t - h)) / (2 * h)
    dD = np.abs((_cheb(cd, t + h) - _cheb(cd, t - h)) / (2 * h))
    r = np.sqrt(((d0 + p * D) ** 2).sum(0))
    pn = np.sqrt((p ** 2).sum(0))
    # several crossings, or a sphere that does not outrun the particle: any of them may be found
    ok &= slope > 0.05 * chi * (chi0 - chi1)
    assert ok.mean() > 0.9
    dt = EPS * (1 + (6 * r ** 2 + 8 * chi * (np.abs(cc).sum() + pn * np.abs(cd).sum())) / slope)
    a = a0 + 0.5 * (t + 1) * (np.longdouble(a1) - a0)
    da = np.abs(rec["a_cross"] - a) / (0.5 * (a1 - a0) * dt + EPS)
    dd = np.abs(rec["d"].T - (d0 + p * D)) / (np.abs(p) * dD * dt + 2 * EPS * (np.abs(d0) + np.abs(p * D)) +
                                             4 * EPS * np.abs(p) * np.abs(cd).sum())
    print(f"a {a0} -> {a1}, radius {chi0:.4g} -> {chi1:.4g}, vel {vel:g}: {len(i)} records, over "
          f"their bounds a {float(da[ok].max()):.3g}, d {float(dd[:, ok].max()):.3g}", flush=True)
    assert da[ok].max() <= 1
    assert dd[:, ok].max() <= 1
