"""DZS coarsening of sets with large cubes (paper Sec. 2.2, eqs. 1 and 3): bit for bit against the
oracle, as everywhere.

A cube that holds two consecutive 512th particles is large and has a kernel of its own, the others
start at the first level at which they are not.  So: cubes of 512 to 1025 members at every place
relative to the 512th particles, at one point (large down to the last level) or spread (large for
some levels), merging at the first level, at deeper ones or not at all, in both criteria.  And a
dense clump that does not merge, or only at deep levels, takes no more than three times as long as
the same particles spread out: its cubes are fewer, and no workgroup visits all of its particles
at every level.
"""
import numpy as np
import pytest

import dzs_ics
import oracle

pytestmark = pytest.mark.gpu

L = 100.0


@pytest.fixture(scope="module")
def dz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_05328_amd as dz
    return dz


def _set(before, members, size, after, seed):
    """`before` particles that come first in key order, a clump, `after` that come behind, uniform
    ones in no order in between"""
    n = before + members + after
    ps = dzs_ics.uniform_random(n, L, seed=seed)
    r = dzs_ics.rng(seed + 1)
    order = r.permutation(n)
    b, m, a = order[:before], order[before:before + members], order[before + members:]
    for k in ("x", "y", "z"):
        v = getattr(ps, k)
        v[b] = 50.0 * r.random(before)
        v[m] = 71.0 + size * r.random(members)
        v[a] = 75.0 + 25.0 * r.random(after)
    for k in ("px", "py", "pz"):
        getattr(ps, k)[:] = r.standard_normal(n) * 300.0
    ps.mult = r.integers(1, 20, n).astype(np.uint32)
    ps.id = r.permutation(n).astype(np.uint32)
    return ps


@pytest.mark.parametrize("before,members,size,theta,R,dyn", [
    (0, 512, 0.0, 1.0, 5.0, False), (0, 513, 0.0, 1.0, 5.0, False), (3, 1023, 0.0, 0.05, 5.0, False),
    (511, 513, 0.0, 1.0, 5.0, False), (511, 514, 0.0, 0.05, 5.0, False),
    (512, 1024, 0.4, 0.05, 5.0, False), (700, 1025, 0.4, 0.01, 5.0, False),
    (255, 2600, 0.0, 1e-4, 0.0, False), (256, 2600, 0.02, 1e-3, 0.0, False),
    (700, 20000, 1.0, 0.02, 5.0, False), (700, 20000, 1.0, 0.5, 90.0, False),
    (40, 9000, 0.05, 0.004, 0.0, False), (700, 9000, 0.5, 1.0, 20.0, True),
    (700, 9000, 0.01, 1.0, 20.0, True)])
def test_large_cubes(dz, before, members, size, theta, R, dyn):
    import torch
    ps = _set(before, members, size, 900, seed=before + members)
    n = ps.n
    prm = dict(x_obs=[20.0, 30.0, 40.0], R_lc=R, b=0.5, theta=theta, k_min=3)
    cp = dz.CoarsenParams()
    for d in range(3):
        cp.x_obs[d] = prm["x_obs"][d]
    cp.R_lc, cp.b, cp.theta, cp.k_min = R, 0.5, theta, 3
    g = None
    box = dz.make_box(L, 1.0, L / 1000)
    if dyn:
        g = 50.0 + dzs_ics.rng(9).random((3, n))
        cp.criterion, cp.alpha_dyn = dz.DZS_CRIT_DYNAMICAL, 1e-4
        res, group_of, nm = oracle.coarsen(ps, **prm, alpha_dyn=1e-4, g=g, Gm0=box.G * box.m0)
    else:
        res, group_of, nm = oracle.coarsen(ps, **prm)
    print(before, members, size, theta, R, "groups", nm, "left", res["x"].shape[0], "of", n,
          flush=True)
    st = dz.State.from_host(ps, g=g) if dyn else dz.State.from_host(ps)
    ctx = dz.Context(n, 16)
    gof = torch.zeros(n, dtype=torch.int32, device="cuda")
    rep = ctx.dzs_coarsen(box, st, cp, group_of=gof)
    torch.cuda.synchronize()
    out = st.to_host()
    ctx.close()
    assert rep.n_groups == nm and rep.n_before == n and rep.n_after == res["x"].shape[0]
    for k in ("x", "y", "z", "px", "py", "pz", "mult", "id", "type"):
        assert np.array_equal(out[k], res[k]), k
    assert np.array_equal(gof.cpu().numpy().astype(np.int64), group_of)


@pytest.mark.parametrize("members,theta,R", [(100000, 0.1, 60.0), (100000, 0.003, 0.0)])
def test_a_clump_takes_no_longer_than_spread_particles(dz, members, theta, R):
    import time

    import torch
    took = []
    for size in (25.0, 0.5):
        ps = _set(20000, members, size, 2000, seed=4)
        cp = dz.CoarsenParams()
        for d in range(3):
            cp.x_obs[d] = 60.0
        cp.R_lc, cp.theta, cp.k_min = R, theta, 4
        ctx = dz.Context(ps.n, 16)
        best = 1e9
        for _ in range(6):
            st = dz.State.from_host(ps)
            torch.cuda.synchronize()
            t = time.perf_counter()
            ctx.dzs_coarsen(dz.make_box(L, 1.0, L / 1000), st, cp)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        ctx.close()
        took.append(best * 1e6)
    print(f"spread {took[0]:.0f} us, clump {took[1]:.0f} us", flush=True)
    assert took[1] <= 3 * took[0]
