"""DZS coarsening (paper Sec. 2.2, eqs. 1 and 3) where the workgroups' tiles end: bit for bit
against the oracle, as everywhere (the sums follow the members' order on both sides).

A workgroup owns the cubes that begin in its 256 particles and holds 336 rows in LDS, rows
behind are read from memory; levels whose cubes hold more than 256 particles on average take a
launch each.  So: counts around 256 and 336, a cube of thousands of members (past the rows in
LDS, over several tiles of its workgroup), particles at one point (equal keys down to the last
level), a k_min of 1 for thousands of particles, nobody near the observer, everybody near.
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


def _set(kind, n):
    if kind == "clump":      # two thirds in a clump of one or two cubes, the rest everywhere
        ps = dzs_ics.uniform_random(n, L, seed=n)
        r = dzs_ics.rng(n + 1)
        m = 2 * n // 3
        for a, k in enumerate(("x", "y", "z")):
            getattr(ps, k)[:m] = 71.0 + 1.0 * r.random(m)
    elif kind == "points":   # runs of equal positions
        ps = dzs_ics.uniform_random(n, L, seed=n)
        for k in ("x", "y", "z"):
            v = getattr(ps, k)
            v[:] = v[np.arange(n) // 5 * 5]
    else:
        ps = dzs_ics.uniform_random(n, L, seed=n)
    r = dzs_ics.rng(n + 2)
    for k in ("px", "py", "pz"):
        getattr(ps, k)[:] = r.standard_normal(n) * 300.0
    ps.mult = r.integers(1, 20, n).astype(np.uint32)
    ps.id = r.permutation(n).astype(np.uint32)
    return ps


@pytest.mark.parametrize("kind,n,k_min,R,theta", [
    ("uniform", 2, 1, 5.0, 1.0), ("uniform", 255, 2, 5.0, 1.0), ("uniform", 256, 2, 5.0, 1.0),
    ("uniform", 257, 2, 5.0, 1.0), ("uniform", 336, 1, 0.0, 4.0), ("uniform", 337, 1, 0.0, 4.0),
    ("uniform", 4001, 1, 20.0, 2.0), ("clump", 9000, 3, 10.0, 1.0), ("clump", 9000, 1, 10.0, 8.0),
    ("points", 3000, 4, 30.0, 0.5), ("uniform", 3000, 3, 86.0, 1.0), ("points", 700, 6, 40.0, 4.0)])
def test_coarsen_tile_edges(dz, kind, n, k_min, R, theta):
    import torch
    ps = _set(kind, n)
    prm = dict(x_obs=[20.0, 30.0, 40.0], R_lc=R, b=1.0, theta=theta, k_min=k_min)
    res, group_of, nm = oracle.coarsen(ps, **prm)
    print(kind, n, k_min, R, "groups", nm, "left", res["x"].shape[0], flush=True)
    st = dz.State.from_host(ps)
    cp = dz.CoarsenParams()
    for d in range(3):
        cp.x_obs[d] = prm["x_obs"][d]
    cp.R_lc, cp.b, cp.theta, cp.k_min = R, 1.0, theta, k_min
    ctx = dz.Context(n, 16)
    gof = torch.zeros(n, dtype=torch.int32, device="cuda")
    rep = ctx.dzs_coarsen(dz.make_box(L, 1.0, L / 1000), st, cp, group_of=gof)
    torch.cuda.synchronize()
    out = st.to_host()
    ctx.close()
    assert rep.n_groups == nm and rep.n_before == n and rep.n_after == res["x"].shape[0]
    for k in ("x", "y", "z", "px", "py", "pz", "mult", "id", "type"):
        assert np.array_equal(out[k], res[k]), k
    assert np.array_equal(gof.cpu().numpy().astype(np.int64), group_of)
