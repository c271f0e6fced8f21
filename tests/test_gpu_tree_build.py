"""The tree build at the edges of its blocks and tiers, through tree_force, against the FP64
oracle's direct sum.

At opening angle 0 every particle within the cutoff is reached exactly once or the pair count is
wrong, and the forces agree to 1e-9.  (The nodes' masses and centres show at opening angles above
0, in the other tree tests.)  Sizes lie around the 1024 particles of a build block and the 32 blocks of a tier; the
clump sets reach the deepest level (coincident particles), leaves are 1 to 64 particles.
"""
import math

import numpy as np
import pytest

import dzs_ics
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_05328_amd as dz
    return dz


def _set(kind, n, L):
    if kind == "uniform":
        return dzs_ics.uniform_random(n, L, seed=n)
    ps = dzs_ics.clustered_random(n, L, seed=n, n_clumps=3, r_clump=L / 2000)
    if kind == "coincident":   # runs of equal positions: leaves at the deepest level
        for a in range(0, n - 200, 397):
            for arr in (ps.x, ps.y, ps.z):
                arr[a:a + 100] = arr[a]
    return ps


@pytest.mark.parametrize("kind,n,leaf", [
    ("uniform", 1, 8), ("uniform", 9, 8), ("uniform", 1023, 8), ("uniform", 1024, 1),
    ("uniform", 1025, 64), ("uniform", 2047, 13), ("uniform", 32767, 8), ("uniform", 32768, 8),
    ("uniform", 32769, 16), ("clump", 5000, 8), ("clump", 33000, 64), ("coincident", 4096, 8),
    ("coincident", 40000, 16)])
def test_tree_build_edges(dz, kind, n, leaf):
    L = 100.0
    r_s = 1.25 * L / 96
    r_cut = 4.5 * r_s
    ps = _set(kind, n, L)
    m0 = dzs_ics.particle_mass(L, n)
    eps = L / max(1, round(n ** (1 / 3))) / 40
    box, obox = dz.make_box(L, m0, eps), oracle.Box(L=L, m0=m0, eps0=eps)
    ctx = dz.Context(4 * n, 0)   # room for leaves of one particle
    st = dz.State.from_host(ps)
    ref = oracle.short_range(ps.x, ps.y, ps.z, ps.mult, obox, r_s, r_cut)
    scale = math.sqrt((ref ** 2).sum()) if ref.any() else 1.0
    ctx.pair_interactions(reset=True)
    ctx.tree_force(box, st, dz.TreeParams(r_s, r_cut, 0.0, leaf, 32, dz.DZS_FP64, 0))
    ctx.check()
    g = np.stack([getattr(st, k)[:n].cpu().numpy() for k in ("gx", "gy", "gz")])
    err = math.sqrt(((g - ref) ** 2).sum()) / scale
    got = ctx.pair_interactions(reset=True)
    ctx.close()
    from scipy.spatial import cKDTree
    pos = np.stack([ps.x, ps.y, ps.z], axis=1)
    pairs = cKDTree(pos, boxsize=L).query_pairs(r_cut * (1 + 1e-12), output_type="ndarray")
    d = pos[pairs[:, 0]] - pos[pairs[:, 1]]
    d -= L * np.round(d / L)
    r2 = (d ** 2).sum(1)
    inside = 2 * int(((r2 < r_cut * r_cut) & (r2 > 0)).sum())
    print(f"{kind} n {n} leaf {leaf}: rms {err:.2e}, pairs {got} of {inside}", flush=True)
    # (a pair within rounding of the cutoff may fall on either side)
    edge = 2 * int((np.abs(r2 - r_cut * r_cut) < 1e-12 * r_cut * r_cut).sum())
    assert err <= 1e-9 and abs(got - inside) <= edge


def test_tree_build_over_capacity_is_flagged_and_stays_exact(dz):
    """Leaves of one particle need more nodes than the context holds: the levels that do not fit
    are left out, which makes their parents leaves; the overflow is reported and the opening-angle-0
    force is still the direct sum."""
    n, L = 30000, 100.0
    r_s = 1.25 * L / 96
    ps = dzs_ics.uniform_random(n, L, seed=1)
    m0 = dzs_ics.particle_mass(L, n)
    box, obox = dz.make_box(L, m0, 0.1), oracle.Box(L=L, m0=m0, eps0=0.1)
    ctx = dz.Context(n, 0)
    st = dz.State.from_host(ps)
    ctx.tree_force(box, st, dz.TreeParams(r_s, 4.5 * r_s, 0.0, 1, 32, dz.DZS_FP64, 0))
    with pytest.raises(dz.DZSError) as e:
        ctx.check()
    assert e.value.code == -3
    g = np.stack([getattr(st, k)[:n].cpu().numpy() for k in ("gx", "gy", "gz")])
    ctx.check()   # reported once
    ctx.close()
    ref = oracle.short_range(ps.x, ps.y, ps.z, ps.mult, obox, r_s, 4.5 * r_s)
    assert math.sqrt(((g - ref) ** 2).sum() / (ref ** 2).sum()) <= 1e-9
