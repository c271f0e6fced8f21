"""The walk's teams, short groups and FP32 force table against the FP64 oracle's direct sum.

Opening angle 0 (every node opened), so the walk is a direct sum over the cutoff: FP64 forces to
1e-9 of the oracle's and FP32 ones to 1e-5 (the precision form's bar) over the targets with no
pair within FP32 rounding of the cutoff, where the force jumps.  The pairs counted are those of
the cutoff sphere, self pairs and coincident particles left out, as a k-d tree finds them.
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


def _near_cut(ps, L, r_cut):
    """Targets with a pair within 1e-6 of r_cut, and the number of pairs (ordered) inside it at
    a separation above zero."""
    from scipy.spatial import cKDTree
    pos = np.stack([ps.x, ps.y, ps.z], axis=1)
    pairs = cKDTree(pos, boxsize=L).query_pairs(r_cut * (1 + 1e-6), output_type="ndarray")
    d = pos[pairs[:, 0]] - pos[pairs[:, 1]]
    d -= L * np.round(d / L)
    r = np.sqrt((d ** 2).sum(1))
    flag = np.zeros(ps.n, bool)
    flag[pairs[r >= r_cut * (1 - 1e-6)].ravel()] = True
    return flag, 2 * int(((r < r_cut) & (r > 0)).sum())


# n and group size: one wave's groups (1, 2, 33 of 64, 64, 65), teams of four (n / group < 1024),
# of two, and none; softening: usual, and so small that close pairs lie below the FP32 table
@pytest.mark.parametrize("n,group,eps_frac", [
    (1, 64, 40), (2, 16, 40), (33, 64, 40), (64, 64, 40), (65, 64, 40), (700, 64, 4e4),
    (3000, 4, 40), (3000, 16, 4e4), (16383, 16, 40), (16384, 16, 40), (65536, 16, 40)])
@pytest.mark.parametrize("fp32", [False, True])
def test_walk_teams_and_short_groups(dz, n, group, eps_frac, fp32):
    L = 100.0
    r_s = 1.25 * L / 64 if n < 10000 else 1.25 * L / 160
    r_cut = 4.5 * r_s
    ps = dzs_ics.merged_state(dzs_ics.clustered_random(n, L, seed=n, r_clump=L / 20), seed=3,
                              max_mult=16)
    if n >= 64:   # coincident particles: no pair
        ps.x[5], ps.y[5], ps.z[5] = ps.x[6], ps.y[6], ps.z[6]
    lam = L / max(1, round(n ** (1 / 3)))
    m0 = dzs_ics.particle_mass(L, n)
    box, obox = dz.make_box(L, m0, lam / eps_frac), oracle.Box(L=L, m0=m0, eps0=lam / eps_frac)
    ctx = dz.Context(n, 0)
    st = dz.State.from_host(ps)
    ctx.pair_interactions(reset=True)
    ctx.tree_force(box, st, dz.TreeParams(r_s, r_cut, 0.0, 8, group,
                                          dz.DZS_FP32 if fp32 else dz.DZS_FP64, 0))
    ctx.check()
    g = np.stack([st.gx[:n].cpu().numpy(), st.gy[:n].cpu().numpy(), st.gz[:n].cpu().numpy()])
    pairs = ctx.pair_interactions(reset=True)
    ctx.close()
    near, inside = _near_cut(ps, L, r_cut)
    if n > 20000:   # the oracle on a sample of the targets
        t = np.sort(dzs_ics.rng(1).choice(n, 4000, replace=False))
    else:
        t = np.arange(n)
    ref = oracle.short_range(ps.x, ps.y, ps.z, ps.mult, obox, r_s, r_cut, targets=t)
    ref = np.stack(ref) if not isinstance(ref, np.ndarray) else ref
    g = g[:, t]
    if fp32:
        assert abs(pairs - inside) <= 2 * int(near.sum())
        g, ref = g[:, ~near[t]], ref[:, ~near[t]]
    else:
        assert pairs == inside
    if n <= 2 and not ref.any():
        assert not g.any()
        return
    err = math.sqrt(((g - ref) ** 2).sum() / (ref ** 2).sum())
    print(f"n {n} group {group} fp32 {fp32}: rms {err:.2e}, pairs {pairs}", flush=True)
    assert err <= (1e-5 if fp32 else 1e-9)
