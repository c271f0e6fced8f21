"""The precision form of the short-range force in any unit of length (paper Sec. 2.1).

The force goes with L^-2 when every length (positions, softening, split scale, cutoff) goes with
L, and the library sets no limit on the unit.  The same set in boxes of 100 2^k: powers of two
change no rounding, in FP64 or FP32, while every intermediate stays in the FP32 range, so the
forces times 4^k are the same bits at every scale (at k = 0 test_gpu_walk_teams compares them
with the oracle's direct sum).  The largest intermediate is some 11 m / h^3 (a pair inside its
softening h): 5e15 at k = 0 and so in range down to k = -25.  Softening far below the spacing, so
that pairs lie in every part of the table of far pairs, to its low end and below.
"""
import numpy as np
import pytest

import dzs_ics

pytestmark = pytest.mark.gpu

L0 = 100.0


@pytest.fixture(scope="module")
def dz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_05328_amd as dz
    return dz


def _force(dz, k, n, group, ng=64, eps_frac=4e4, mass=1.0):
    """The FP32 short-range force in a box of 100 2^k, in units of the force at k = 0, mass = 1."""
    s = 2.0 ** k
    ps = dzs_ics.merged_state(dzs_ics.clustered_random(n, L0, seed=n, r_clump=L0 / 50), seed=3,
                              max_mult=16)
    rng = dzs_ics.rng(n + 1)
    for a in ("x", "y", "z"):   # one in eight beside its neighbour, at all small separations
        v = getattr(ps, a)
        m = np.arange(0, n - 1, 8)
        v[m] = v[m + 1] + rng.standard_normal(len(m)) * 10.0 ** rng.uniform(-4, -1, len(m))
        v[:] = np.mod(v, L0) * s
    ps.L = L0 * s
    r_s = 1.25 * ps.L / ng
    box = dz.make_box(ps.L, dzs_ics.particle_mass(L0, n) * mass,
                      ps.L / round(n ** (1 / 3)) / eps_frac)
    ctx = dz.Context(n, 0)
    st = dz.State.from_host(ps)
    ctx.tree_force(box, st, dz.TreeParams(r_s, 4.5 * r_s, 0.0, 8, group, dz.DZS_FP32, 0))
    ctx.check()
    g = np.stack([getattr(st, a)[:n].cpu().numpy() for a in ("gx", "gy", "gz")])
    ctx.close()
    return g * s * s / mass


# teams of four waves, groups on few lanes (the masked loop at 4), one wave a group
@pytest.mark.parametrize("n,group", [(700, 64), (3000, 4), (70001, 16)])
def test_fp32_force_scales_with_the_unit_of_length(dz, n, group):
    one = _force(dz, 0, n, group)
    assert np.isfinite(one).all() and np.abs(one).max() > 0
    for k in (-10, -14, -20, 14, 24):
        g = _force(dz, k, n, group)
        print(f"n {n} group {group} box {L0 * 2.0 ** k:.3g}: {(~np.isfinite(g)).sum()} not finite, "
              f"largest difference {np.abs(g - one).max() / np.abs(one).max():.1e}", flush=True)
        assert np.array_equal(g, one), f"box {L0 * 2.0 ** k:.3g}"


def test_fp32_force_where_the_table_begins_later(dz):
    """r_cut^2 = 2^-67.7: the table of far pairs begins at 2^-83, above r_cut^2 / 2^16, so that its
    coefficients are in range.  The pairs below lie inside the softening here (h from r_cut / 18,
    the table from r_cut / 200), whose force is the same arithmetic at every scale: the same bits.
    A mass unit of 2^-60 keeps mass over h^3 in range."""
    one = _force(dz, 0, 3000, 16, ng=16, eps_frac=10.0)
    g = _force(dz, -39, 3000, 16, ng=16, eps_frac=10.0, mass=2.0 ** -60)
    print(f"largest difference {np.abs(g - one).max() / np.abs(one).max():.1e}", flush=True)
    assert np.isfinite(one).all() and np.array_equal(g, one)
