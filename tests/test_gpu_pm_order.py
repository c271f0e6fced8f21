"""pm_force of particles in no order (sorted by their keys' top digits into scratch first)
against the direct kernels (paper Sec. 2.1).

The deposit adds 32.32 fixed-point contributions with integer atomics and the interpolation
evaluates each particle by itself, so the order the particles are worked in changes no bit: the
default must equal tile_chunk = -1, which neither sorts nor tiles.  Sizes: below, at and above
the least count that is sorted, an odd count, a mesh fine enough for four sort passes and one
too fine to sort for; lattice order (taken as it is) and random order; both forms; the
accumulated force; positions on the box's edges.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

L = 100.0


@pytest.fixture(scope="module")
def dz():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2005_05328_amd as dz
    return dz


def _state(dz, n, order, seed):
    import torch
    rng = np.random.default_rng(seed)
    if order == "clump":   # nine in ten in a few dense clumps
        c = rng.uniform(0, L, (5, 3))
        x = np.where(rng.random((n, 1)) < 0.9, c[rng.integers(0, 5, n)] + rng.normal(0, 0.4, (n, 3)),
                     rng.uniform(0, L, (n, 3)))
        x = np.mod(x, L)
    else:
        x = rng.uniform(0, L, (n, 3))
        x[:64] = 0.0
        x[64:128] = np.nextafter(L, 0.0)
    x[x >= L] = 0.0
    if order == "lattice":
        x = x[np.lexsort((np.floor(x[:, 2] / 2), np.floor(x[:, 1] / 2), np.floor(x[:, 0] / 2)))]
    st = dz.State(n)
    st.n = n
    for a, k in enumerate(("x", "y", "z")):
        getattr(st, k)[:n] = torch.tensor(x[:, a])
    st.mult[:n] = torch.tensor(rng.integers(1, 9, n).astype(np.int32))
    return st


def _g(st):
    import torch
    torch.cuda.synchronize()
    return np.stack([getattr(st, k)[:st.n].cpu().numpy() for k in ("gx", "gy", "gz")])


@pytest.mark.parametrize("n,ng,order,fp32", [
    (131071, 32, "random", False), (131072, 32, "random", False), (131073, 64, "clump", False),
    (262145, 64, "clump", True), (150001, 96, "lattice", False), (800003, 288, "random", True),
    (131072, 192, "random", False)])
def test_unordered_particles_get_the_same_force(dz, n, ng, order, fp32):
    st = _state(dz, n, order, seed=n + ng)
    box = dz.make_box(L, 1.0, L / 2000)
    ctx = dz.Context(n, ng)
    out = {}
    for chunk in (-1, 0):
        for acc in (0, 1):
            for k in ("gx", "gy", "gz"):
                getattr(st, k).fill_(3.0)
            prm = dz.PMParams(ng, dz.DZS_FP32 if fp32 else dz.DZS_FP64, 1.25 * L / ng, acc, chunk)
            ctx.pm_force(box, st, prm)
            out[chunk, acc] = _g(st)
    ctx.close()
    print(n, ng, order, float(np.abs(out[-1, 0]).max()), flush=True)
    assert np.abs(out[-1, 0]).max() > 0
    assert np.array_equal(out[0, 0], out[-1, 0])
    assert np.array_equal(out[0, 1], out[-1, 1])
