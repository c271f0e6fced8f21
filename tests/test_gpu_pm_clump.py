"""pm_force of a set in no order with most particles in one dense clump (paper Sec. 2.1).

The particles of a clump smaller than a sixteenth of the box are close to each other in any order,
so closeness alone does not show one; taken as they come, a clump's atomics queue on the same mesh
points (forty times the time of the same set in key order).  The shuffled set must take no more
than four times the time of the ordered one: the sort costs about as much as the force itself.
The forces are the same bits, particle by particle, as without sort and tiles (tile_chunk = -1),
for sets in no order, in key order and at few points.  Where nothing is sorted (few particles, fine
meshes) the lanes of a wave that share a mesh cell add their integers up first.
"""
import time

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


def _state(dz, x):
    import torch
    n = len(x)
    st = dz.State(n)
    st.n = n
    for a, k in enumerate(("x", "y", "z")):
        getattr(st, k)[:n] = torch.tensor(x[:, a])
    st.mult[:n] = torch.tensor((np.arange(n) % 7 + 1).astype(np.int32))
    return st


def _key_order(x):
    c = (x * (32768 / L)).astype(np.int64)
    key = np.zeros(len(x), np.int64)
    for b in range(15):
        for d in range(3):
            key |= ((c[:, d] >> b) & 1) << (3 * b + 2 - d)
    return x[np.argsort(key, kind="stable")]


def _compare(dz, n, ng, size):
    """The forces of the set in key order and shuffled, each with the bits of the direct kernels,
    and the shuffled one's time against the ordered one's."""
    import torch
    rng = np.random.default_rng(n + ng)
    x = rng.uniform(0, L, (n, 3))
    m = 9 * n // 10
    x[:m] = 71.0 + size * rng.random((m, 3))
    x = x[rng.permutation(n)]
    box = dz.make_box(L, 1.0, L / 2000)
    ctx = dz.Context(n, ng)
    took = []
    for pos in (_key_order(x), x):
        st = _state(dz, pos)
        out = []
        for chunk in (-1, 0):
            prm = dz.PMParams(ng, dz.DZS_FP64, 1.25 * L / ng, 0, chunk)
            ctx.pm_force(box, st, prm)
            torch.cuda.synchronize()
            out.append(np.stack([getattr(st, k)[:n].cpu().numpy() for k in ("gx", "gy", "gz")]))
        assert np.abs(out[0]).max() > 0 and np.array_equal(out[0], out[1])
        best = 1e9
        for _ in range(6):
            t = time.perf_counter()
            for _ in range(4):
                ctx.pm_force(box, st, prm)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        took.append(best / 4 * 1e6)
    ctx.close()
    print(f"{n} on {ng}^3, clump {size}: ordered {took[0]:.0f} us, shuffled {took[1]:.0f} us",
          flush=True)
    assert took[1] <= 4 * took[0]


@pytest.mark.parametrize("n,ng,size", [(131072, 64, 0.5), (300001, 64, 5.0), (131072, 64, 0.0)])
def test_a_shuffled_clump_is_sorted(dz, n, ng, size):
    _compare(dz, n, ng, size)


# too few particles for the sort, or too fine a mesh; waves of 64 alone and four to a workgroup, a
# last one of 1 and of 33 lanes
@pytest.mark.parametrize("n,ng,size", [(4097, 32, 0.5), (60001, 64, 0.5), (70049, 64, 0.0),
                                       (131072, 162, 0.5)])
def test_a_shuffled_clump_adds_up_before_its_atomics(dz, n, ng, size):
    _compare(dz, n, ng, size)
