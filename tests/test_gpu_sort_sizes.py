"""The sort at the edges of its forms: by counting (up to 32768 keys), tiles of 4096, column
segments of 64 tiles and several segments.  dzs_sort_state's permutation is the stable order of
the keys, bit for bit, on scattered, nearly sorted and heavily repeated keys."""
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


@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 8191, 8192, 8193, 12289, 262144, 262145,
                               300001, 700003])
@pytest.mark.parametrize("kind", ["random", "near", "few"])
def test_sort_sizes(dz, n, kind):
    import torch
    L = 64.0
    ps = dzs_ics.uniform_random(n, L, seed=n)
    if kind == "few":        # 27 distinct positions: long runs of equal keys
        for a in (ps.x, ps.y, ps.z):
            a[:] = np.floor(a / (L / 3)) * (L / 3) + 1.0
    elif kind == "near":     # key order with one in fifty moved
        o = np.argsort(oracle.morton_keys(ps.x, ps.y, ps.z, L), kind="stable")
        moved = dzs_ics.rng(n + 1).random(n) < 0.02
        for a in (ps.x, ps.y, ps.z):
            a[:] = a[o]
        ps.x[moved] = (ps.x[moved] + 0.3) % L
    box = dz.make_box(L, 1.0, 1.0)
    ctx = dz.Context(n, 0)
    st = dz.State.from_host(ps)
    perm = torch.zeros(n, dtype=torch.int32, device="cuda")
    ctx.sort_state(box, st, perm=perm)
    torch.cuda.synchronize()
    ref = np.argsort(oracle.morton_keys(ps.x, ps.y, ps.z, L), kind="stable")
    assert np.array_equal(perm.cpu().numpy(), ref)
    assert np.array_equal(st.id[:n].cpu().numpy(), ref.astype(np.int32))
    assert np.array_equal(st.px[:n].cpu().numpy(), ps.px[ref])
    ctx.close()


@pytest.mark.parametrize("n", [127, 256, 257, 511, 513, 20000, 32767, 32768, 32769])
@pytest.mark.parametrize("few", [False, True])
def test_sort_by_counting_sizes(dz, n, few):
    """Up to 32768 keys are placed by counting, in segments and blocks of 256: the same stable
    order."""
    import torch
    L = 64.0
    ps = dzs_ics.uniform_random(n, L, seed=n)
    if few:                  # one cell in eight of 8, equal keys across every segment
        for a in (ps.x, ps.y, ps.z):
            a[:] = np.floor(a / (L / 2)) * (L / 2) + 1.0
    ctx = dz.Context(n, 0)
    st = dz.State.from_host(ps)
    perm = torch.zeros(n, dtype=torch.int32, device="cuda")
    ctx.sort_state(dz.make_box(L, 1.0, 1.0), st, perm=perm)
    torch.cuda.synchronize()
    ref = np.argsort(oracle.morton_keys(ps.x, ps.y, ps.z, L), kind="stable")
    assert np.array_equal(perm.cpu().numpy(), ref)
    assert np.array_equal(st.id[:n].cpu().numpy(), ref.astype(np.int32))
    ctx.close()
