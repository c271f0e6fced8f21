"""The measured workloads of the gravity step: listed cases and draws of the same ranges.

Every case is one call that a simulation program makes through the public entry points, with
the context, the state and the parameter blocks such a program keeps between its calls:

  step      kdk_step: one global kick-drift-kick step, with or without DZS coarsening
  coarsen   dzs_coarsen alone (run control between steps)
  batch     kdk_step_batch: one step of an ensemble of uneven boxes
  hier      kdk_step_hier: one global step with individual time steps
  pm        pm_force (or pm_force_noalloc): the long-range force alone
  tree      tree_force: the short-range force alone, of all particles or of a subset
  cone      lightcone_emit: the crossing test and solve of one drift

Inputs are made on the GPU from the seed: a lattice displaced by a Gaussian random field
(linear-theory positions and momenta), or a clustered set (Plummer clumps over a uniform
background).  Steps advance the state by a short interval in ln a, so that repeated passes
stay in the same epoch.  A pass that merges particles starts from a snapshot of its state,
which it restores first: a merged state has nothing left to merge.

The precision form computes the force in FP32 and stores it in FP64 arrays; the programs of
its cases keep the force as FP32 output, which is what they return.
"""
from __future__ import annotations

import math

import torch

import paper_2005_05328_amd as dz

G = 43.0091
OMEGA_M = 0.3
RHO = OMEGA_M * 3.0e4 / (8.0 * math.pi * G)   # mean matter density, 1e10 Msun/h (Mpc/h)^-3
DLNA = 1e-4                                   # the interval of one step
ARRAYS = ("x", "y", "z", "px", "py", "pz", "gx", "gy", "gz", "mult", "id", "type")
DEV = "cuda:0"


def listed():
    return [
        # the smallest run: 20^3 particles, a few hundred microseconds of short launches
        dict(name="step_20cube_fp64", kind="step", n_side=20, L=50.0, ng=48, a=0.3, disp=0.5,
             prec="fp64", leaf=8, group=32, cone=False, merge=""),
        # the 128^3 run in the plain form: mesh twice as fine as the particles
        dict(name="step_128cube_fp64", kind="step", n_side=128, L=256.0, ng=256, a=0.1, disp=0.35,
             prec="fp64", leaf=16, group=32, cone=True, merge=""),
        # the 256^3, 2 Gpc/h run in the precision form, the sphere inside the box
        dict(name="step_256cube_fp32", kind="step", n_side=256, L=2000.0, ng=256, a=0.75,
             disp=0.6, prec="fp32", leaf=8, group=64, cone=True, merge=""),
        # the 512^3, 1 Gpc/h run in the precision form, the largest that runs in three copies
        dict(name="step_512cube_fp32", kind="step", n_side=512, L=1000.0, ng=512, a=0.1,
             disp=0.35, prec="fp32", leaf=8, group=64, cone=True, merge=""),
        # a step whose DZS pass merges most of a 128^3 box outside the lightcone
        dict(name="step_128cube_merging", kind="step", n_side=128, L=2000.0, ng=128, a=0.9,
             disp=0.6, prec="fp32", leaf=8, group=64, cone=True, merge="geometric"),
        # one coarsening of a 96^3 box, as an ensemble's run control does before it re-packs
        dict(name="coarsen_96cube", kind="coarsen", n_side=96, L=384.0, disp=0.6, R=0.25,
             theta=1.0, lmax=4, crit="geometric"),
        # an ensemble of 64 uneven boxes in one call, mixed multiplicities
        dict(name="batch_64_boxes", kind="batch", boxes=64, sides="16,24,32,48", prec="fp32",
             leaf=16, group=64, merged=True),
        # individual time steps over four bins, the long-range force on the global step
        dict(name="hier_48cube_fp64", kind="hier", n=110592, L=100.0, ng=64, bins=3, prec="fp64",
             pm_global=True),
        # the long-range force of a clustered set in no order, an odd count, a 2^a 3^b mesh
        dict(name="pm_1e6_mesh192", kind="pm", n=1000003, L=300.0, ng=192, prec="fp64",
             clustered=True, noalloc=False),
        # the smallest call: the allocation-free long-range force on a small mesh
        dict(name="pm_noalloc_mesh32", kind="pm", n=4099, L=50.0, ng=32, prec="fp64",
             clustered=False, noalloc=True),
        # the short-range force of a subset of targets in a clustered set in no order
        dict(name="tree_200k_subset", kind="tree", n=200003, L=100.0, targets=20011, prec="fp64",
             leaf=8, group=16, opening="geometric"),
        # the lightcone output of one drift of 4 million particles
        dict(name="cone_4e6", kind="cone", n=4000037, L=500.0, a=0.95, dlna=2e-3),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


MESHES = (8, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144, 162, 192, 216, 256, 288,
          324, 384, 432, 486, 512)   # even 2^a 3^b sides


def _mesh(side):
    return min(MESHES, key=lambda m: abs(math.log(m / side)))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "coarsen", "batch", "hier", "pm", "pm", "tree",
                       "tree", "cone"))
    prec = rng.choice(("fp64", "fp32"))
    if kind == "step":
        n_side = int(round(_log(rng, 16, 300 if prec == "fp32" else 160)))
        lam = rng.choice((2.0, 4.0, 8.0)) * rng.uniform(0.8, 1.25)
        merge = rng.choice(("", "", "geometric", "dynamical")) if n_side >= 32 else ""
        return dict(kind=kind, n_side=n_side, L=round(n_side * lam, 3),
                    ng=_mesh(min(512, n_side * rng.choice((1.0, 1.0, 2.0)))),
                    a=round(rng.uniform(0.05, 0.9), 3), disp=round(rng.uniform(0.1, 0.6), 3),
                    prec=prec, leaf=rng.choice((8, 16)),
                    group=64 if prec == "fp32" else rng.choice((16, 32)),
                    cone=rng.random() < 0.7, merge=merge)
    if kind == "coarsen":
        n_side = int(round(_log(rng, 16, 160)))
        return dict(kind=kind, n_side=n_side, L=round(4.0 * n_side, 3),
                    disp=round(rng.uniform(0.1, 0.6), 3), R=round(rng.uniform(0.1, 0.4), 3),
                    theta=rng.choice((0.1, 0.5, 1.0)), lmax=rng.choice((2, 4, 8)),
                    crit=rng.choice(("geometric", "dynamical")))
    if kind == "batch":
        sides = [str(rng.choice((16, 18, 24, 32, 36, 48))) for _ in range(rng.randint(2, 4))]
        return dict(kind=kind, boxes=rng.randint(3, 64), sides=",".join(sides), prec=prec,
                    leaf=rng.choice((8, 16, 32)), group=rng.choice((32, 64)),
                    merged=rng.random() < 0.5)
    if kind == "hier":
        n = int(_log(rng, 5000, 300000))
        return dict(kind=kind, n=n, L=100.0, ng=rng.choice((48, 64, 96)), bins=rng.randint(1, 3),
                    prec=prec, pm_global=rng.random() < 0.5)
    if kind == "pm":
        if rng.random() < 0.3:
            return dict(kind=kind, n=int(_log(rng, 500, 100000)), L=50.0,
                        ng=rng.choice((16, 24, 32, 48, 64)), prec=prec, clustered=False,
                        noalloc=True)
        return dict(kind=kind, n=int(_log(rng, 1000, 8e6)), L=300.0,
                    ng=_mesh(_log(rng, 32, 384)), prec=prec, clustered=rng.random() < 0.5,
                    noalloc=False)
    if kind == "tree":
        n = int(_log(rng, 1000, 500000))
        return dict(kind=kind, n=n, L=100.0, targets=rng.choice((0, max(1, n // 10), n // 2)),
                    prec=prec, leaf=rng.choice((8, 16)), group=rng.choice((16, 32, 64)),
                    opening=rng.choice(("geometric", "geometric", "relative")))
    return dict(kind=kind, n=int(_log(rng, 1000, 2e7)), L=500.0,
                a=round(rng.uniform(0.93, 0.97), 4), dlna=round(_log(rng, 2e-4, 5e-3), 6))


# ---- inputs ----------------------------------------------------------------------------------

def _prec(case):
    return dz.DZS_FP32 if case["prec"] == "fp32" else dz.DZS_FP64


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 11)
    return g


def _rate(a):
    """a^2 H(a) f(a), the momentum of a unit linear displacement (flat LCDM)."""
    e2 = OMEGA_M * a ** -3 + 1.0 - OMEGA_M
    return a * a * 100.0 * math.sqrt(e2) * (OMEGA_M * a ** -3 / e2) ** 0.55


def _wrap(v, L):
    v = torch.remainder(v, L)
    return torch.where(v >= L, torch.zeros_like(v), v)


def _displaced(n_side, L, a, disp, gen):
    """A lattice displaced by a Gaussian field with P(k) ~ k^-2, rms `disp` spacings per axis."""
    lam = L / n_side
    dk = torch.fft.rfftn(torch.randn((n_side,) * 3, generator=gen, device=DEV,
                                     dtype=torch.float64))
    k1 = torch.fft.fftfreq(n_side, 1.0 / n_side, device=DEV, dtype=torch.float64)
    k3 = torch.fft.rfftfreq(n_side, 1.0 / n_side, device=DEV, dtype=torch.float64)
    ks = (k1[:, None, None], k1[None, :, None], k3[None, None, :])
    k2 = ks[0] ** 2 + ks[1] ** 2 + ks[2] ** 2
    k2[0, 0, 0] = 1.0
    dk *= k2 ** -1.5          # the field, k^-1, over k^2
    dk[0, 0, 0] = 0.0
    del k2
    q = (torch.arange(n_side, device=DEV, dtype=torch.float64) + 0.5) * lam
    pos, mom, unit = [], [], None
    for axis in range(3):
        psi = torch.fft.irfftn(1j * ks[axis] * dk, s=(n_side,) * 3)
        if unit is None:
            unit = disp * lam / float(psi.square().mean().sqrt())
        psi = psi.mul_(unit)
        shape = [1, 1, 1]
        shape[axis] = n_side
        pos.append(_wrap((psi + q.view(shape)).reshape(-1), L))
        mom.append((psi * _rate(a)).reshape(-1))
    return pos, mom


def _clustered(n, L, gen, frac=0.7, clumps=8):
    """`frac` of the points in Plummer clumps of scale L/40, the rest uniform, in no order."""
    u = torch.rand((n, 4), generator=gen, device=DEV, dtype=torch.float64)
    d = torch.randn((n, 3), generator=gen, device=DEV, dtype=torch.float64)
    mom = torch.randn((n, 3), generator=gen, device=DEV, dtype=torch.float64) * 300.0
    centres = torch.rand((clumps, 3), generator=gen, device=DEV, dtype=torch.float64) * L
    which = torch.randint(0, clumps, (n,), generator=gen, device=DEV)
    r = (L / 40.0) / torch.sqrt(u[:, 3].clamp(1e-6, 0.999) ** (-2.0 / 3.0) - 1.0)
    r = r.clamp(max=L / 4.0)
    inside = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) < frac
    p = torch.where(inside[:, None], centres[which] + d / d.norm(dim=1, keepdim=True) * r[:, None],
                    u[:, :3] * L)
    return [_wrap(p[:, k], L) for k in range(3)], [mom[:, k].clone() for k in range(3)]


def _state(pos, mom, mult=None, capacity=None):
    n = pos[0].shape[0]
    st = dz.State(capacity or n, DEV)
    for k, v in zip(("x", "y", "z", "px", "py", "pz"), pos + mom):
        getattr(st, k)[:n] = v
    st.mult[:n] = 1 if mult is None else mult
    if mult is not None:
        st.type[:n] = (mult > 1).to(torch.uint8)
    st.id[:n] = torch.arange(1, n + 1, device=DEV, dtype=torch.int32)
    st.n = n
    return st


def _mixed(n, gen):
    m = torch.randint(2, 65, (n,), generator=gen, device=DEV, dtype=torch.int32)
    return torch.where(torch.rand(n, generator=gen, device=DEV) < 0.3, m, torch.ones_like(m))


def _box(L, n):
    return dz.make_box(L, RHO * L ** 3 / n, L / n ** (1.0 / 3.0) / 40.0, G)


def _split(L, ng):
    r_s = 1.25 * L / ng
    return r_s, 4.5 * r_s


def _k_min(n_side, lmax):
    k = 1
    while n_side > lmax * (1 << k):
        k += 1
    return k


def _coarsen_params(n_side, L, R, b, theta, lmax, crit):
    cp = dz.CoarsenParams()
    cp.R_lc, cp.b, cp.theta, cp.k_min = R * L, b * L / n_side, theta, _k_min(n_side, lmax)
    if crit == "dynamical":
        cp.criterion, cp.alpha_dyn = dz.DZS_CRIT_DYNAMICAL, 1e-2
    return cp


def _still(sp):
    """The same parameters as a force evaluation: no kick, no drift, nothing merged."""
    s = dz.StepParams.from_buffer_copy(sp)
    s.K1 = s.K2 = s.lc.D = 0.0
    s.do_lightcone = s.do_coarsen = 0
    return s


class _Case:
    pass


def _snapshot(st, names=ARRAYS):
    return {k: getattr(st, k)[:st.n].clone() for k in names}


def _restore(s):
    torch._foreach_copy_([getattr(s.st, k) for k in s.snap], list(s.snap.values()))
    s.st.n = s.n0


def _clear_rest(s):
    """The slots past the count to zero: a merging state's outputs are its whole arrays."""
    torch._foreach_zero_([getattr(s.st, k)[s.st.n:] for k in ARRAYS])


def prepare(case, seed):
    s, gen, kind = _Case(), _gen(seed), case["kind"]
    s.case, s.ring, s.snap = case, None, None
    s.fp32 = case.get("prec") == "fp32"
    if kind in ("step", "coarsen"):
        n_side, L = case["n_side"], case["L"]
        pos, mom = _displaced(n_side, L, case.get("a", 0.5), case["disp"], gen)
        n = n_side ** 3
        s.box, s.st = _box(L, n), _state(pos, mom)
        del pos, mom
    if kind == "step":
        ng = case["ng"]
        r_s, r_cut = _split(L, ng)
        s.ctx = dz.Context(n, ng, fp32_meshes=s.fp32, no_copies=True)
        a = case["a"]
        sp = s.prm = dz.step_factors(a, a * math.exp(DLNA), OMEGA_M)
        sp.do_lightcone, sp.do_coarsen = int(case["cone"]), int(case["merge"] != "")
        if case["merge"]:
            sp.coarsen = _coarsen_params(n_side, L, 0.15, 5.0, 0.1, 4, case["merge"])
        sp.pm = dz.PMParams(ng, _prec(case), r_s, 0, 0)
        sp.tree = dz.TreeParams(r_s, r_cut, 0.5, case["leaf"], case["group"], _prec(case), 0)
        if case["cone"]:
            s.ring = dz.LCRing(max(4096, n // 512), DEV)
        s.ctx.kdk_step(s.box, s.st, _still(sp))   # the force that the first kick reads
        if case["merge"]:
            s.n0, s.snap = s.st.n, _snapshot(s.st)
    elif kind == "coarsen":
        s.ctx = dz.Context(n, 0, no_copies=True)
        s.prm = _coarsen_params(n_side, L, case["R"], 0.0, case["theta"], case["lmax"],
                                case["crit"])
        for k, m in zip(("gx", "gy", "gz"), ("px", "py", "pz")):
            getattr(s.st, k).copy_(getattr(s.st, m))
        s.n0 = n
        s.snap = _snapshot(s.st)
        s.group_of = torch.zeros(n, dtype=torch.int32, device=DEV)
    elif kind == "batch":
        sides = [int(v) for v in case["sides"].split(",")]
        pos, mom, s.boxes, s.first, s.ng = [[], [], []], [[], [], []], [], [0], []
        for b in range(case["boxes"]):
            n_side = sides[b % len(sides)]
            L = 128.0 + 256.0 * (b % 8) / 7.0
            p, m = _displaced(n_side, L, 0.1, 0.3, gen)
            for k in range(3):
                pos[k].append(p[k])
                mom[k].append(m[k])
            s.boxes.append(_box(L, n_side ** 3))
            s.first.append(s.first[-1] + n_side ** 3)
            s.ng.append(2 * n_side)
        n = s.first[-1]
        s.st = _state([torch.cat(v) for v in pos], [torch.cat(v) for v in mom],
                      _mixed(n, gen) if case["merged"] else None)
        rs = [_split(bx.L, g) for bx, g in zip(s.boxes, s.ng)]
        s.rs, s.rc = [v[0] for v in rs], [v[1] for v in rs]
        cells, side = sum(g ** 3 for g in s.ng), 8
        while side ** 3 < cells:
            side += 1
        s.ctx = dz.Context(n, side, fp32_meshes=s.fp32, no_copies=True,
                           max_boxes=case["boxes"])
        sp = s.prm = dz.step_factors(0.1, 0.1 * math.exp(DLNA), OMEGA_M)
        sp.do_lightcone = sp.do_coarsen = 0
        sp.pm = dz.PMParams(0, _prec(case), 0.0, 0, 0)
        sp.tree = dz.TreeParams(0.0, 0.0, 0.5, case["leaf"], case["group"], _prec(case), 0)
        s.ctx.kdk_step_batch(s.boxes, s.first, s.ng, s.rs, s.rc, s.st, _still(sp))
    elif kind == "hier":
        n, L, ng = case["n"], case["L"], case["ng"]
        s.box, s.st = _box(L, n), _state(*_clustered(n, L, gen))
        r_s, r_cut = _split(L, ng)
        s.ctx = dz.Context(n, ng, hier_split=True)
        sp = s.prm = dz.StepParams()
        sp.pm = dz.PMParams(ng, _prec(case), r_s, 0, 0)
        sp.tree = dz.TreeParams(r_s, r_cut, 0.5, 8, 32, _prec(case), 0)
        sp.lc.D = 0.0
        s.a0, s.a1 = 0.5, 0.5 * math.exp(DLNA)
        # the usual accuracy parameter for a step of 0.05 in ln a, scaled to this interval
        s.eta = 0.1 * (DLNA / 0.05) ** 2
        s.bins = torch.zeros(n, dtype=torch.uint8, device=DEV)
        s.ctx.kdk_step(s.box, s.st, _still(sp))
    elif kind in ("pm", "tree"):
        n, L = case["n"], case["L"]
        if kind == "tree" or case["clustered"]:
            pos, mom = _clustered(n, L, gen)
        else:
            pos = list((torch.rand((3, n), generator=gen, device=DEV, dtype=torch.float64) * L))
            mom = [torch.zeros_like(p) for p in pos]
        s.box, s.st = _box(L, n), _state(pos, mom)
        if kind == "pm":
            s.ctx = None if case["noalloc"] else dz.Context(n, case["ng"], fp32_meshes=s.fp32,
                                                            no_copies=True)
            s.prm = dz.PMParams(case["ng"], _prec(case), _split(L, case["ng"])[0], 0, 0)
        else:
            s.ctx = dz.Context(n, 0)
            relative = case["opening"] == "relative"
            s.prm = dz.TreeParams(*_split(L, 64), 0.5, case["leaf"], case["group"], _prec(case),
                                  0, dz.DZS_OPEN_RELATIVE if relative else dz.DZS_OPEN_GEOMETRIC,
                                  0, 0.005)
            s.targets = None
            if case["targets"]:
                s.targets = torch.randperm(n, generator=gen, device=DEV)[:case["targets"]].to(
                    torch.int32)
            s.old = None
            if relative:   # the accelerations of the previous step
                for k in ("gx", "gy", "gz"):
                    getattr(s.st, k).copy_(1e4 + 1e3 * torch.rand(n, generator=gen, device=DEV,
                                                                  dtype=torch.float64))
                s.old = _snapshot(s.st, ("gx", "gy", "gz"))
    else:
        n, L = case["n"], case["L"]
        pos = list((torch.rand((3, n), generator=gen, device=DEV, dtype=torch.float64) * L))
        mom = list(torch.randn((3, n), generator=gen, device=DEV, dtype=torch.float64) * 300.0)
        s.box, s.st = _box(L, n), _state(pos, mom)
        s.ctx = dz.Context(n, 0, no_copies=True)
        s.prm = _cone_params(case).lc
        chi = math.sqrt(s.prm.chi2_0), math.sqrt(s.prm.chi2_1)
        shell = 4.0 / 3.0 * math.pi * (chi[0] ** 3 - chi[1] ** 3) / L ** 3
        s.ring = dz.LCRing(256 + int(1.1 * n * shell), DEV)
        s.table = torch.zeros((n + 1, 8), dtype=torch.float64, device=DEV)
    if s.fp32:
        s.g32 = torch.zeros((3, s.st.capacity), dtype=torch.float32, device=DEV)
    return s


def _cone_params(case):
    sp = dz.step_factors(case["a"], case["a"] * math.exp(case["dlna"]), OMEGA_M)
    for d in range(3):
        sp.lc.x_obs[d] = 0.5 * case["L"]
    return sp


# ---- passes ----------------------------------------------------------------------------------

def _rows(s):
    return s.st.n if s.snap is None else s.n0


def _force(s):
    n = _rows(s)
    if not s.fp32:
        return [s.st.gx[:n], s.st.gy[:n], s.st.gz[:n]]
    out = s.g32[:, :n]
    for k, v in enumerate((s.st.gx, s.st.gy, s.st.gz)):
        out[k].copy_(v[:n])
    return [out[0], out[1], out[2]]


def _particles(s, force=True):
    if s.snap is not None:
        _clear_rest(s)
    n = _rows(s)
    out = {k: getattr(s.st, k)[:n] for k in ("x", "y", "z", "px", "py", "pz", "mult", "id",
                                             "type")}
    if force:
        out["g"] = _force(s)
    return out


def _records(ring):
    """The step's records in the order of their ids (unused slots, id 0, first)."""
    words = ring.buf.view(torch.int32).view(-1, 16)
    rows = ring.buf.view(-1, 8).index_select(0, torch.argsort(words[:, 0]))
    ring.buf.zero_()
    return [ring.count.clone(), rows.view(torch.int32).view(-1, 16)[:, :2], rows[:, 1:]]


def run(s):
    kind = s.case["kind"]
    if s.snap is not None:
        _restore(s)
    if kind == "step":
        if s.ring is not None:
            s.ring.reset()
        rep = s.ctx.kdk_step(s.box, s.st, s.prm, s.ring)
        out = _particles(s)
        if s.ring is not None:
            out["records"] = _records(s.ring)
        return [out, int(rep.n_after), int(rep.n_groups)]
    if kind == "coarsen":
        rep = s.ctx.dzs_coarsen(s.box, s.st, s.prm, s.group_of)
        return [_particles(s, False), s.group_of, int(rep.n_after), int(rep.n_groups)]
    if kind == "batch":
        s.ctx.kdk_step_batch(s.boxes, s.first, s.ng, s.rs, s.rc, s.st, s.prm)
        return _particles(s)
    if kind == "hier":
        s.ctx.kdk_step_hier(s.box, s.st, s.prm, s.case["bins"], s.eta, s.a0, s.a1, OMEGA_M,
                            bins_out=s.bins, pm_global=s.case["pm_global"])
        return [_particles(s), s.bins]
    if kind == "pm":
        if s.ctx is None:
            dz.pm_force_noalloc(s.box, s.st, s.prm)
        else:
            s.ctx.pm_force(s.box, s.st, s.prm)
        return _force(s)
    if kind == "tree":
        if s.old is not None:
            torch._foreach_copy_([getattr(s.st, k) for k in s.old], list(s.old.values()))
        s.ctx.tree_force(s.box, s.st, s.prm, s.targets)
        return _force(s)
    # the records go to the row of their particle in the run's catalogue
    s.ring.reset()
    s.ctx.lightcone_emit(s.box, s.st, s.prm, s.ring)
    rows = s.ring.buf.view(-1, 8)
    s.table.index_copy_(0, s.ring.buf.view(torch.int32).view(-1, 16)[:, 0].long(), rows)
    return [s.table.view(torch.int32).view(-1, 16)[:, :2], s.table[:, 1:], s.ring.count]


# ---- what a pass cannot do without -----------------------------------------------------------

def _pairs(n, L, ng):
    """Particles inside the cutoff of each particle of a uniform set, over all particles."""
    return n * n * 4.0 / 3.0 * math.pi * (_split(L, ng)[1] / L) ** 3


def _mesh_flops(ng):
    return 2 * 2.5 * ng ** 3 * math.log2(ng ** 3)


def work(case):
    kind = case["kind"]
    if kind == "step":
        n = case["n_side"] ** 3
        return dict(bytes=2.0 * 81 * n,
                    flops=24.0 * _pairs(n, case["L"], case["ng"]) + _mesh_flops(case["ng"]))
    if kind == "coarsen":
        n = case["n_side"] ** 3
        return dict(bytes=(57.0 + 57.0 / 8 + 4.0) * n, flops=14.0 * n)
    if kind == "batch":
        sides = [int(v) for v in case["sides"].split(",")]
        ns = [sides[b % len(sides)] for b in range(case["boxes"])]
        return dict(bytes=2.0 * 81 * sum(v ** 3 for v in ns),
                    flops=sum(24.0 * _pairs(v ** 3, 1.0, 2 * v) + _mesh_flops(2 * v) for v in ns))
    if kind == "hier":
        n = case["n"]
        return dict(bytes=2.0 * 81 * n,
                    flops=24.0 * _pairs(n, case["L"], case["ng"]) + 2 * _mesh_flops(case["ng"]))
    if kind == "pm":
        return dict(bytes=52.0 * case["n"], flops=_mesh_flops(case["ng"]))
    if kind == "tree":
        n, t = case["n"], case["targets"] or case["n"]
        return dict(bytes=28.0 * n + 28.0 * t, flops=24.0 * t / n * _pairs(n, case["L"], 64))
    return dict(bytes=48.0 * case["n"], flops=40.0 * case["n"])


# ---- the same in 64 bits ---------------------------------------------------------------------

def _exact_pm(st, box, ng, r_s):
    n, L = st.n, box.L
    d = L / ng
    m = st.mult[:n].to(torch.float64)
    base, w = [], []
    for k in ("x", "y", "z"):
        u = getattr(st, k)[:n] * (1.0 / d)
        f = torch.floor(u)
        base.append(f.long())
        w.append((1.0 - (u - f), u - f))
    corners = [(a, b, c) for a in (0, 1) for b in (0, 1) for c in (0, 1)]

    def cell(a, b, c):
        return (((base[0] + a) % ng) * ng + (base[1] + b) % ng) * ng + (base[2] + c) % ng

    rho = torch.zeros(ng ** 3, dtype=torch.float64, device=DEV)
    for a, b, c in corners:
        rho.index_add_(0, cell(a, b, c), m * w[0][a] * w[1][b] * w[2][c])
    rho = rho.view(ng, ng, ng) * (box.m0 / d ** 3)
    k1 = torch.fft.fftfreq(ng, 1.0 / ng, device=DEV, dtype=torch.float64) * (2 * math.pi / L)
    k3 = torch.fft.rfftfreq(ng, 1.0 / ng, device=DEV, dtype=torch.float64) * (2 * math.pi / L)

    def green(k):
        return torch.exp(-k * k * r_s * r_s) / torch.sinc(k * d / (2 * math.pi)) ** 4

    k2 = (k1 ** 2)[:, None, None] + (k1 ** 2)[None, :, None] + (k3 ** 2)[None, None, :]
    k2[0, 0, 0] = 1.0
    gk = (-4 * math.pi * box.G) * green(k1)[:, None, None] * green(k1)[None, :, None] * \
        green(k3)[None, None, :] / k2
    gk[0, 0, 0] = 0.0
    phi = torch.fft.irfftn(torch.fft.rfftn(rho) * gk, s=(ng,) * 3)
    out = []
    for ax in range(3):
        g = (2.0 / 3.0) * (torch.roll(phi, -1, ax) - torch.roll(phi, 1, ax)) - \
            (1.0 / 12.0) * (torch.roll(phi, -2, ax) - torch.roll(phi, 2, ax))
        g = g.reshape(-1)
        out.append(-sum(w[0][a] * w[1][b] * w[2][c] * g[cell(a, b, c)]
                        for a, b, c in corners) / d)
    return out


def _exact_short(st, box, r_s, r_cut, targets):
    """The direct sum over every source within the cutoff, target by target."""
    n, L = st.n, box.L
    src = torch.stack([st.x[:n], st.y[:n], st.z[:n]])
    mu = st.mult[:n].to(torch.float64)
    mass, h = box.m0 * mu, 2.8 * box.eps0 * mu ** (1.0 / 3.0)
    out = torch.zeros((3, targets.numel()), dtype=torch.float64, device=DEV)
    step = max(1, 20_000_000 // n)
    for i in range(0, targets.numel(), step):
        t = targets[i:i + step]
        d = src[:, None, :] - src[:, t][:, :, None]
        d = d - L * torch.floor(d / L + 0.5)
        r2 = d.square().sum(0)
        near = (r2 < r_cut * r_cut) & (r2 > 0)
        r = torch.where(near, r2, torch.ones_like(r2)).sqrt()
        hh = torch.maximum(h[None, :], h[t][:, None])
        u = r / hh
        inner = torch.where(u < 0.5, 32.0 / 3.0 + u * u * (32.0 * u - 38.4),
                            64.0 / 3.0 - 48.0 * u + 38.4 * u * u - (32.0 / 3.0) * u ** 3 -
                            1.0 / (15.0 * u ** 3)) / hh ** 3
        v = r / r_s
        f = torch.where(u < 1.0, inner, r ** -3) * near * (box.G * mass)[None, :] * (
            torch.erfc(0.5 * v) + v / math.sqrt(math.pi) * torch.exp(-0.25 * v * v))
        out[:, i:i + step] = (f * d).sum(2)
    return out


def _exact_cone(case, s):
    """Crossings of the shrinking sphere by bisection on the series the call was given."""
    lc, L, n = s.prm, case["L"], s.st.n

    def cheb(c, t):
        b1 = torch.zeros_like(t)
        b2 = torch.zeros_like(t)
        for k in range(lc.n_cheb - 1, 0, -1):
            b1, b2 = 2 * t * b1 - b2 + c[k], b1
        return t * b1 - b2 + c[0]

    x = torch.stack([s.st.x, s.st.y, s.st.z])
    p = torch.stack([s.st.px, s.st.py, s.st.pz])
    xo = torch.tensor(list(lc.x_obs), dtype=torch.float64, device=DEV)[:, None]

    def near(d):
        return d - L * torch.floor(d / L + 0.5)

    d0 = near(x - xo)
    d1 = near(torch.remainder(x + p * lc.D, L) - xo)
    hit = (d0.square().sum(0) < lc.chi2_0) & (d1.square().sum(0) >= lc.chi2_1)
    at = torch.nonzero(hit)[:, 0]
    d0, p = d0[:, at], p[:, at]
    lo, hi = torch.full_like(d0[0], -1.0), torch.full_like(d0[0], 1.0)
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        pos = d0 + p * cheb(lc.cheb_drift, mid)
        inside = pos.square().sum(0) < cheb(lc.cheb_chi, mid).square()
        lo, hi = torch.where(inside, mid, lo), torch.where(inside, hi, mid)
    t = 0.5 * (lo + hi)
    rows = torch.zeros((n + 1, 7), dtype=torch.float64, device=DEV)
    rows[at + 1, 0] = lc.a0 + 0.5 * (t + 1.0) * (lc.a1 - lc.a0)
    rows[at + 1, 1:4] = (d0 + p * cheb(lc.cheb_drift, t)).T
    rows[at + 1, 4:] = p.T
    return [None, rows, None]


def exact(case, seed):
    kind = case["kind"]
    if kind == "pm" and case["n"] <= 2e6 and case["ng"] <= 256:
        s = prepare(case, seed)
        return _exact_pm(s.st, s.box, case["ng"], s.prm.r_s)
    if kind == "tree" and case["n"] * (case["targets"] or case["n"]) <= 6e9 and \
            case["opening"] == "geometric":
        s = prepare(case, seed)
        n = case["n"]
        t = s.targets.long() if s.targets is not None else torch.arange(n, device=DEV)
        g = torch.zeros((3, n), dtype=torch.float64, device=DEV)
        g[:, t] = _exact_short(s.st, s.box, s.prm.r_s, s.prm.r_cut, t)
        return [g[0], g[1], g[2]]
    if kind == "cone":
        return _exact_cone(case, prepare(case, seed))
    # steps, the ensemble and the individual steps: a whole step in 64 bits (its tree force
    # differs from the direct sum by the opening angle's error) takes too long above a few
    # thousand particles; a coarsening's results are decisions and are compared as they are
    if kind == "step" and case["n_side"] <= 24 and not case["merge"] and not case["cone"]:
        s = prepare(case, seed)
        st, sp, L, n = s.st, s.prm, case["L"], s.st.n
        for k in "xyz":
            p = getattr(st, "p" + k)
            p[:n] += getattr(st, "g" + k)[:n] * sp.K1
            v = _wrap(getattr(st, k)[:n] + p[:n] * sp.lc.D, L)
            getattr(st, k)[:n] = v
        cells = [(getattr(st, k)[:n] * (2097152.0 / L)).long() >> 6 for k in "xyz"]
        key = torch.zeros(n, dtype=torch.int64, device=DEV)
        for bit in range(15):
            for d in range(3):
                key |= ((cells[d] >> bit) & 1) << (3 * bit + 2 - d)
        order = torch.sort(key, stable=True)[1]
        for k in ("x", "y", "z", "px", "py", "pz", "mult"):
            getattr(st, k)[:n] = getattr(st, k)[:n][order]
        r_s, r_cut = _split(L, case["ng"])
        g = torch.stack(_exact_pm(st, s.box, case["ng"], r_s))
        g += _exact_short(st, s.box, r_s, r_cut, torch.arange(n, device=DEV))
        out = {k: getattr(st, k)[:n] for k in ("x", "y", "z")}
        for k, v in zip(("px", "py", "pz"), g):
            out[k] = getattr(st, k)[:n] + v * sp.K2
        out.update(mult=None, id=None, type=None, g=[g[0], g[1], g[2]])
        return [out, None, None]
    return None
