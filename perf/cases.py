"""The work a user of this framework has it do, as timed cases.

Every case is one call sequence through the public entry points of
paper_2604_11008_amd.pm on seeded synthetic inputs with the shapes and
statistics of the repository's workloads (gen.CONFIGS): a solenoidal
random-mode velocity field on a periodic box of side 2 pi, particles uniform,
clustered in Gaussian blobs or spread unevenly over the subdomains, log-uniform
relaxation times, and a pool in the cell order that pm_sort leaves, `age` steps
after that sort (particles drift away from the order as they move).

`listed()` names the cases, `draw(rng)` gives more of the same ranges,
`prepare(case, seed)` builds the device state, `run(state)` is one pass,
`exact(case, seed)` the same outputs from plain float64 torch, and
`work(case)` the bytes and operations a pass cannot do without.

A case's fields:
  kind       step (pm_step), noalloc (pm_step_noalloc), staged
             (pm_step_staged), coupled (pm_field_interleave of a new float64
             field to float32, then pm_step in mixed precision on it),
             exchange (pm_classify_scan_pack and pm_compact_append of advanced
             particles), sort (pm_sort), interp (pm_interp), interleave
             (pm_field_interleave)
  n, np, px, py, pz   grid cells per axis, particles, subdomains per axis
  dist       uniform, blobs (70% in Gaussian blobs of sigma two cells) or
             uneven (lognormal numbers per subdomain)
  field      split, ilv (node-interleaved) or mac; mixed: float32 field and
             velocities; halo: one-cell halo; drag: stokes or nonlinear
  step       the time step: half a cell at the largest speed (rule) or at the
             rms speed (rms)
  age        steps since the pool was in cell order; -1: never sorted
  graph      replay pm_step as a HIP graph
"""
import math

import numpy as np
import torch

from paper_2604_11008_amd import gen, pm

L = 2.0 * math.pi
DEV = "cuda"
BLOBS_PER = 16384       # blob particles per blob at the least
MODES = 48              # random Fourier modes of a field
UMAX = 7.0              # no smaller than the largest speed (the field's rms is 1 per component)

BASE = dict(kind="step", n=64, np=65536, px=1, py=1, pz=1, dist="uniform", field="split",
            mixed=False, halo=False, drag="stokes", step="rule", age=10, gravity=False,
            graph=False)


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest workload of the repository (64^3, 65,536 particles in
        # 2x2x2): a test problem or one rank's share of a small run, where
        # launches and latency count
        _case(name="step_small", n=64, np=65536, px=2, py=2, pz=2, age=10),
        # one rank's field with its halo, all 26 neighbours periodic images of
        # the one subdomain, 25 steps after a re-sort: the ordinary step
        _case(name="step_halo_256", n=256, np=4194304, halo=True, gravity=True, age=25),
        # many small subdomains and a large time step: a few percent migrate
        _case(name="step_migrating_256", n=256, np=4194304, px=8, py=8, pz=8, step="rms",
              gravity=True, age=4),
        # clustered particles in float64, the arrays of a solver as they are:
        # the large step that is quoted first
        _case(name="step_blobs_512", n=512, np=1 << 26, px=4, py=4, pz=4, dist="blobs", age=10),
        # the largest: mixed precision on the 1024^3 field of a solver that
        # stores its velocity node-interleaved, clustered particles
        _case(name="step_mixed_ilv_1024", n=1024, np=1 << 27, px=8, py=8, pz=8, dist="blobs",
              field="ilv", mixed=True, age=10),
        # uneven subdomains (ragged segments, some nearly empty) on an
        # interleaved float64 field, long after the last sort
        _case(name="step_uneven_ilv_384", n=384, np=20000003, px=8, py=8, pz=8, dist="uneven",
              field="ilv", age=50),
        # a solver coupled to mixed-precision particles: its new float64 field
        # is rounded and interleaved, then the particles step (odd sizes,
        # nonlinear drag)
        _case(name="coupled_mixed_320", n=320, np=5000001, px=3, py=5, pz=2, field="split",
              mixed=True, drag="nonlinear", age=15, kind="coupled"),
        # the velocity on the faces, as a MAC solver keeps it
        _case(name="step_mac_300", n=300, np=3000017, px=2, py=3, pz=4, field="mac", age=10),
        # migration after each Runge-Kutta stage with the 17-value record, on
        # the per-rank shape of the paper's table at half its side
        _case(name="staged_halo_375", n=375, np=6591797, halo=True, gravity=True, age=10,
              kind="staged"),
        # the exchange alone (scan, pack, compact, append): what the paper
        # measures, at its per-rank number of particles
        _case(name="exchange_750", n=750, np=52734375, gravity=True, age=10, kind="exchange"),
        # the periodic re-sort of a pool that has drifted for 25 steps
        _case(name="sort_256", n=256, np=4194304, px=4, py=4, pz=4, age=25, kind="sort"),
        # velocities at given points (starting a run with V = U(X))
        _case(name="interp_512", n=512, np=8388607, age=0, kind="interp"),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["noalloc", "staged", "coupled", "exchange", "sort", "sort",
                                      "interp", "interleave"])
    n = _spread(rng, 32, 400)
    big = kind in ("step", "exchange", "sort")
    npart = _spread(rng, 4000, 3e7 if big else 6e6)
    age = rng.choice([0, 5, 10, 25, 50, -1])
    dist = rng.choice(["uniform", "blobs", "uneven"])
    if age < 0 and kind != "sort":  # a pool without any order: every stencil on its own
        npart = min(npart, 4000000)
    side = [1, 1, 1] if rng.random() < 0.25 else [rng.randint(1, 8) for _ in range(3)]
    if kind == "noalloc":  # its fixed scratch holds small problems
        npart, dist = min(npart, 300000), "uniform"
        side = [min(p, 3) for p in side]
    side = [max(1, min(p, n // 16)) for p in side]
    one = side == [1, 1, 1]
    field = rng.choice(["split", "split", "ilv", "ilv", "mac"])
    if kind == "staged" and field == "mac":
        field = "split"
    if kind in ("coupled", "interleave"):
        field = "split"
    mixed = kind == "coupled" or rng.random() < 0.4
    return _case(kind=kind, n=n, np=npart, px=side[0], py=side[1], pz=side[2],
                 dist=dist, field=field, mixed=mixed,
                 halo=one and field != "mac" and rng.random() < 0.6,
                 drag=rng.choice(["stokes", "stokes", "nonlinear"]),
                 step="rms" if dist == "uniform" and not one and rng.random() < 0.4 else "rule",
                 age=age, gravity=rng.random() < 0.4,
                 graph=kind == "step" and rng.random() < 0.15)


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _gen(seed, k):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + k) % (1 << 62))


def _modes(case, seed):
    """Wavevectors (3, m), solenoidal amplitudes (3, m) and phases (m): energy
    around wavenumber n / 32, as the repository's fields have it."""
    g = np.random.default_rng([int(seed), 77])
    k0 = max(2.0, case["n"] / 32.0)
    k = []
    while len(k) < MODES:
        v = np.rint(g.normal(0.0, 0.65 * k0, 3))
        if 0 < v @ v <= (case["n"] / 8.0) ** 2:
            k.append(v)
    k = np.array(k).T
    a = g.normal(size=(3, MODES))
    a -= (a * k).sum(0) / (k * k).sum(0) * k
    a /= np.sqrt((a * a).sum(0))
    # sum of m cosines of amplitude s |a|: <|u|^2> = m s^2 / 2 = 3
    return k, a * math.sqrt(6.0 / MODES), g.uniform(0.0, L, MODES)


def _node_phases(case, k, axis, half, dtype=torch.float64):
    n, h = case["n"], int(case["halo"])
    i = (torch.arange(n + 2 * h, device=DEV, dtype=torch.float64) - h) % n
    x = (i + half) * (L / n)
    return torch.outer(x, torch.from_numpy(k[axis]).to(DEV)).to(dtype)


def _component(case, modes, c, dtype, out=None):
    """Component c at the stored nodes, (nz*ny*nx) values, written into `out`."""
    k, a, ph = modes
    st = case["n"] + 2 * int(case["halo"])
    off = [0.0 if case["field"] == "mac" and c == ax else 0.5 for ax in range(3)]
    px, py, pz = (_node_phases(case, k, ax, off[ax]) for ax in range(3))
    amp = torch.from_numpy(a[c]).to(DEV)
    ex = torch.cat([torch.cos(px).T, torch.sin(px).T]).contiguous()     # (2m, nx)
    if out is None:
        out = torch.empty(st * st * st, dtype=dtype, device=DEV)
    view = out.view(st, st * st)
    slab = max(1, (1 << 18) // st)
    for z in range(0, st, slab):
        th = pz[z:z + slab, None] + py[None] + torch.from_numpy(ph).to(DEV)
        th = th.reshape(-1, MODES)
        lhs = torch.cat([amp * torch.cos(th), -amp * torch.sin(th)], dim=1)
        view[z:z + slab] = (lhs @ ex).view(-1, st * st).to(dtype)
    return out


def _velocity_at(modes, X):
    """The modes summed at positions X (3, m), for starting velocities."""
    k, a, ph = (torch.from_numpy(t).to(DEV) for t in modes)
    U = torch.zeros_like(X)
    for j in range(0, X.shape[1], 1 << 20):
        th = (X[:, j:j + (1 << 20)].T.float() @ k.float()) + ph.float()
        U[:, j:j + (1 << 20)] = (a.float() @ torch.cos(th).T).double()
    return U


def _positions(case, seed):
    g, n, m = _gen(seed, 1), case["n"], case["np"]
    rnd = lambda *s: torch.rand(*s, generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
    if case["dist"] == "uniform":
        X = rnd(3, m) * L
    elif case["dist"] == "blobs":
        nb = int(0.7 * m)
        blobs = max(1, min(4096, nb // BLOBS_PER))
        X = rnd(3, m) * L
        for c in range(3):
            X[c, :nb] = torch.randn(nb, generator=g, device=DEV, dtype=torch.float64)
        pick = torch.randint(blobs, (nb,), generator=g, device=DEV)
        X[:, :nb] = X[:, :nb] * (2.0 * L / n) + (rnd(3, blobs) * L)[:, pick]
    else:
        p = [case["px"], case["py"], case["pz"]]
        ns = p[0] * p[1] * p[2]
        w = torch.exp(torch.randn(ns, generator=g, device=DEV, dtype=torch.float64))
        cdf = torch.cumsum(w / w.sum(), 0)
        s = torch.searchsorted(cdf, rnd(m)).clamp_(max=ns - 1)
        X = rnd(3, m)
        for c, q in enumerate((s % p[0], (s // p[0]) % p[1], s // (p[0] * p[1]))):
            X[c] = (X[c] + q) * (L / p[c])
    return _into_box(X)


def _into_box(X):
    X = torch.remainder(X, L)
    return torch.where(X >= L, torch.full_like(X, np.nextafter(L, 0.0)), X)


def _dt(case):
    cell = L / case["n"]
    return 0.5 * cell if case["step"] == "rms" else \
        0.5 * cell / (UMAX + (1.0 if case["gravity"] else 0.0))


def _gravity(case):
    return (0.0, 0.0, -1.0) if case["gravity"] else (0.0, 0.0, 0.0)


def _params(case):
    return pm.Params(_dt(case), _gravity(case), drag=case["drag"])


def _decomp(case):
    p = (case["px"], case["py"], case["pz"])
    return p, gen.bounds(p, L)


def _owner(X, bnds, p):
    idx = [(torch.searchsorted(torch.from_numpy(bnds[a]).to(DEV), X[a].contiguous(), right=True) - 1)
           .clamp_(0, p[a] - 1) for a in range(3)]
    return idx[0] + p[0] * (idx[1] + p[1] * idx[2])


def _cell_key(case, X):
    n = case["n"]
    return gen.cell_key(*[torch.floor(X[a] * (n / L)).to(torch.int64).clamp_(0, n - 1)
                          for a in range(3)])


class _State:
    pass


def _records(case, seed):
    """Positions, velocities, tau and ids in pool order with their owners, the
    order that of the cells the particles were in `age` steps ago."""
    modes = _modes(case, seed)
    g = _gen(seed, 2)
    m = case["np"]
    X = _positions(case, seed)
    V = _velocity_at(modes, X)
    tau = torch.exp(math.log(0.01) + math.log(100.0) *
                    torch.rand(m, generator=g, device=DEV, dtype=torch.float64))
    # particles lag behind the flow, more so the slower they respond
    for c in range(3):
        V[c] += 0.25 * torch.sqrt(tau) * torch.randn(m, generator=g, device=DEV,
                                                     dtype=torch.float64)
    vd = torch.float32 if case["mixed"] else torch.float64
    V, tau = V.to(vd), tau.to(vd)
    p, bnds = _decomp(case)
    own = _owner(X, bnds, p)
    bits = 3 * int(case["n"] - 1).bit_length() + 1
    if case["age"] < 0:
        key = torch.randint(1 << 30, (m,), generator=g, device=DEV)
        bits = 30
    else:
        key = _cell_key(case, _into_box(X - (case["age"] * _dt(case)) * V.double()))
    perm = torch.sort(key + (own << bits), stable=True).indices
    del key
    return X[:, perm], V[:, perm], tau[perm], perm, own[perm], modes


def _pool(case, rec):
    """The records in segments with room for growth; the host layout beside."""
    X, V, tau, ids, own, _ = rec
    p, _ = _decomp(case)
    nsub = p[0] * p[1] * p[2]
    count = torch.bincount(own, minlength=nsub)
    counts = count.cpu().numpy()
    uneven = case["dist"] == "uneven"
    slack, extra = (0.25, 4096) if nsub > 1 else (0.05, 1024)
    base, cap = gen.layout(counts, slack=slack, extra=extra, p=p if uneven else None)
    # arrays of one size whatever the seed: the most such a layout can take
    size = int(case["np"] * (1.0 + slack + (1.3 if uneven else 0.0))) + nsub * (extra + 64)
    at = torch.arange(case["np"], device=DEV)
    first = torch.from_numpy(np.cumsum(counts) - counts).to(DEV)
    at += (torch.from_numpy(base).to(DEV) - first)[own]
    pool = pm.DevicePool.empty(base, cap, vdtype=V.dtype, device=DEV, size=size)
    for c in range(3):
        pool.x[c, at] = X[c]
        pool.v[c, at] = V[c]
    pool.tau[at] = tau
    pool.id[at] = ids
    pool.count.copy_(count)
    return pool, base, cap, counts


def _send_layout(case, counts):
    roomy = case["step"] == "rms" or (case["np"] < 8000000 and case["kind"] != "noalloc")
    f = (0.2, 0.05, 0.03) if roomy else (0.05, 0.01, 0.005)
    base, cap = gen.send_layout(counts, *f)
    return base, cap, int(case["np"] * (6 * f[0] + 12 * f[1] + 8 * f[2])) + 26 * 256 * len(counts)


def _field(case, modes, dtype):
    n = case["n"]
    if case["field"] == "ilv":
        st = (n + 2 * int(case["halo"])) ** 3
        u = torch.empty((st, 3), dtype=dtype, device=DEV)
        tmp = torch.empty(st, dtype=dtype, device=DEV)
        for c in range(3):
            u[:, c] = _component(case, modes, c, dtype, tmp)
        return pm.DeviceField(u, n, int(case["halo"]), L, device=DEV, interleaved=True)
    u = [_component(case, modes, c, dtype) for c in range(3)]
    return pm.DeviceField(u, n, int(case["halo"]), L, device=DEV, stagger=case["field"] == "mac")


def _outs(*pools, **more):
    """The arrays of the pools a call wrote (their unused room keeps its zeros)."""
    d = dict(more)
    for i, q in enumerate(pools):
        for name in ("x", "v", "tau", "id", "count", "xs", "vs", "a"):
            if getattr(q, name, None) is not None:
                d["%d_%s" % (i, name)] = getattr(q, name)
    return d


def prepare(case, seed):
    s = _State()
    kind = case["kind"]
    s.kind = kind
    ft = torch.float32 if case["mixed"] and kind not in ("coupled", "interleave") else torch.float64
    if kind == "interleave":
        s.field = _field(case, _modes(case, seed), torch.float64)
        s.to = torch.float32 if case["mixed"] else torch.float64
        s.out = torch.empty((s.field.u[0].numel(), 3), dtype=s.to, device=DEV)
        return s
    rec = _records(case, seed)
    if kind == "interp":
        s.field = _field(case, rec[5], ft)
        s.X = rec[0].contiguous()
        s.ctx = pm.Context(1, 1, 1, device=DEV)
        return s
    if kind != "exchange":
        s.field = _field(case, rec[5], ft)
    else:  # the particles have just moved: some are outside their owner's box
        X = rec[0] + _dt(case) * rec[1].double()
        rec = (X,) + rec[1:]
    s.pin, base, cap, counts = _pool(case, rec)
    del rec
    p, bnds = _decomp(case)
    s.dc = pm.Decomp(p, bnds)
    vd = s.pin.v.dtype
    sb, sc, ssize = _send_layout(case, counts)
    s.send = pm.DevicePool.empty(sb, sc, vdtype=vd, device=DEV, size=ssize)
    s.pout = pm.DevicePool.empty(base, cap, vdtype=vd, device=DEV, size=s.pin.size)
    s.params = _params(case)
    s.outs = _outs(s.pout, s.send)
    if kind == "noalloc":
        s.flags = torch.zeros(1, dtype=torch.int32, device=DEV)
        return s
    s.ctx = pm.Context(s.pin.size, s.send.size, s.dc.nsub, device=DEV)
    if case["graph"]:
        s.ctx.set_graph(True)
    if kind == "staged":
        s.mid = pm.DeviceStagePool.empty(base, cap, vdtype=vd, device=DEV, size=s.pin.size)
        s.mid_send = pm.DeviceStagePool.empty(sb, sc, vdtype=vd, device=DEV, size=ssize)
        s.outs = _outs(s.pout, s.send, s.mid, s.mid_send)
    elif kind == "coupled":
        s.ilv = torch.empty((s.field.u[0].numel(), 3), dtype=torch.float32, device=DEV)
        s.outs = _outs(s.pout, s.send, field=s.ilv)
    elif kind == "sort":
        s.outs = _outs(s.pout)
    return s


def run(s):
    if s.kind == "step":
        s.ctx.step(s.field, s.dc, s.pin, s.pout, s.send, s.params)
    elif s.kind == "noalloc":
        pm.step_noalloc(s.field, s.dc, s.pin, s.pout, s.send, s.params, s.flags)
    elif s.kind == "staged":
        s.ctx.step_staged(s.field, s.dc, s.pin, s.mid, s.mid_send, s.pout, s.send, s.params)
    elif s.kind == "coupled":
        f = pm.interleave_field(s.field, out=s.ilv, dtype=torch.float32)
        s.ctx.step(f, s.dc, s.pin, s.pout, s.send, s.params)
    elif s.kind == "exchange":
        s.ctx.classify_scan_pack(s.dc, s.pin, s.send)
        s.ctx.compact_append(s.dc, s.pin, s.send, s.pout)
    elif s.kind == "sort":
        s.ctx.sort(s.field, s.pin, s.pout)
    elif s.kind == "interp":
        return s.ctx.interp(s.field, s.X)
    else:
        pm.interleave_field(s.field, out=s.out, dtype=s.to)
        return s.out
    return s.outs


# ----------------------------------------------------------------------------
# the same outputs from plain float64 torch
# ----------------------------------------------------------------------------

def _value(f, comp, idx):
    return (f.u[0].view(-1, 3)[idx, comp] if f.interleaved else f.u[comp][idx]).double()


def _interp64(f, X):
    n, h = f.n[0], f.halo
    st = n + 2 * h
    U = torch.empty_like(X)
    for j in range(0, X.shape[1], 1 << 22):
        Y = X[:, j:j + (1 << 22)]
        for c in range(3):
            lo, fr = [], []
            for a in range(3):
                t = Y[a] * (n / L) - (0.0 if f.stagger and a == c else 0.5)
                k = torch.floor(t)
                fr.append(t - k)
                lo.append(k.to(torch.int64))
            acc = 0.0
            for q in range(8):
                o = (q & 1, q >> 1 & 1, q >> 2)
                i = [lo[a] + o[a] + 1 if h else (lo[a] + o[a]) % n for a in range(3)]
                w = 1.0
                for a in range(3):
                    w = w * (fr[a] if o[a] else 1.0 - fr[a])
                acc = acc + w * _value(f, c, i[0] + st * (i[1] + st * i[2]))
            U[c, j:j + (1 << 22)] = acc
    return U


def _accel64(case, par, U, V, tau):
    s = U - V
    if case["drag"] == "nonlinear":
        r = torch.sqrt(4.5 * tau * par.nu / par.density_ratio)
        re = 2.0 * r * torch.sqrt((s * s).sum(0)) / par.nu
        s = s * (1.0 + 0.15 * re ** 0.687)
    return s / tau + torch.tensor(par.g, dtype=torch.float64, device=DEV)[:, None]


def _migrate64(case, own, test, move, plain, base, sbase):
    """Where every record goes: the stayers of each segment in order, then what
    it receives by direction.  `test`: positions that decide; `move`: arrays
    shifted into the receiver's image like them (`plain`: without the clamp at
    the box side).  Returns places in out, counts, leavers and their places."""
    p, bnds = _decomp(case)
    k = (own % p[0], (own // p[0]) % p[1], own // (p[0] * p[1]))
    d = torch.zeros_like(own)
    to = []
    for a in range(3):
        b = torch.from_numpy(bnds[a]).to(DEV)
        o = (test[a] >= b[k[a] + 1]).long() - (test[a] < b[k[a]]).long()
        d += (o + 1) * 3 ** a
        up, down = (o > 0) & (k[a] == p[a] - 1), (o < 0) & (k[a] == 0)
        shift = down.double() * L - up.double() * L
        for t in move + plain:
            t[a] += shift
        for t in move:
            t[a] = torch.where(down & (t[a] >= L), torch.full_like(t[a], np.nextafter(L, 0.0)), t[a])
        to.append((k[a] + o) % p[a])
    dest = to[0] + p[0] * (to[1] + p[1] * to[2])
    stay = d == 13
    order = torch.sort(dest * 28 + torch.where(stay, torch.zeros_like(d), d + 1), stable=True).indices
    nsub = p[0] * p[1] * p[2]
    count = torch.bincount(dest, minlength=nsub)
    at = torch.empty_like(order)
    at[order] = torch.arange(len(order), device=DEV)
    at += (torch.from_numpy(base).to(DEV) - (torch.cumsum(count, 0) - count))[dest]
    gone = torch.nonzero(~stay).squeeze(1)
    q = own[gone] * 27 + d[gone]
    scount = torch.bincount(q, minlength=nsub * 27)
    so = torch.sort(q, stable=True).indices
    sat = torch.empty_like(so)
    sat[so] = torch.arange(len(so), device=DEV)
    sat += (torch.from_numpy(sbase).to(DEV) - (torch.cumsum(scount, 0) - scount))[q]
    return at, count, gone, sat, scount, dest


def _place(d, i, size, ssize, recs, ids, where):
    """Outputs `i` (pool) and `i + 1` (send buffers) of a migration."""
    at, count, gone, sat, scount, _ = where
    for name, v in recs.items():
        full = torch.zeros(v.shape[:-1] + (size,), dtype=torch.float64, device=DEV)
        full[..., at] = v
        d["%d_%s" % (i, name)] = full
        full = torch.zeros(v.shape[:-1] + (ssize,), dtype=torch.float64, device=DEV)
        full[..., sat] = v[..., gone]
        d["%d_%s" % (i + 1, name)] = full
    for k, m, to, src in ((i, size, at, ids), (i + 1, ssize, sat, ids[gone])):
        full = torch.zeros(m, dtype=torch.int64, device=DEV)
        full[to] = src
        d["%d_id" % k] = full
    d["%d_count" % i], d["%d_count" % (i + 1)] = count, scount


def exact(case, seed):
    kind = case["kind"]
    modes = _modes(case, seed)
    if kind == "interleave":
        u = torch.empty(((case["n"] + 2 * int(case["halo"])) ** 3, 3), dtype=torch.float64, device=DEV)
        for c in range(3):
            u[:, c] = _component(case, modes, c, torch.float64)
        return u
    X, V, tau, ids, own, _ = rec = _records(case, seed)
    if kind == "interp":
        return _interp64(_field(case, modes, torch.float32 if case["mixed"] else torch.float64), X)
    if kind == "exchange":
        X = X + _dt(case) * V.double()
        rec = (X,) + rec[1:]
    _, bnds = _decomp(case)
    pool, base, cap, counts = _pool(case, rec)
    size = pool.size
    del pool, rec
    V, tau = V.double(), tau.double()
    if kind == "sort":
        key = _cell_key(case, X)
        perm = torch.sort(key + (own << 40), stable=True).indices
        at = torch.arange(case["np"], device=DEV)
        at += torch.from_numpy(base - (np.cumsum(counts) - counts)).to(DEV)[own]
        d = {"0_count": torch.from_numpy(counts).to(DEV)}
        for name, v in (("x", X), ("v", V), ("tau", tau)):
            full = torch.zeros(v.shape[:-1] + (size,), dtype=torch.float64, device=DEV)
            full[..., at] = v[..., perm]
            d["0_" + name] = full
        d["0_id"] = torch.zeros(size, dtype=torch.int64, device=DEV)
        d["0_id"][at] = ids[perm]
        return d
    sb, _, ssize = _send_layout(case, counts)
    d = {}
    if kind == "exchange":
        where = _migrate64(case, own, X.clone(), [X], [], base, sb)
        _place(d, 0, size, ssize, {"x": X, "v": V, "tau": tau}, ids, where)
        return d
    par, h = _params(case), _dt(case)
    f = _field(case, modes, torch.float32 if case["mixed"] and kind != "coupled" else torch.float64)
    if kind == "coupled":
        d["field"] = torch.stack(f.u, dim=1)
        f.u = [u.float() for u in f.u]
    A1 = _accel64(case, par, _interp64(f, X), V, tau)
    Xs, Vs = X + h * V, V + h * A1
    if kind == "staged":
        where = _migrate64(case, own, Xs.clone(), [Xs], [X], base, sb)
        _place(d, 2, size, ssize, {"x": X, "v": V, "xs": Xs, "vs": Vs, "a": A1, "tau": tau}, ids, where)
        # the mid-step pool's order is the order stage 2 works in
        order = torch.argsort(where[0])
        X, V, Xs, Vs, A1, tau = (t[..., order] for t in (X, V, Xs, Vs, A1, tau))
        ids, own = ids[order], where[5][order]
    A2 = _accel64(case, par, _interp64(f, Xs), Vs, tau)
    X = X + 0.5 * h * (V + Vs)
    V = V + 0.5 * h * (A1 + A2)
    del f, A1, A2, Xs, Vs
    where = _migrate64(case, own, X.clone(), [X], [], base, sb)
    _place(d, 0, size, ssize, {"x": X, "v": V, "tau": tau}, ids, where)
    return d


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _touched(case, stages=1):
    """Field nodes the stencils read, expected: a node is read if one of the
    cells around it holds a particle (clustered particles: their uniform share
    and the cells of the blobs)."""
    nodes = float(case["n"]) ** 3
    rho = case["np"] / nodes
    if case["dist"] == "blobs":
        nb = 0.7 * case["np"]
        blob = max(1, min(4096, int(nb) // BLOBS_PER)) * 1500.0
        return min(nodes, nodes * -math.expm1(-8.0 * 0.3 * rho) + min(blob, 8 * nb))
    return nodes * -math.expm1(-8.0 * rho)


def work(case):
    m, kind = case["np"], case["kind"]
    fs = 4 if case["mixed"] else 8
    rec = 32 + 4 * fs
    nodes = (case["n"] + 2.0 * int(case["halo"])) ** 3
    stencil = 2 * 3 * 7 * 2
    heun = 2 * stencil + 60 + (80 if case["drag"] == "nonlinear" else 0)
    if kind == "interleave":
        return {"bytes": nodes * 3 * (8 + fs), "flops": 0.0}
    if kind == "interp":
        return {"bytes": m * (24.0 + 3 * fs) + _touched(case) * 3 * fs, "flops": m * float(stencil)}
    if kind in ("exchange", "sort"):
        return {"bytes": 2.0 * rec * m, "flops": 12.0 * m}
    field = nodes * 3 * (8 + 4) if kind == "coupled" else 0.0
    if kind == "staged":  # the mid-step pool is an output of its own
        mid = 8 * 7 + 10 * fs
        return {"bytes": 2.0 * (rec + mid) * m + 2 * _touched(case) * 3 * fs, "flops": float(heun) * m}
    return {"bytes": 2.0 * rec * m + _touched(case) * 3 * fs + field, "flops": float(heun) * m}
