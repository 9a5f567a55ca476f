"""What is timed: the work that a program has this library do, through
`paper_1204_5849_amd.sim.Simulation` and the binding, over the sizes, schemes,
precisions and call forms it offers.

A case is a block tree (a problem, its base blocks and its levels), the scheme
parameters, and one call on the state: `graph` and `advance` are whole cycles
of the main loop, `output` is what a program does when it writes a snapshot or
looks at the solution, `regrid` moves the state onto the tree the estimator
asks for.  `exact` is the method once more, in plain torch in 64 bits on
padded tiles, as formulas over whole arrays.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1204_5849_amd import native as N
from paper_1204_5849_amd import workloads as W
from paper_1204_5849_amd.sim import Simulation

NB, NG, NV = 16, 2, 9
RHO, MX, BX, EN, PSI = 0, 1, 4, 7, 8
CRITERIA = [("var", RHO, 1e-12), ("bmag", 0, 0.1)]

DEFAULT = dict(problem="ot", nx=8, ny=8, nz=1, levels=1, nsims=1, kmax=32, precision="fp64",
               scheme="lf", limiter="minmod", riemann="rusanov", cond="off", eta=0.0,
               call="graph", steps=2, tuned=True)


def _case(name=None, **kw):
    c = dict(DEFAULT, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a program that steps a 64^2 vortex itself and
        # looks at the records after every step (eager, default launches)
        _case("vortex64_step", nx=4, ny=4, call="advance", steps=1, tuned=False),
        # the paper's 2-D test at its own size, cycles replayed as graphs
        _case("vortex128_lf", steps=10),
        # the same vortex on a static AMR tree of about 2000 leaves, modified
        # MacCormack and van Leer
        _case("vortex_amr_mmc", problem="ot_amr", nx=16, ny=16, levels=3, scheme="mmc",
              limiter="vanleer", steps=4),
        # 64 independent Kelvin-Helmholtz runs of uneven sizes in one context
        _case("kh64_lf", problem="kh", nsims=64, precision="fp32", steps=4),
        # a 3-D blast with one refined sphere, the ordinary 3-D size
        _case("blast128_lf", problem="blast", nx=8, ny=8, nz=8, levels=2, precision="fp32"),
        # modified MacCormack on 3-D blocks
        _case("blast64_mmc", problem="blast", nx=4, ny=4, nz=4, levels=2, scheme="mmc"),
        # the resistive current sheet: FP64 state
        _case("sheet64_lf64", problem="harris", nx=4, ny=4, nz=4, levels=4, eta=1e-3),
        # third-order WENO with the HLLC flux
        _case("sheet64_weno_hllc", problem="harris", nx=4, ny=4, nz=4, levels=4, eta=1e-3,
              precision="fp32", scheme="weno", riemann="hllc"),
        # with the conduction subcycle along the field
        _case("sheet64_cond", problem="harris", nx=4, ny=4, nz=4, levels=4, eta=1e-3,
              precision="fp32", cond="field"),
        # a snapshot of the large sheet: complete ghost frames, conserved
        # totals and the per-block estimate
        _case("sheet128_output", problem="harris", nx=8, ny=8, nz=8, levels=4, eta=1e-3,
              precision="fp32", call="output", steps=1),
        # one regrid of the blast: estimate, tree edit (a third level at the
        # shell, the quiet outer blocks dropped), new plan, state moved
        _case("blast128_regrid", problem="blast", nx=8, ny=8, nz=8, levels=2, precision="fp32",
              call="regrid", steps=1),
        # the largest: 22016 blocks, 79.2 M leaf cells
        _case("sheet128_lf", problem="harris", nx=8, ny=8, nz=8, levels=4, eta=1e-3,
              precision="fp32", steps=4),
    ]


def _cost(c):
    """Rough work of a case in FP32 LF cell-updates of a 3-D block."""
    keys, leaf = _tree(c["problem"], c["nx"], c["ny"], c["nz"], c["levels"], c["nsims"], c["kmax"])
    f = 2.4 if c["precision"] == "fp64" else 1.0
    f *= {"lf": 1.0, "weno": 3.0, "mmc": 4.0}[c["scheme"]]
    f *= 3.0 if c["cond"] != "off" else 1.0
    return float(leaf.sum()) * NB ** _ndim(c) * f * c["steps"]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    top = 2.9e8
    while True:
        prob = rng.choice(["ot", "ot", "ot_amr", "kh", "blast", "harris", "harris"])
        c = dict(problem=prob, precision=rng.choice(["fp32", "fp64"]),
                 scheme=rng.choice(["lf", "lf", "weno", "mmc"]),
                 limiter=rng.choice(["minmod", "minmod", "vanleer"]),
                 call=rng.choice(["graph"] * 6 + ["advance"] * 2 + ["output", "regrid"]),
                 steps=rng.randint(1, 6), tuned=rng.random() < 0.7)
        c["riemann"] = "rusanov" if c["scheme"] == "mmc" else rng.choice(["rusanov", "rusanov", "hllc"])
        c["cond"] = rng.choice(["off", "off", "off", "off", "iso", "field"])
        if prob == "ot":
            c.update(nx=log(2, 48), ny=log(2, 48), eta=rng.choice([0.0, 1e-3]))
        elif prob == "ot_amr":
            c.update(nx=rng.randint(7, 20), ny=rng.randint(7, 20), levels=rng.choice([2, 3]))
        elif prob == "kh":
            c.update(nsims=log(2, 64), kmax=rng.randint(5, 32))
        elif prob == "blast":
            n = log(2, 8)
            c.update(nx=n, ny=n, nz=rng.choice([n, max(2, n - 1)]), levels=rng.choice([1, 2]))
        else:
            n = rng.randint(2, 7)
            c.update(nx=n, ny=n, nz=n, levels=rng.choice([2, 3, 4]), eta=rng.choice([0.0, 1e-3]))
        if c["call"] in ("output", "regrid"):
            c["steps"] = 1
        c = _case(**c)
        if _cost(c) <= top:
            return c


# ---------------------------------------------------------------- trees and inputs
def _ndim(c):
    return 3 if c["problem"] in ("blast", "harris") else 2


def _sims(problem, nx, ny, nz, nsims, kmax):
    per, out = ("periodic", "periodic"), ("outflow", "outflow")
    if problem == "kh":
        ks, _ = W.kh_sizes(nsims, 1204, 4, kmax)
        return [W.SimDesc((0.0, -0.5, 0.0), (1.0, 0.5, 1.0), (k, k, 1), (per, out, per)) for k in ks]
    if problem == "blast":
        return [W.SimDesc((-0.5,) * 3, (0.5,) * 3, (nx, ny, nz), (per,) * 3)]
    if problem == "harris":
        return [W.SimDesc((-2.0,) * 3, (2.0,) * 3, (nx, ny, nz), (per, out, per))]
    return [W.SimDesc((0.0, 0.0, 0.0), (1.0, 1.0, 1.0), (nx, ny, 1), (per,) * 3)]


@functools.lru_cache(maxsize=32)
def _tree(problem, nx, ny, nz, levels, nsims, kmax):
    """Block keys [n, 5] and which of them are leaves."""
    sims = _sims(problem, nx, ny, nz, nsims, kmax)
    ndim = 3 if problem in ("blast", "harris") else 2

    def pred(si, lv, lo, hi):
        if problem == "harris":  # the sheet: |y| < 0.5 / 2^(l-1)
            lim = 0.5 / (1 << (lv - 1))
            return lo[1] < lim and hi[1] > -lim
        near = [min(max(0.5 if problem == "ot_amr" else 0.0, a), b) for a, b in zip(lo, hi)]
        if problem == "ot_amr":  # a disc of the vortex, tighter with the level
            return math.hypot(near[0] - 0.5, near[1] - 0.5) <= 0.6 / lv
        return sum(v * v for v in near) <= 0.09  # the blast's sphere

    keys = W.refine_geometric(sims, ndim, levels, pred)
    up = keys[keys[:, 1] > 1].copy()
    up[:, 1] -= 1
    up[:, 2:] >>= 1
    parents = set(map(tuple, np.unique(up, axis=0).tolist()))
    leaf = np.array([tuple(k) not in parents for k in keys.tolist()], dtype=bool)
    return keys, leaf


def _workload(c):
    keys, _ = _tree(c["problem"], c["nx"], c["ny"], c["nz"], c["levels"], c["nsims"], c["kmax"])
    three = _ndim(c) == 3
    return W.Workload(name=c["problem"], ndim=_ndim(c),
                      sims=_sims(c["problem"], c["nx"], c["ny"], c["nz"], c["nsims"], c["kmax"]),
                      keys=keys, ic=None, scheme=c["scheme"], limiter=c["limiter"],
                      riemann=c["riemann"], cond=c["cond"], cond_max_sub=8,
                      kappa0=0.4 if c["problem"] == "harris" else 0.01, kappa_exp=2.5,
                      glm_mode="fastspeed" if three else "paper", eta=c["eta"],
                      precision=c["precision"])


def _primitives(c, wl, rows, seed, dev):
    """rho, v, B, p, psi at the cell centres of the blocks `rows` of wl.keys,
    [n, 9, nz, 16, 16] in 64 bits: the problem's own fields with amplitudes,
    phases and noise of the seed."""
    k = torch.from_numpy(np.ascontiguousarray(wl.keys[rows]).astype(np.int64)).to(dev)
    lo = torch.tensor([s.lo for s in wl.sims], dtype=torch.float64, device=dev)[k[:, 0]]
    hi = torch.tensor([s.hi for s in wl.sims], dtype=torch.float64, device=dev)[k[:, 0]]
    nb = torch.tensor([list(s.nbase) for s in wl.sims], dtype=torch.float64, device=dev)[k[:, 0]]
    n = len(rows)
    nz = NB if wl.ndim == 3 else 1
    i = torch.arange(NB, dtype=torch.float64, device=dev)
    xyz = []
    for d in range(3):
        w = (hi[:, d] - lo[:, d]) / (nb[:, d] * 2.0 ** (k[:, 1] - 1).to(torch.float64) * NB)
        x = lo[:, d, None] + (k[:, 2 + d, None] * NB + i + 0.5) * w[:, None]
        if d == 2 and wl.ndim == 2:
            x = torch.zeros((n, 1), dtype=torch.float64, device=dev)
        shape = [n, 1, 1, 1]
        shape[3 - d] = x.shape[1]
        xyz.append(x.view(shape).expand(n, nz, NB, NB))
    x, y, z = xyz
    r = np.random.default_rng([int(seed), 1204])
    f = torch.empty((n, NV, nz, NB, NB), dtype=torch.float64, device=dev)
    f.zero_()
    tp = 2.0 * math.pi
    if c["problem"] in ("ot", "ot_amr"):
        a, p1, p2 = 1.0 + 0.1 * r.random(), tp * r.random(), tp * r.random()
        s4 = 1.0 / math.sqrt(4.0 * math.pi)
        f[:, 0] = 25.0 / (36.0 * math.pi)
        f[:, 1] = -a * torch.sin(tp * y + p1)
        f[:, 2] = a * torch.sin(tp * x + p2)
        f[:, 3] = 0.1 * torch.sin(tp * (x + y))
        f[:, 4] = -s4 * torch.sin(tp * y + p1)
        f[:, 5] = s4 * torch.sin(2.0 * tp * x + p2)
        f[:, 6] = 0.05 * torch.cos(tp * x)
        f[:, 7] = 5.0 / (12.0 * math.pi)
    elif c["problem"] == "kh":
        m = torch.from_numpy(1.0 + r.integers(0, 4, len(wl.sims))).to(dev)[k[:, 0]].view(n, 1, 1, 1)
        ph = torch.from_numpy(tp * r.random(len(wl.sims))).to(dev)[k[:, 0]].view(n, 1, 1, 1)
        f[:, 0] = 1.0
        f[:, 1] = 0.5 * torch.tanh(y / 0.05)
        f[:, 2] = 0.01 * torch.sin(tp * m * x + ph)
        f[:, 4] = 0.1
        f[:, 7] = 1.0
    elif c["problem"] == "blast":
        th, pin = tp * r.random(), 10.0 * (1.0 + r.random())
        core = x * x + y * y + z * z < 0.01
        f[:, 0] = torch.where(core, 2.0 + r.random(), 1.0)
        f[:, 4] = math.cos(th) * 0.7
        f[:, 5] = math.sin(th) * 0.7
        f[:, 6] = 0.1
        f[:, 7] = torch.where(core, pin, 0.5)
    else:
        g = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + int(rows[0]))
        s = 1.0 / torch.cosh(y / 0.5) ** 2
        f[:, 0] = 1.0 + s
        f[:, 1:4] = 1e-3 * (2.0 * torch.rand((n, 3, nz, NB, NB), generator=g, dtype=torch.float64,
                                            device=dev) - 1.0)
        f[:, 2] += 0.02 * torch.sin(math.pi * x + tp * r.random()) * s
        f[:, 4] = torch.tanh(y / 0.5)
        f[:, 7] = 0.1 + 0.5 * s
    return f


CHUNK = 1024


def _chunks(rows):
    return [rows[i:i + CHUNK] for i in range(0, len(rows), CHUNK)]


# one stream for every state, as one program has
_STREAM = []


def prepare(case, seed):
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    wl = _workload(c)
    dev = torch.device("cuda:0")
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream(device=dev))
    sim = Simulation(wl, device=dev, stream=_STREAM[0])
    _, leaf = _tree(c["problem"], c["nx"], c["ny"], c["nz"], c["levels"], c["nsims"], c["kmax"])
    inside = sim.interior_view()
    with torch.cuda.stream(sim.stream):
        for rows in _chunks(np.nonzero(leaf)[0]):
            at = torch.from_numpy(sim.slot_of_key[rows].astype(np.int64)).to(dev)
            inside[at] = _primitives(c, wl, rows, seed, dev).to(sim.dtype)
    sim.stream.synchronize()
    N.map_prim_to_cons(sim.ctx, sim.U, sim.sp)
    N.map_restrict(sim.ctx, sim.U, sim.sp)
    N.map_fill_ghosts(sim.ctx, sim.U, sim.sp)
    if c["tuned"] and c["call"] in ("graph", "advance"):
        sim.autotune()
    sim.sync()
    return {"sim": sim, "case": c}


def _records(sim):
    return {"dt": sim.dt[:, :5], "nsub": sim.dt.view(torch.int32)[:, 10]}


def run(state):
    sim, c = state["sim"], state["case"]
    if c["call"] == "graph":
        sim.graph_run(c["steps"])
    elif c["call"] == "advance":
        sim.advance(c["steps"])
    elif c["call"] == "output":
        sim.fill()
        return {"U": sim.U, "totals": sim.totals(), "err": sim.estimate(CRITERIA)}
    else:
        new = sim.regrid(CRITERIA, 0.3, 0.1, c["levels"] + (c["problem"] == "blast"))
        new.sync()
        return {"U": new.interior_view(), "keys": new.wl.keys}
    # same-level ghosts hold unspecified values after a cycle: the interiors
    return {"U": sim.interior_view(), **_records(sim)}


def work(case):
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    keys, leaf = _tree(c["problem"], c["nx"], c["ny"], c["nz"], c["levels"], c["nsims"], c["kmax"])
    nd, w = _ndim(c), 8 if c["precision"] == "fp64" else 4
    cells = float(leaf.sum()) * NB ** nd
    if c["call"] == "output":  # every ghost cell written, every interior read
        tile = (NB + 2 * NG) ** nd
        return {"bytes": len(keys) * NV * w * tile, "flops": cells * 60.0}
    if c["call"] == "regrid":
        return {"bytes": 2 * len(keys) * NV * w * (NB + 2 * NG) ** nd, "flops": cells * 40.0}
    # a cycle reads and writes the leaves' interiors; operations per cell of
    # the update, an FMA as two
    per = {("lf", 3): 1785, ("lf", 2): 1123, ("weno", 3): 3315, ("weno", 2): 2225,
           ("mmc", 3): 900, ("mmc", 2): 600}[c["scheme"], nd]
    if c["eta"] > 0:
        per += 75 if nd == 3 else 60
    if c["cond"] != "off":
        per += 3 * 120
    return {"bytes": 2 * NV * w * cells * c["steps"], "flops": per * cells * c["steps"]}


# ---------------------------------------------------------------- the method in 64 bits
GAMMA, CFL, CD, CR = 5.0 / 3.0, 0.4, 0.18, 0.18


class _Mesh:
    """The block tree as index tables, in the library's slot order: by
    simulation, then Morton code at the finest level, then level."""

    def __init__(self, c, wl):
        self.c, self.wl, self.nd = c, wl, wl.ndim
        k = wl.keys.astype(np.int64)
        lmax = int(k[:, 1].max())
        code = np.zeros(len(k), dtype=np.int64)
        for d in range(self.nd):
            v = k[:, 2 + d] << (lmax - k[:, 1])
            for b in range(20):
                code |= ((v >> b) & 1) << (self.nd * b + d)
        self.order = np.lexsort((k[:, 1], code, k[:, 0]))
        self.k = k[self.order]
        self.lmax = lmax
        packed = self._pack(self.k)
        self.by = np.argsort(packed)
        self.sorted = packed[self.by]
        up = self.k.copy()
        up[:, 1] -= 1
        up[:, 2:] >>= 1
        self.parent = np.where(self.k[:, 1] > 1, self._find(up), -1)
        self.leaf = np.ones(len(k), dtype=bool)
        self.leaf[self.parent[self.parent >= 0]] = False
        self.cpos = sum((self.k[:, 2 + d] & 1) << d for d in range(self.nd))
        self.nbase = np.array([s.nbase for s in wl.sims], dtype=np.int64)[self.k[:, 0]]
        self.dx = np.ones((len(k), 3))
        for d in range(self.nd):
            ext = np.array([s.hi[d] - s.lo[d] for s in wl.sims])[self.k[:, 0]]
            self.dx[:, d] = ext / (self.nbase[:, d] * NB << (self.k[:, 1] - 1))
        self.outflow = np.array([[s.bc[d][0] == "outflow" for d in range(3)] for s in wl.sims])[self.k[:, 0]]
        z = (0,) if self.nd == 2 else (-1, 0, 1)
        self.dirs = [(a, b, e) for e in z for b in (-1, 0, 1) for a in (-1, 0, 1) if (a, b, e) != (0, 0, 0)]
        self.near = {d: self._neighbour(d) for d in self.dirs}
        self.leaves = np.nonzero(self.leaf)[0]

    @staticmethod
    def _pack(k):
        return ((k[:, 0] << 47) | (k[:, 1] << 42) | (k[:, 2] << 28) | (k[:, 3] << 14) | k[:, 4])

    def _find(self, k):
        p = self._pack(np.maximum(k, 0))
        i = np.minimum(np.searchsorted(self.sorted, p), len(self.sorted) - 1)
        return np.where(self.sorted[i] == p, self.by[i], -1)

    def _neighbour(self, dir_):
        """Index of the same-level block in a direction (periodic wrap; past
        an outflow side the block itself), -1 if none, and per dimension
        whether the side was clamped."""
        k, clamp = self.k.copy(), np.zeros((len(self.k), 3), dtype=bool)
        for d in range(self.nd):
            n = self.nbase[:, d] << (k[:, 1] - 1)
            v = k[:, 2 + d] + dir_[d]
            off = (v < 0) | (v >= n)
            clamp[:, d] = off & self.outflow[:, d]
            k[:, 2 + d] = np.where(clamp[:, d], k[:, 2 + d], v % n)
        return self._find(k), clamp

    # ------------------------------------------------------------ boundary procedure
    def span(self, a):
        return {-1: slice(0, NG), 0: slice(NG, NG + NB), 1: slice(NG + NB, NB + 2 * NG)}[a]

    def fill(self, U):
        dev = U.device
        for dr in self.dirs:
            src, clamp = self.near[dr]
            for combo in np.unique(clamp[src >= 0], axis=0):
                rows = np.nonzero((src >= 0) & (clamp == combo).all(axis=1))[0]
                at = [torch.arange(NB, device=dev) + NG if self.nd == 3 or d < 2 else torch.zeros(1, dtype=torch.long, device=dev)
                      for d in range(3)]
                to = [self.span(dr[d]) if self.nd == 3 or d < 2 else slice(0, 1) for d in range(3)]
                for d in range(self.nd):
                    if dr[d]:
                        first = {-1: [NB, NB + 1], 1: [NG, NG + 1]}[dr[d]]
                        edge = {-1: [NG, NG], 1: [NB + 1, NB + 1]}[dr[d]]
                        at[d] = torch.tensor(edge if combo[d] else first, device=dev)
                for part in _chunks(rows):
                    s = torch.from_numpy(src[part]).to(dev)
                    v = U[s[:, None, None, None], :, at[2][None, :, None, None], at[1][None, None, :, None],
                          at[0][None, None, None, :]].permute(0, 4, 1, 2, 3)
                    U[torch.from_numpy(part).to(dev), :, to[2], to[1], to[0]] = v
        for lv in range(2, self.lmax + 1):
            miss = {dr: (self.near[dr][0] < 0) & (self.k[:, 1] == lv) for dr in self.dirs}
            any_ = np.zeros(len(self.k), dtype=bool)
            for m in miss.values():
                any_ |= m
            for part in _chunks(np.nonzero(any_)[0]):
                P = self.prolong(U, part)
                for dr in self.dirs:
                    sel = np.nonzero(miss[dr][part])[0]
                    if len(sel):
                        to = [self.span(dr[d]) if self.nd == 3 or d < 2 else slice(0, 1) for d in range(3)]
                        s = torch.from_numpy(sel).to(dev)
                        U[torch.from_numpy(part[sel]).to(dev), :, to[2], to[1], to[0]] = P[s, :, to[2], to[1], to[0]]

    def prolong(self, U, rows):
        """Padded tiles of the blocks `rows` from their parents' padded tiles."""
        dev = U.device
        out = torch.empty((len(rows),) + U.shape[1:], dtype=U.dtype, device=dev)
        for cp in range(1 << self.nd):
            sel = np.nonzero(self.cpos[rows] == cp)[0]
            if not len(sel):
                continue
            T = U[torch.from_numpy(self.parent[rows[sel]]).to(dev)]
            at = [((cp >> d) & 1) * (NB // 2) - 1 + NG for d in range(3)]
            n = NB // 2 + 2

            def cut(o):
                z = slice(at[2] + o[2], at[2] + o[2] + n) if self.nd == 3 else slice(0, 1)
                return T[:, :, z, at[1] + o[1]:at[1] + o[1] + n, at[0] + o[0]:at[0] + o[0] + n]

            mid = cut((0, 0, 0))
            v = mid
            for d in range(self.nd):
                o = [0, 0, 0]
                o[d] = 1
                s = _minmod(cut(o) - mid, mid - cut([-q for q in o])) * 0.25
                ax = 4 - d
                # fine cells 2i (-) and 2i+1 (+) along d
                for e in range(d):
                    s = s.repeat_interleave(2, dim=4 - e)
                v = torch.stack((v - s, v + s), dim=ax + 1).flatten(ax, ax + 1)
            out[torch.from_numpy(sel).to(dev)] = v
        return out

    def restrict(self, U):
        dev = U.device
        for lv in range(self.lmax, 1, -1):
            kids = np.nonzero(self.k[:, 1] == lv)[0]
            for cp in range(1 << self.nd):
                for part in _chunks(kids[self.cpos[kids] == cp]):
                    c = self.inside(U[torch.from_numpy(part).to(dev)])
                    m = c.unfold(4, 2, 2).mean(-1).unfold(3, 2, 2).mean(-1)
                    if self.nd == 3:
                        m = m.unfold(2, 2, 2).mean(-1)
                    o = [slice(NG + ((cp >> d) & 1) * 8, NG + ((cp >> d) & 1) * 8 + 8) for d in range(3)]
                    if self.nd == 2:
                        o[2] = slice(0, 1)
                    U[torch.from_numpy(self.parent[part]).to(dev), :, o[2], o[1], o[0]] = m

    def inside(self, T, ring=0):
        s = slice(NG - ring, NG + NB + ring)
        return T[..., s, s, s] if self.nd == 3 else T[..., s, s]

    def shifted(self, T, d, o, ring):
        """The cells of inside(T, ring), moved by o cells along d."""
        s = [slice(NG - ring, NG + NB + ring)] * 3
        s[d] = slice(NG - ring + o, NG + NB + ring + o)
        return T[..., s[2], s[1], s[0]] if self.nd == 3 else T[..., s[1], s[0]]

    def reflux(self, U, F, dts, v=slice(None)):
        """Coarse leaves take the mean of the finer faces' fluxes; F[d][side]
        holds every block's face fluxes [nb, NV, t2, t1]."""
        dev = U.device
        for d in range(self.nd):
            for side in (0, 1):
                dr = [0, 0, 0]
                dr[d] = 1 if side else -1
                src, clamp = self.near[tuple(dr)]
                rows = np.nonzero(self.leaf & (src >= 0) & ~clamp[:, d])[0]
                rows = rows[~self.leaf[src[rows]]]
                tr = [e for e in range(self.nd) if e != d]
                for part in _chunks(rows):
                    fine = torch.empty((len(part),) + F[d][0][:, v].shape[1:], dtype=U.dtype, device=dev)
                    kid = self.k[src[part]].copy()
                    kid[:, 1] += 1
                    kid[:, 2:2 + self.nd] *= 2
                    kid[:, 2 + d] += 0 if side else 1
                    for h in range(1 << len(tr)):
                        kk = kid.copy()
                        to = [slice(0, 1), slice(0, 16)]
                        for j, e in enumerate(tr):
                            b = (h >> j) & 1
                            kk[:, 2 + e] += b
                            to[1 - j] = slice(8 * b, 8 * b + 8)
                        f = F[d][1 - side][torch.from_numpy(self._find(kk)).to(dev)][:, v]
                        f = f.unfold(3, 2, 2).mean(-1)
                        if self.nd == 3:
                            f = f.unfold(2, 2, 2).mean(-1)
                        fine[:, :, to[0], to[1]] = f
                    at = torch.from_numpy(part).to(dev)
                    r = torch.from_numpy(dts[self.k[part, 0]] / self.dx[part, d]).to(dev).view(-1, 1, 1, 1)
                    delta = r * (F[d][side][at][:, v] - fine)
                    ix = [slice(NG, NG + NB)] * 3 if self.nd == 3 else [slice(NG, NG + NB)] * 2 + [slice(0, 1)]
                    ix[d] = slice(NG + NB - 1, NG + NB) if side else slice(NG, NG + 1)
                    shape = [len(part), delta.shape[1]] + [(NB if self.nd == 3 or e < 2 else 1) for e in (2, 1, 0)]
                    shape[4 - d] = 1
                    delta = delta.reshape(shape)
                    cell = U[at, v, ix[2], ix[1], ix[0]]
                    U[at, v, ix[2], ix[1], ix[0]] = cell + delta if side else cell - delta


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))


def _limit(kind, a, b):
    if kind == "minmod":
        return _minmod(a, b)
    ab = a * b
    return torch.where(ab > 0, 2.0 * ab / torch.where(ab > 0, a + b, torch.ones_like(a)), torch.zeros_like(a))


def _pressure(u):
    ke = 0.5 * (u[:, 1:4] ** 2).sum(1) / u[:, 0]
    return (GAMMA - 1.0) * (u[:, EN] - ke - 0.5 * (u[:, 4:7] ** 2).sum(1))


def _admissible(u):
    return (u[:, 0] > 0) & (_pressure(u) > 0)


def _flux(u, d, ch):
    v, B, p = u[:, 1:4] / u[:, :1], u[:, 4:7], _pressure(u)
    pt = p + 0.5 * (B ** 2).sum(1)
    vd, Bd = v[:, d], B[:, d]
    f = torch.empty_like(u)
    f[:, 0] = u[:, MX + d]
    f[:, 1:4] = u[:, 1:4] * vd[:, None] - B * Bd[:, None]
    f[:, MX + d] += pt
    f[:, 4:7] = B * vd[:, None] - v * Bd[:, None]
    f[:, BX + d] = u[:, PSI]
    f[:, EN] = (u[:, EN] + pt) * vd - Bd * (v * B).sum(1)
    f[:, PSI] = ch * ch * Bd
    return f


def _fast(u, d):
    a2, b2 = GAMMA * _pressure(u) / u[:, 0], (u[:, 4:7] ** 2).sum(1) / u[:, 0]
    s = a2 + b2
    disc = (s * s - 4.0 * a2 * u[:, BX + d] ** 2 / u[:, 0]).clamp(min=0)
    return (0.5 * (s + disc.sqrt())).clamp(min=0).sqrt()


def _rusanov(L, R, d, ch):
    sl = (L[:, MX + d] / L[:, 0]).abs() + _fast(L, d)
    sr = (R[:, MX + d] / R[:, 0]).abs() + _fast(R, d)
    a = torch.maximum(sl, sr)[:, None].expand_as(L).clone()
    a[:, BX + d] = ch
    a[:, PSI] = ch
    return 0.5 * (_flux(L, d, ch) + _flux(R, d, ch)) - 0.5 * a * (R - L)


def _hllc(L, R, d, ch):
    Bm = 0.5 * (L[:, BX + d] + R[:, BX + d]) - (R[:, PSI] - L[:, PSI]) / (2.0 * ch)
    pm = 0.5 * (L[:, PSI] + R[:, PSI]) - 0.5 * ch * (R[:, BX + d] - L[:, BX + d])
    S = []
    for u in (L, R):
        u = u.clone()
        p = _pressure(u) + (GAMMA - 1.0) * 0.5 * (u[:, BX + d] ** 2 - Bm ** 2)
        u[:, BX + d] = Bm
        S.append((u, _flux(u, d, ch), u[:, MX + d] / u[:, 0], p + 0.5 * (u[:, 4:7] ** 2).sum(1), _fast(u, d),
                  (u[:, 1:4] * u[:, 4:7]).sum(1) / u[:, 0]))
    (UL, FL, vL, ptL, cL, vbL), (UR, FR, vR, ptR, cR, vbR) = S
    c = torch.maximum(cL, cR)
    SL, SR = torch.minimum(vL, vR) - c, torch.maximum(vL, vR) + c
    h = (SR[:, None] * UR - SL[:, None] * UL - FR + FL) / (SR - SL)[:, None]
    h[:, BX + d] = Bm
    SM = h[:, MX + d] / h[:, 0]
    vbh = (h[:, 1:4] * h[:, 4:7]).sum(1) / h[:, 0]
    ps = 0.5 * (UL[:, 0] * (SL - vL) * (SM - vL) + ptL + UR[:, 0] * (SR - vR) * (SM - vR) + ptR)
    f = torch.empty_like(L)
    for u, F, v, pt, vb, Sk, side in ((UL, FL, vL, ptL, vbL, SL, SM >= 0), (UR, FR, vR, ptR, vbR, SR, SM < 0)):
        st = torch.empty_like(u)
        den = Sk - SM
        st[:, 0] = u[:, 0] * (Sk - v) / den
        st[:, 1:4] = (u[:, 1:4] * (Sk - v)[:, None] - Bm[:, None] * (h[:, 4:7] - u[:, 4:7])) / den[:, None]
        st[:, MX + d] = st[:, 0] * SM
        st[:, 4:7] = h[:, 4:7]
        st[:, EN] = (u[:, EN] * (Sk - v) - pt * v + ps * SM + Bm * (vb - vbh)) / den
        st[:, PSI] = u[:, PSI]
        f = torch.where(side[:, None], F + Sk[:, None] * (st - u), f)
    f = torch.where((SL >= 0)[:, None], FL, torch.where((SR <= 0)[:, None], FR, f))
    f[:, BX + d] = pm
    f[:, PSI] = ch * ch * Bm
    return f


def _weno(um, u, up):
    sm, sp = (1e-12 + (u - um) ** 2) ** 2, (1e-12 + (up - u) ** 2) ** 2
    L = (2.0 * sm * 0.5 * (u + up) + sp * 0.5 * (3.0 * u - um)) / (2.0 * sm + sp)
    R = (sm * 0.5 * (3.0 * u - up) + 2.0 * sp * 0.5 * (u + um)) / (sm + 2.0 * sp)
    return L, R


def _part(A, nd, d, lo, hi):
    """Cells lo..hi-1 along d, interior ones along the others, of an array on
    the interior and one ring."""
    s = [slice(1, NB + 1)] * 3
    s[d] = slice(lo + 1, hi + 1)
    return A[..., s[2], s[1], s[0]] if nd == 3 else A[..., s[1], s[0]]


def _update(M, T, r, rows, c):
    """(u + dt L(u) without damping, face fluxes per dimension) of padded
    tiles T; r: the records of their simulations, rows: their blocks."""
    nd, dev = M.nd, T.device
    col = lambda x: torch.as_tensor(x, dtype=torch.float64, device=dev).view(-1, 1, 1, 1, 1)  # noqa: E731
    sc = lambda x: col(x)[:, 0]  # noqa: E731
    dt, ch = col(r["dt"]), sc(r["ch"])
    dx = [col(M.dx[rows, d]) for d in range(nd)]
    u1 = M.inside(T, 1)
    F = []
    if c["scheme"] == "mmc":
        al = []
        for d in range(nd):
            a = sc(r["alpha"])[:, None].expand(len(rows), NV, 1, 1, 1).clone()
            a[:, BX + d] = ch
            a[:, PSI] = ch
            al.append(a)
        fp = [0.5 * (_flux(T, d, ch) + al[d] * T) for d in range(nd)]
        fm = [0.5 * (_flux(T, d, ch) - al[d] * T) for d in range(nd)]
        ut = u1.clone()
        for d in range(nd):
            hp = M.inside(fp[d], 1) + M.shifted(fm[d], d, 1, 1)
            hm = M.shifted(fp[d], d, -1, 1) + M.inside(fm[d], 1)
            ut -= dt / dx[d] * (hp - hm)
        for d in range(nd):
            ft = _flux(ut, d, ch)
            tp, tm = 0.5 * (ft + al[d] * ut), 0.5 * (ft - al[d] * ut)

            def pad(A, o):  # cells -1+o .. 15+o along d of a padded array
                s = [slice(NG, NG + NB)] * 3
                s[d] = slice(NG - 1 + o, NG + NB + o)
                return A[..., s[2], s[1], s[0]] if nd == 3 else A[..., s[1], s[0]]

            t0p, t1p = _part(tp, nd, d, -1, NB), _part(tp, nd, d, 0, NB + 1)
            t0m, t1m = _part(tm, nd, d, -1, NB), _part(tm, nd, d, 0, NB + 1)
            h = pad(fp[d], 0) + pad(fm[d], 1)
            F.append(h + 0.5 * (_limit(c["limiter"], t0p - pad(fp[d], -1), t1p - pad(fp[d], 0)) -
                                _limit(c["limiter"], pad(fm[d], 2) - t1m, pad(fm[d], 1) - t0m)))
    else:
        face = _rusanov if c["riemann"] == "rusanov" else _hllc
        if c["scheme"] == "lf":
            dl = [_limit(c["limiter"], u1 - M.shifted(T, d, -1, 1), M.shifted(T, d, 1, 1) - u1) for d in range(nd)]
            ok, acc = True, 0.0
            for d in range(nd):
                a, b = u1 + 0.5 * dl[d], u1 - 0.5 * dl[d]
                ok = ok & _admissible(a) & _admissible(b)
                acc = acc + 0.5 * dt / dx[d] * (_flux(a, d, ch) - _flux(b, d, ch))
            ok = ok[:, None]
            back = torch.where(ok, u1 - acc, u1)
            dl = [torch.where(ok, s, torch.zeros_like(s)) for s in dl]
        else:
            back = u1
        for d in range(nd):
            if c["scheme"] == "lf":
                L, R = back + 0.5 * dl[d], back - 0.5 * dl[d]
            else:
                L, R = _weno(M.shifted(T, d, -1, 1), u1, M.shifted(T, d, 1, 1))
            L = torch.where(_admissible(L)[:, None], L, back)
            R = torch.where(_admissible(R)[:, None], R, back)
            F.append(face(_part(L, nd, d, -1, NB), _part(R, nd, d, 0, NB + 1), d, ch))
    u = M.inside(T)
    out = u.clone()
    for d in range(nd):
        ax = 4 - d
        out -= dt / dx[d] * (F[d].narrow(ax, 1, NB) - F[d].narrow(ax, 0, NB))
    t = dt[:, 0]
    grad = lambda A, d, ring=0: (M.shifted(A, d, 1, ring) - M.shifted(A, d, -1, ring)) * (0.5 / dx[d][:, 0])  # noqa: E731
    div = sum(grad(T[:, BX + d], d) for d in range(nd))
    out[:, 1:4] -= t[:, None] * div[:, None] * u[:, 4:7]
    out[:, EN] -= t * sum(u[:, BX + d] * grad(T[:, PSI], d) for d in range(nd))
    if c["eta"] > 0:
        zero = torch.zeros_like(u1[:, 0])
        g = lambda v, d: grad(T[:, v], d, 1) if d < nd else zero  # noqa: E731
        J = [g(6, 1) - g(5, 2), g(4, 2) - g(6, 0), g(5, 0) - g(4, 1)]
        B = [u1[:, 4], u1[:, 5], u1[:, 6]]
        Q = [J[2] * B[1] - J[1] * B[2], J[0] * B[2] - J[2] * B[0], J[1] * B[0] - J[0] * B[1]]

        def dif(A, d):  # central difference of an array on the interior and one ring
            if d >= nd:
                return 0.0
            return (_part(A, nd, d, 1, NB + 1) - _part(A, nd, d, -1, NB - 1)) * (0.5 / dx[d][:, 0])

        et = c["eta"] * t
        out[:, 4] -= et * (dif(J[2], 1) - dif(J[1], 2))
        out[:, 5] -= et * (dif(J[0], 2) - dif(J[2], 0))
        out[:, 6] -= et * (dif(J[1], 0) - dif(J[0], 1))
        out[:, EN] += et * sum(dif(Q[d], d) for d in range(nd))
    return out, F


def _conduct(M, U, c, wl, r):
    """nsub sub-steps of the energy."""
    nd, dev = M.nd, U.device
    for sub in range(int(max(r["nsub"]))):
        on = M.leaves[r["nsub"][M.k[M.leaves, 0]] > sub]
        F = [[torch.zeros((len(M.k), NV, NB if nd == 3 else 1, NB), dtype=U.dtype, device=dev) for _ in (0, 1)]
             for _ in range(nd)]
        new = []
        for part in _chunks(on):
            at = torch.from_numpy(part).to(dev)
            T = U[at]
            tt = _pressure(T) / T[:, 0]
            kap = (wl.kappa0 * tt ** wl.kappa_exp).clamp(min=0).sqrt()
            dx = [torch.from_numpy(M.dx[part, d]).to(dev).view(-1, 1, 1, 1) for d in range(nd)]
            acc = 0.0
            for d in range(nd):
                def cells(A, o, e=None, oe=0):  # cells -1+o .. 15+o along d, moved by oe along e
                    s = [slice(NG, NG + NB)] * 3
                    s[d] = slice(NG - 1 + o, NG + NB + o)
                    if e is not None:
                        s[e] = slice(NG + oe, NG + NB + oe)
                    return A[..., s[2], s[1], s[0]] if nd == 3 else A[..., s[1], s[0]]

                kf = cells(kap, 0) * cells(kap, 1)
                gd = (cells(tt, 1) - cells(tt, 0)) / dx[d]
                if c["cond"] == "iso":
                    f = -kf * gd
                else:
                    B = [0.5 * (cells(T[:, 4 + j], 0) + cells(T[:, 4 + j], 1)) for j in range(3)]
                    bb = B[0] ** 2 + B[1] ** 2 + B[2] ** 2
                    bg = B[d] * gd
                    for e in range(nd):
                        if e != d:
                            bg = bg + B[e] * 0.25 / dx[e] * (
                                cells(tt, 0, e, 1) - cells(tt, 0, e, -1) + cells(tt, 1, e, 1) - cells(tt, 1, e, -1))
                    f = torch.where(bb > 0, -kf * B[d] * bg / torch.where(bb > 0, bb, torch.ones_like(bb)),
                                    torch.zeros_like(bb))
                ax = 3 - d
                acc = acc + (f.narrow(ax, 1, NB) - f.narrow(ax, 0, NB)) / dx[d]
                for side, x in ((0, f.select(ax, 0)), (1, f.select(ax, NB))):
                    F[d][side][at, EN] = x
            h = torch.from_numpy(r["dt_sub"][M.k[part, 0]]).to(dev).view(-1, 1, 1, 1)
            new.append((at, M.inside(T)[:, EN] - h * acc))
        for at, e in new:
            M.inside(U)[at, EN] = e
        act = np.where(r["nsub"] > sub, r["dt_sub"], 0.0)
        M.reflux(U, F, act, v=slice(EN, EN + 1))
        M.restrict(U)
        M.fill(U)


def _cycle(M, U, c, wl):
    nd, dev, ns = M.nd, U.device, len(wl.sims)
    alpha, kmax = np.zeros(ns), np.zeros(ns)
    for part in _chunks(M.leaves):
        u = M.inside(U[torch.from_numpy(part).to(dev)])
        s = torch.stack([(u[:, MX + d] / u[:, 0]).abs() + _fast(u, d) for d in range(nd)]).amax(0)
        np.maximum.at(alpha, M.k[part, 0], s.flatten(1).amax(1).cpu().numpy())
        if c["cond"] != "off":
            q = wl.kappa0 * (_pressure(u) / u[:, 0]) ** wl.kappa_exp / u[:, 0]
            np.maximum.at(kmax, M.k[part, 0], q.flatten(1).amax(1).cpu().numpy())
    dxm = np.full(ns, np.inf)
    np.minimum.at(dxm, M.k[M.leaves, 0], M.dx[M.leaves][:, :nd].min(1))
    dt = CFL * dxm / (nd * alpha)
    if c["eta"] > 0:
        dt = np.minimum(dt, CFL * dxm ** 2 / (nd * c["eta"]))
    r = {"alpha": alpha, "nsub": np.zeros(ns, dtype=np.int64), "dt_sub": np.zeros(ns)}
    if c["cond"] != "off":
        dtc = CFL * dxm ** 2 / (nd * kmax)
        dt = np.minimum(dt, wl.cond_max_sub * dtc)
        r["nsub"] = np.clip(np.ceil(dt / dtc), 1, wl.cond_max_sub).astype(np.int64)
        r["dt_sub"] = dt / r["nsub"]
    r["dt"] = dt
    if wl.glm_mode == "paper":
        r["ch"], r["damp"] = CFL * dxm / dt, np.full(ns, CD)
    else:
        r["ch"], r["damp"] = alpha, np.exp(-dt * alpha / CR)

    def sweep(V):
        out = torch.empty_like(V)
        out.copy_(V)
        F = [[torch.zeros((len(M.k), NV, NB if nd == 3 else 1, NB), dtype=V.dtype, device=dev) for _ in (0, 1)]
             for _ in range(nd)]
        size = max(1, CHUNK // 2)
        for i in range(0, len(M.leaves), size):
            part = M.leaves[i:i + size]
            at = torch.from_numpy(part).to(dev)
            rr = {k: r[k][M.k[part, 0]] for k in ("dt", "ch", "alpha")}
            o, f = _update(M, V[at], rr, part, c)
            M.inside(out)[at] = o
            for d in range(nd):
                F[d][0][at], F[d][1][at] = f[d].select(4 - d, 0), f[d].select(4 - d, NB)
        return out, F

    def damp(V):
        w = torch.from_numpy(np.where(M.leaf, r["damp"][M.k[:, 0]], 1.0)).to(dev)
        M.inside(V)[:, PSI] *= w.view(-1, 1, 1, 1)

    new, F = sweep(U)
    if c["scheme"] == "weno":
        M.restrict(new)
        M.fill(new)
        two, F2 = sweep(new)
        new = 0.5 * (U + two)
        F = [[0.5 * (a + b) for a, b in zip(F[d], F2[d])] for d in range(nd)]
    damp(new)
    M.reflux(new, F, dt)
    M.restrict(new)
    M.fill(new)
    if c["cond"] != "off":
        _conduct(M, new, c, wl, r)
    return new, r


def _estimate(M, U):
    """Per block the largest estimate of its interior and first ring, in the
    caller's key order."""
    nd, dev = M.nd, U.device
    err = np.zeros(len(M.k))
    for part in _chunks(np.arange(len(M.k))):
        T = U[torch.from_numpy(part).to(dev)]
        for mode, var, eps in CRITERIA:
            v = (T[:, 4:7] ** 2).sum(1).sqrt() if mode == "bmag" else T[:, var]
            m = M.inside(v, 1)
            p, q = zip(*[(M.shifted(v, d, 1, 1), M.shifted(v, d, -1, 1)) for d in range(nd)])
            d1 = 0.5 * math.sqrt(3.0) * sum((a - b) ** 2 for a, b in zip(p, q)).sqrt()
            d2 = sum((a - 2.0 * m + b) ** 2 for a, b in zip(p, q)).sqrt()
            av = m.abs() + eps
            e = 0.6 * d1 / av + 0.4 * d2 / (d1 + 0.05 * av)
            err[part] = np.maximum(err[part], e.flatten(1).amax(1).cpu().numpy())
    out = np.zeros_like(err)
    out[M.order] = err
    return out


def exact(case, seed):
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    if c["call"] == "regrid":
        return None
    wl = _workload(c)
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    M = _Mesh(c, wl)
    n = NB + 2 * NG
    U = torch.zeros((len(M.k), NV, n if M.nd == 3 else 1, n, n), dtype=torch.float64, device=dev)
    slot = np.empty(len(M.k), dtype=np.int64)
    slot[M.order] = np.arange(len(M.k))
    held = torch.float64 if c["precision"] == "fp64" else torch.float32
    inside = M.inside(U)
    _, leaf = _tree(c["problem"], c["nx"], c["ny"], c["nz"], c["levels"], c["nsims"], c["kmax"])
    for rows in _chunks(np.nonzero(leaf)[0]):
        f = _primitives(c, wl, rows, seed, dev).to(held).to(torch.float64)
        u = f.clone()
        u[:, 1:4] = f[:, :1] * f[:, 1:4]
        u[:, EN] = f[:, EN] / (GAMMA - 1.0) + 0.5 * f[:, 0] * (f[:, 1:4] ** 2).sum(1) + 0.5 * (f[:, 4:7] ** 2).sum(1)
        inside[torch.from_numpy(slot[rows]).to(dev)] = u.to(held).to(torch.float64)
    M.restrict(U)
    M.fill(U)
    if c["call"] == "output":
        tot = np.zeros((len(wl.sims), NV))
        for part in _chunks(M.leaves):
            vol = M.dx[part].prod(1)[:, None]
            s = M.inside(U[torch.from_numpy(part).to(dev)]).flatten(2).sum(2).cpu().numpy() * vol
            np.add.at(tot, M.k[part, 0], s)
        return {"U": U, "totals": tot, "err": _estimate(M, U)}
    for _ in range(c["steps"]):
        U, r = _cycle(M, U, c, wl)
    dt = np.stack([r["dt"], r["ch"], r["damp"], r["alpha"], r["dt_sub"]], axis=1)
    return {"U": M.inside(U), "dt": torch.from_numpy(dt), "nsub": None}
