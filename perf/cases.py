"""The work this framework is timed on.

Every case is one pass of a program that holds a block hierarchy on the device
and drives it through the public entry points: steps of a simulation (as one
captured step per `advance`, or stage by stage), a step of a pool of
independent jobs, or one adaptive cycle.  The listed cases are the workloads
of bench.py and of the test suite at their own sizes; `draw` gives others of
the same ranges (any block counts, limiters, fluxes, schemes, precisions).

Initial states are made on the device from the seed alone.  Each step is
checked against `exact`, the same scheme written out in plain torch in 64
bits.
"""
import ctypes
import functools
import math

import numpy as np
import torch

from paper_2303_03026_amd import amrvac, inputs

NV = 9
RHO, VX, VY, VZ, PR, BX, BY, BZ, PSI = range(NV)
PERIODIC, ZEROGRAD, REFLECT, FIXED = 0, 1, 2, 3
LIMITERS = {"vanleer": 0, "koren": 1, "cada3": 2, "weno5": 3, "wenoz5": 4, "mp5": 5, "wenozp5": 6}
FLUXES = {"hll": 0, "hlld": 1, "hllc": 2}
LOHNER_EPS, LOHNER_REFINE, LOHNER_COARSEN = 0.01, 0.1, 0.025


def _case(**kw):
    c = dict(kind="advance", state="modes", ndim=3, bx=4, by=4, bz=4, nx=16, levels=1, limiter="vanleer",
             flux="hll", mixed=False, plain=False, stages=3, steps=1, graph=True)
    c.update(kw)
    if c["ndim"] == 2:
        c["bz"] = 1
    return c


def listed():
    return [
        # the smallest grid of the test suite, 16 blocks: nothing but launches
        # and the latency of one block; steps in one captured graph
        _case(name="vortex_64_2d", state="vortex", ndim=2, bx=4, by=4, stages=2, steps=10),
        # a typical 2D job of the serving mix: a few hundred blocks, FP32-mixed
        _case(name="modes_256_2d_mixed", ndim=2, bx=16, by=16, mixed=True, steps=5),
        # the Kelvin-Helmholtz run: 6 levels in 2D, the five-cell
        # reconstruction and HLLC; under a million cells, so launches count
        _case(name="shear_layer_6_levels_wenozp5_hllc", state="shear", ndim=2, bx=8, by=4, levels=6,
              limiter="wenozp5", flux="hllc"),
        # the 2D MHD shock-cloud comparison: 6 levels, koren and HLLD, FP32-mixed
        _case(name="alfven_6_levels_koren_hlld_mixed", state="alfven", ndim=2, bx=8, by=8, levels=6,
              limiter="koren", flux="hlld", mixed=True),
        # one adaptive cycle of the Kelvin-Helmholtz run: the device's
        # refinement indicator, the host's plan, the transfer into a new context
        _case(name="shear_layer_6_levels_adapt", kind="adapt", state="shear", ndim=2, bx=8, by=4, levels=6,
              flux="hllc", graph=False),
        # a block size that only the per-kernel path takes, on a 3-level grid
        _case(name="modes_8cubed_blocks_3_levels_plain", bx=6, by=6, bz=6, nx=8, levels=3, plain=True, graph=False),
        # the serving engine's round: independent 3D jobs advanced together
        _case(name="pool_of_3d_jobs", kind="pool", bx=2, by=8, bz=6, graph=False),
        # the low-beta current sheet with walls, driven stage by stage
        _case(name="sheet_192_walls_staged", kind="staged", state="sheet", bx=12, by=12, bz=12, graph=False),
        # the headline grid in both precisions
        _case(name="modes_256_3d", bx=16, by=16, bz=16),
        _case(name="modes_256_3d_mixed", bx=16, by=16, bz=16, mixed=True),
        # the 3D shock cloud on 3 levels with inflow: ghost fills and flux corrections
        _case(name="cloud_3_levels_3d", state="cloud", bx=8, by=8, bz=8, levels=3),
        # the five-cell reconstruction on the headline grid: the largest pass
        _case(name="modes_256_3d_wenozp5_hllc", bx=16, by=16, bz=16, limiter="wenozp5", flux="hllc"),
    ]


def draw(rng):
    def size(lo, hi):  # log-uniform whole number
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))

    what = rng.random()
    flux = rng.choice(["hll", "hll", "hlld", "hllc"])
    two = ["vanleer", "vanleer", "koren", "cada3"]
    five = ["weno5", "wenoz5", "mp5", "wenozp5"]
    if what < 0.3:  # uniform 2D grids
        return _case(ndim=2, bx=size(2, 40), by=size(2, 40), limiter=rng.choice(two + five[3:]), flux=flux,
                     mixed=rng.random() < 0.5, stages=rng.choice([2, 3, 3, 4, 5]), steps=rng.randint(1, 8))
    if what < 0.55:  # uniform 3D grids, the two-ghost-layer limiters
        return _case(bx=size(2, 14), by=size(2, 14), bz=size(2, 14), limiter=rng.choice(two), flux=flux,
                     mixed=rng.random() < 0.5, stages=rng.choice([2, 3, 3, 4, 5]), steps=rng.randint(1, 2),
                     kind=rng.choice(["advance", "advance", "staged"]))
    if what < 0.65:  # uniform 3D grids, the five-cell ones
        return _case(bx=size(2, 9), by=size(2, 9), bz=size(2, 9), limiter=rng.choice(five), flux=flux,
                     mixed=rng.random() < 0.5)
    if what < 0.75:  # refined 3D grids
        return _case(state=rng.choice(["cloud", "modes"]), bx=size(3, 7), by=size(3, 7), bz=size(3, 7),
                     levels=rng.randint(2, 3), limiter=rng.choice(two), flux=flux, mixed=rng.random() < 0.5)
    if what < 0.85:  # refined 2D grids
        state = rng.choice(["shear", "alfven"])
        return _case(state=state, ndim=2, bx=size(4, 12), by=size(4, 12), levels=rng.randint(2, 5),
                     limiter=rng.choice(two + five[3:]) if state == "shear" else rng.choice(two), flux=flux,
                     mixed=rng.random() < 0.5, steps=rng.randint(1, 4))
    if what < 0.93:  # the per-kernel path's block sizes
        return _case(bx=size(2, 8), by=size(2, 8), bz=size(2, 8), nx=rng.choice([4, 6, 8, 10, 12, 16]), plain=True,
                     levels=rng.randint(1, 2), limiter=rng.choice(two), flux=flux, graph=rng.random() < 0.5)
    return _case(kind="pool", bx=size(2, 4), by=size(4, 8), bz=rng.randint(2, 9), mixed=rng.random() < 0.5,
                 limiter=rng.choice(two), flux=flux, graph=False)


# ---------------------------------------------------------------------------
# grids


def _nest(leaves, ndim, base, periodic):
    """Refine until face, edge and corner neighbours differ by one level at most."""
    offs = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in ((-1, 0, 1) if ndim == 3 else (0,))]
    todo = sorted(leaves, reverse=True)
    while todo:
        key = todo.pop()
        if key not in leaves or key[0] < 3:
            continue
        l = key[0]
        for o in offs:
            p = [key[1 + d] + o[d] for d in range(3)]
            n = [base[d] << (l - 1) for d in range(3)]
            if any(not 0 <= p[d] < n[d] and not periodic[d] for d in range(ndim)):
                continue
            p = [p[d] % n[d] if d < ndim else 0 for d in range(3)]
            m = l
            while m > 0 and (m,) + tuple(p) not in leaves:
                m, p = m - 1, [q >> 1 for q in p]
            if 0 < m < l - 1:
                leaves.discard((m,) + tuple(p))
                born = _children((m,) + tuple(p), ndim)
                leaves.update(born)
                todo.extend(born)
                todo.append(key)
    return leaves


def _children(k, ndim):
    return [(k[0] + 1, 2 * k[1] + a, 2 * k[2] + b, 2 * k[3] + c if ndim == 3 else 0)
            for c in ((0, 1) if ndim == 3 else (0,)) for b in (0, 1) for a in (0, 1)]


def _box(case):
    """Lower and upper corner of the domain and its boundary kinds per axis."""
    base = (case["bx"], case["by"], case["bz"])
    state = case["state"]
    if state == "vortex":
        return (0.0,) * 3, (2 * math.pi, 2 * math.pi, 1.0), (PERIODIC,) * 3, (PERIODIC,) * 3
    if state == "sheet":
        bc = (PERIODIC, REFLECT, PERIODIC)
        return (-0.5,) * 3, (0.5,) * 3, bc, bc
    if state == "cloud":
        return (0.0,) * 3, (1.0,) * 3, (FIXED, ZEROGRAD, ZEROGRAD), (ZEROGRAD,) * 3
    if state == "shear":
        bc = (PERIODIC, REFLECT, PERIODIC)
        return (-1.5, -0.75, 0.0), (1.5, 0.75, 1.0), bc, bc
    if state == "alfven":
        bc = (ZEROGRAD, ZEROGRAD, PERIODIC)
        return (-0.5, -1.0, 0.0), (3.0, 2.5, 1.0), bc, bc
    big = float(max(base[:case["ndim"]]))
    hi = tuple(base[d] / big if d < case["ndim"] else 1.0 for d in range(3))
    return (0.0,) * 3, hi, (PERIODIC,) * 3, (PERIODIC,) * 3


CLOUD_CENTRE = (0.40464485, 0.41939646, 0.6256903)


@functools.lru_cache(maxsize=64)
def _leaves(state, ndim, base, levels, lo, hi, bc_lo):
    """Leaf blocks (level, i, j, k): a shell around a sphere in 3D, a band
    around the shear layer, the rectangle of the cloud and the shock."""
    def wanted(k):
        w = [(hi[d] - lo[d]) / (base[d] << (k[0] - 1)) for d in range(3)]
        a = [lo[d] + k[1 + d] * w[d] for d in range(3)]
        b = [a[d] + w[d] for d in range(3)]
        if state == "shear":
            return a[1] - 0.05 <= 0.0 <= b[1] + 0.05
        if state == "alfven":
            return (a[0] <= 1.0 and b[0] >= 0.0 and a[1] <= 1.5 and b[1] >= 0.0) or a[0] <= -0.3 <= b[0]
        c = [lo[d] + CLOUD_CENTRE[d] * (hi[d] - lo[d]) for d in range(3)]
        near = math.sqrt(sum(max(0.0, a[d] - c[d], c[d] - b[d]) ** 2 for d in range(ndim)))
        far = math.sqrt(sum(max(abs(a[d] - c[d]), abs(b[d] - c[d])) ** 2 for d in range(ndim)))
        return near <= 0.25 and (k[0] == 1 or far >= 0.2)

    leaves = {(1, i, j, k) for k in range(base[2]) for j in range(base[1]) for i in range(base[0])}
    for l in range(1, levels):
        for k in [k for k in leaves if k[0] == l and wanted(k)]:
            leaves.discard(k)
            leaves.update(_children(k, ndim))
    if levels > 2:
        leaves = _nest(leaves, ndim, base, [b == PERIODIC for b in bc_lo])
    keys = sorted(leaves, key=lambda t: (t[0], t[3], t[2], t[1]))  # x fastest within a level
    arr = np.array(keys, dtype=np.int32)
    return arr[:, 0].copy(), arr[:, 1:].copy()


class _Grid:
    """Blocks, spacing and cell centres of a case."""

    def __init__(self, case, dev):
        self.ndim, self.nx = case["ndim"], case["nx"]
        self.ng = 3 if LIMITERS[case["limiter"]] >= 3 else 2
        self.base = (case["bx"], case["by"], case["bz"])
        self.lo, self.hi, self.bc_lo, self.bc_hi = _box(case)
        self.level, self.ijk = _leaves(case["state"], self.ndim, self.base, case["levels"], self.lo, self.hi,
                                       self.bc_lo)
        self.nb = len(self.level)
        self.shape = (self.nb,) + (self.nx,) * self.ndim
        self.dx = np.array([[(self.hi[d] - self.lo[d]) / ((self.base[d] << (int(l) - 1)) * self.nx)
                             for d in range(3)] for l in range(1, int(self.level.max()) + 1)])[self.level - 1]
        self.fixed = np.zeros((3, 2, NV))
        if case["state"] == "cloud":
            self.fixed[0, 0, [RHO, VX, PR, BX]] = 1.0, 2.0, 1.0, 1.0
        self.dev = dev

    def centres(self):
        out = []
        for d in range(self.ndim):
            g = torch.from_numpy(self.ijk[:, d].astype(np.float64)).to(self.dev)[:, None] * self.nx
            g = g + torch.arange(self.nx, device=self.dev, dtype=torch.float64) + 0.5
            c = self.lo[d] + g * torch.from_numpy(self.dx[:, d].copy()).to(self.dev)[:, None]
            view = [self.nb] + [1] * self.ndim
            view[self.ndim - d] = self.nx
            out.append(c.reshape(view))
        return out

    def workload(self, case):
        return inputs.Workload(case["state"], self.ndim, self.nx, self.base, self.lo, self.hi, self.bc_lo, self.bc_hi,
                               self.level, self.ijk, None, nstages=case["stages"], ng=self.ng,
                               limiter=LIMITERS[case["limiter"]], flux=FLUXES[case["flux"]], bc_fixed_prim=self.fixed)


def _modes(rng, ndim, vector):
    ks = [k for k in np.ndindex(9, 9, 9 if ndim == 3 else 1)]
    ks = np.array([(a - 4, b - 4, c - 4 if ndim == 3 else 0) for a, b, c in ks])
    n2 = (ks ** 2).sum(1)
    half = [next((c for c in k if c), 0) > 0 for k in ks]
    ks = ks[(n2 >= 1) & (n2 <= 16) & half]
    ks = ks[rng.choice(len(ks), size=min(32, len(ks)), replace=False)]
    phase = rng.uniform(0.0, 2 * math.pi, size=len(ks))
    amp = math.sqrt(2.0 / len(ks)) * np.ones((len(ks), 1))
    if vector:  # across k: divergence-free
        a = rng.normal(size=(len(ks), 3))
        a -= (a * ks).sum(1, keepdims=True) / (ks ** 2).sum(1, keepdims=True) * ks
        amp = amp * a / np.linalg.norm(a, axis=1, keepdims=True)
    return ks, phase, amp


def _initial(case, seed, dev):
    """The case's grid and its primitive state [block][var][(z)][y][x]."""
    G = _Grid(case, dev)
    c = G.centres()
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    noise = lambda: 2.0 * torch.rand(G.shape, generator=gen, device=dev, dtype=torch.float64) - 1.0  # noqa: E731
    p = torch.zeros((G.nb, NV) + G.shape[1:], device=dev, dtype=torch.float64)
    x, y = c[0], c[1]
    state = case["state"]
    if state == "vortex":
        p[:, RHO] = 25.0 / 9.0 + 1e-3 * noise()
        p[:, VX], p[:, VY], p[:, PR] = -torch.sin(y), torch.sin(x), 5.0 / 3.0
        p[:, BX], p[:, BY] = -torch.sin(y), torch.sin(2 * x)
    elif state == "sheet":
        p[:, RHO], p[:, PR] = 1.0, 0.005
        for q in (VX, VY, VZ):
            p[:, q] = 1e-2 * noise()
        p[:, BX], p[:, BZ] = torch.tanh(y / 0.05), 1.0 / torch.cosh(y / 0.05)
    elif state == "cloud":
        r2 = sum((c[d] - CLOUD_CENTRE[d]) ** 2 for d in range(3))
        p[:, RHO] = torch.where(r2 <= 0.0625, 10.0, 1.0) * (1.0 + 1e-3 * noise())
        p[:, PR], p[:, BX] = 1.0, 1.0
    elif state == "shear":
        up = (y > 0.0).expand(G.shape)
        p[:, RHO], p[:, VX] = torch.where(up, 1.5, 1.0).double(), torch.where(up, 0.08, -0.12).double()
        p[:, VY], p[:, PR] = 1e-3 * noise(), 0.6
    elif state == "alfven":  # an intermediate shock of compression 2.5 moving into a cloud
        up = (1.0, 0.0, 0.0, 0.0, 0.6, -2.65365579, 2.2266816, 0.0, 0.0)
        down = (2.5, 1.71359706, -2.67923539, 0.0, 7.75735858, -2.65365579, -0.65684353, 0.0, 0.0)
        post = (x < -0.3).expand(G.shape)
        for q in range(NV):
            p[:, q] = torch.where(post, down[q], up[q]).double()
        r = np.random.Generator(np.random.PCG64(int(seed)))
        img = torch.zeros(G.shape, device=dev, dtype=torch.float64)
        for _ in range(12):
            cx, cy, w, a = r.uniform(0, 1), r.uniform(0, 1.5), r.uniform(0.03, 0.15), r.uniform(0.3, 1)
            img += a * torch.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (2 * w * w))
        inside = (x >= 0.0) & (x <= 1.0) & (y >= 0.0) & (y <= 1.5)
        p[:, RHO] = torch.where(inside, 1.0 + 128.0 * img.clamp(max=1.0), p[:, RHO])
    else:
        rng = np.random.Generator(np.random.PCG64(int(seed)))
        p[:, RHO], p[:, PR], p[:, BX] = 1.0, 1.0, 1.0
        for q, n, scale in ((RHO, 1, 0.1), (VX, 3, 0.1), (BX, 3, 1.0)):
            ks, phase, amp = _modes(rng, G.ndim, n == 3)
            for k, ph, a in zip(ks, phase, amp):
                wave = torch.cos(sum(2 * math.pi * int(k[d]) / (G.hi[d] - G.lo[d]) * c[d] for d in range(G.ndim)) + ph)
                for m in range(n):
                    p[:, q + m] += scale * float(a[m]) * wave
    return G, p


# ---------------------------------------------------------------------------
# passes


def _pool_jobs(case):
    """The resident jobs of a pool: `bz` grids from bx to by blocks a side."""
    n = case["bz"]
    sides = [int(round(case["bx"] * (case["by"] / case["bx"]) ** (j / max(1, n - 1)))) for j in range(n)]
    return [dict(case, kind="advance", bx=s, by=s, bz=s) for s in sides]


def _views(slot, nb, ndim, nx, ng, mixed, lead):
    """The interior of a state slot, as views on its memory: all variables,
    or the FP32 variables and the FP64 energy of a mixed slot."""
    pn = nx + 2 * ng
    pc, cells = pn ** ndim, (slice(ng, ng + nx),) * ndim
    if not mixed:
        return {"u": slot[lead:].view(torch.float64).view((nb, NV) + (pn,) * ndim)[(slice(None),) * 2 + cells]}
    raw = slot[:nb * 40 * pc].view(nb, 40 * pc)
    f = raw[:, :32 * pc].view(torch.float32).view((nb, 8) + (pn,) * ndim)
    e = raw[:, 32 * pc:].view(torch.float64).view((nb,) + (pn,) * ndim)
    return {"f": f[(slice(None),) * 2 + cells], "e": e[(slice(None),) + cells]}


def prepare(case, seed):
    dev = torch.device("cuda")
    precision = amrvac.FP32_MIXED if case["mixed"] else amrvac.FP64
    if case["kind"] == "pool":
        jobs = [_initial(j, seed + 1000 * n, dev) for n, j in enumerate(_pool_jobs(case))]
        ws = [G.workload(case) for G, _ in jobs]
        torch.cuda.synchronize()
        batch = amrvac.Batch(ws[0], sum(G.nb for G, _ in jobs), len(jobs), nstages=case["stages"],
                             precision=precision)
        for w, (_, p) in zip(ws, jobs):
            w.prim = p
            if batch.add_job(w, nsteps=1 << 30) is None:
                raise RuntimeError("the pool does not hold its jobs")
        batch.stream.synchronize()
        out = _views(batch.slots[0], batch.capacity, 3, 16, ws[0].ng, case["mixed"], amrvac.slot_lead(precision))
        return {"case": case, "batch": batch, "out": out, "stream": batch.stream}
    G, p = _initial(case, seed, dev)
    w = G.workload(case)
    path = amrvac.PATH_PLAIN if case["plain"] else amrvac.PATH_FUSED
    sim = amrvac.Simulation(w, precision=precision, path=path, set_initial=False)
    torch.cuda.synchronize()
    rc = sim.lib.amrvac_set_primitive(sim.ctx, 0, ctypes.c_void_p(p.data_ptr()))
    if rc:
        raise amrvac.AmrvacError(rc, "set_primitive")
    sim.synchronize()
    out = _views(sim.slots[0], G.nb, G.ndim, G.nx, G.ng, case["mixed"], amrvac.slot_lead(precision))
    return {"case": case, "sim": sim, "out": out, "stream": sim.stream}


def _snapshot(s):
    """A program's result of a pass.  FP64 states are used where they lie;
    FP32-mixed ones carry FP32 accuracy and are kept as one FP32 snapshot."""
    if "u" in s["out"]:
        return s["out"]["u"]
    f, e = s["out"]["f"], s["out"]["e"]
    with torch.cuda.stream(s["stream"]):
        return torch.cat([f[:, :PR], e[:, None].float(), f[:, PR:]], dim=1)


def run(s):
    case = s["case"]
    if case["kind"] == "pool":
        for _ in range(case["steps"]):
            s["batch"].step()
        return _snapshot(s)
    sim = s["sim"]
    if case["kind"] == "adapt":
        ind = sim.lohner(wavefilter=LOHNER_EPS)
        flags = np.where(ind > LOHNER_REFINE, 1, np.where(ind < LOHNER_COARSEN, -1, 0)).astype(np.int32)
        level, ijk = sim.regrid_plan(flags, max_level=case["levels"])
        new = sim.regrid(level, ijk)
        u = _views(new.slots[0], new.nb, sim.w.ndim, sim.w.nx, sim.w.ng, False, amrvac.slot_lead(amrvac.FP64))["u"]
        new.close()  # the state stays in its slots, which torch owns
        return {"indicator": ind, "level": level, "ijk": ijk, "u": u}
    if case["kind"] == "advance":
        sim.advance(case["steps"], case["stages"], graph=case["graph"])
        return _snapshot(s)
    for _ in range(case["steps"]):  # stage by stage, the next step's CFL rate folded into the last
        rows = {2: [(0, 0, 1, 1.0), (1, 0, 0, 0.5)],
                3: [(0, 0, 1, 1.0), (1, 0, 2, 0.25), (2, 0, 0, 2.0 / 3.0)]}[2 if case["stages"] == 2 else 3]
        sim.cfl(0)
        for n, (i, b, o, wt) in enumerate(rows):
            sim.fill(i)
            sim.stage(i, b, o, wt, cfl=n == len(rows) - 1)
    return _snapshot(s)


def _cells(case):
    if case["kind"] == "pool":
        return sum(_cells(j) for j in _pool_jobs(case))
    G = _Grid(case, "cpu")
    return G.nb * case["nx"] ** case["ndim"]


def work(case):
    """A step reads the state and writes the next one; per cell and stage the
    scheme takes a reconstruction of 9 variables on both sides of a face per
    direction (about 10 operations each, 75 for the five-cell ones), the
    interface flux (about 200, 300 for HLLD and HLLC) and 100 for the
    conversion, the update and the time step."""
    cells, state = _cells(case), 40 if case["mixed"] else 72
    if case["kind"] == "adapt":
        return {"bytes": 2.0 * 72 * cells, "flops": 30.0 * cells}
    recon = 75 if LIMITERS[case["limiter"]] >= 3 else 10
    flux = 200 if case["flux"] == "hll" else 300
    per = case["ndim"] * (18 * recon + flux) + 100
    return {"bytes": 2.0 * state * cells * case["steps"], "flops": float(per) * cells * case["steps"] * case["stages"]}


# ---------------------------------------------------------------------------
# the same scheme in plain torch, 64 bits

GAMMA, CFL, ALPHA = 5.0 / 3.0, 0.8, 0.5


def _cons(w):
    r, v, b = w[:, RHO], w[:, VX:VZ + 1], w[:, BX:BZ + 1]
    e = w[:, PR] / (GAMMA - 1) + 0.5 * r * (v * v).sum(1) + 0.5 * (b * b).sum(1)
    return torch.cat([r[:, None], r[:, None] * v, e[:, None], b, w[:, PSI:]], 1)


def _prim(u):
    r, m, b = u[:, RHO], u[:, VX:VZ + 1], u[:, BX:BZ + 1]
    p = (GAMMA - 1) * (u[:, PR] - 0.5 * (m * m).sum(1) / r - 0.5 * (b * b).sum(1))
    return torch.cat([r[:, None], m / r[:, None], p[:, None], b, u[:, PSI:]], 1)


def _fast(w, d):
    a2, b2 = GAMMA * w[:, PR] / w[:, RHO], (w[:, BX:BZ + 1] ** 2).sum(1) / w[:, RHO]
    s = a2 + b2
    return torch.sqrt(0.5 * (s + torch.sqrt((s * s - 4 * a2 * w[:, BX + d] ** 2 / w[:, RHO]).clamp(min=0))))


def _minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))


def _phi(name, r):
    """The limiter functions of the ratio of the differences."""
    if name == "koren":
        return torch.clamp(torch.minimum(torch.minimum(2 * r, (1 + 2 * r) / 3), torch.full_like(r, 2.0)), min=0)
    inner = torch.minimum(torch.minimum(2 * r, (2 + r) / 3), torch.full_like(r, 1.6))
    return torch.clamp(torch.minimum((2 + r) / 3, torch.maximum(-0.5 * r, inner)), min=0)


def _ratio(a, b):
    return torch.where(b != 0, a / torch.where(b != 0, b, torch.ones_like(b)), torch.zeros_like(a))


def _weno(name, m2, m1, z, p1, p2, lam):
    q = ((2 * m2 - 7 * m1 + 11 * z) / 6, (-m1 + 5 * z + 2 * p1) / 6, (2 * z + 5 * p1 - p2) / 6)
    b = (13 / 12 * (m2 - 2 * m1 + z) ** 2 + 0.25 * (m2 - 4 * m1 + 3 * z) ** 2,
         13 / 12 * (m1 - 2 * z + p1) ** 2 + 0.25 * (m1 - p1) ** 2,
         13 / 12 * (z - 2 * p1 + p2) ** 2 + 0.25 * (3 * z - 4 * p1 + p2) ** 2)
    d, tau, eps = (0.1, 0.6, 0.3), (b[0] - b[2]).abs(), 1e-40
    if name == "weno5":
        a = [d[k] / (1e-6 + b[k]) ** 2 for k in range(3)]
    elif name == "wenoz5":
        a = [d[k] * (1 + tau / (b[k] + eps)) for k in range(3)]
    else:
        a = [d[k] * (1 + (tau / (b[k] + eps)) ** 2 + lam * (b[k] + eps) / (tau + eps)) for k in range(3)]
    return (a[0] * q[0] + a[1] * q[1] + a[2] * q[2]) / (a[0] + a[1] + a[2])


def _mp5(m2, m1, z, p1, p2):
    def mm(*v):
        s = torch.stack(v)
        return torch.where((s > 0).all(0), s.amin(0), torch.where((s < 0).all(0), s.amax(0), torch.zeros_like(v[0])))

    u = (2 * m2 - 13 * m1 + 47 * z + 27 * p1 - 3 * p2) / 60
    ump = z + mm(p1 - z, 4 * (z - m1))
    dm, d0, dp = m2 - 2 * m1 + z, m1 - 2 * z + p1, z - 2 * p1 + p2
    cp, cm = mm(4 * d0 - dp, 4 * dp - d0, d0, dp), mm(4 * d0 - dm, 4 * dm - d0, d0, dm)
    ul, md, lc = z + 4 * (z - m1), 0.5 * (z + p1) - 0.5 * cp, z + 0.5 * (z - m1) + 4 / 3 * cm
    lo = torch.maximum(torch.minimum(torch.minimum(z, p1), md), torch.minimum(torch.minimum(z, ul), lc))
    hi = torch.minimum(torch.maximum(torch.maximum(z, p1), md), torch.maximum(torch.maximum(z, ul), lc))
    return torch.where((u - z) * (u - ump) <= 0, u, u + mm(lo - u, hi - u))


def _faces(name, c, lam):
    """Left and right states of the faces in the middle of four or six cells."""
    if name == "mp5":
        return _positive(_mp5(*c[:5]), _mp5(*c[:0:-1]), c[2], c[3])
    if len(c) == 6:
        return _positive(_weno(name, *c[:5], lam), _weno(name, *c[:0:-1], lam), c[2], c[3])
    m, a, b, p = c
    dm, d0, dp = a - m, b - a, p - b
    if name == "vanleer":
        def half(x, y):
            return torch.where(x * y > 0, x * y / torch.where(x + y != 0, x + y, torch.ones_like(x)), 0.0 * x)
        l, r = a + half(dm, d0), b - half(d0, dp)
    elif name == "koren":
        l, r = a + 0.5 * _phi(name, _ratio(d0, dm)) * dm, b - 0.5 * _phi(name, _ratio(d0, dp)) * dp
    else:
        l, r = a + 0.5 * _phi(name, _ratio(dm, d0)) * d0, b - 0.5 * _phi(name, _ratio(dp, d0)) * d0
    return _positive(l, r, a, b)


def _positive(l, r, a, b):
    bad = ~((l[:, RHO] > 0) & (l[:, PR] > 0) & (r[:, RHO] > 0) & (r[:, PR] > 0))[:, None]
    return torch.where(bad, a, l), torch.where(bad, b, r)


def _physical(w, u, d):
    """Flux along d (without the parts of B_n and psi)."""
    vn, bn = w[:, VX + d], w[:, BX + d]
    pt = w[:, PR] + 0.5 * (w[:, BX:BZ + 1] ** 2).sum(1)
    vb = (w[:, VX:VZ + 1] * w[:, BX:BZ + 1]).sum(1)
    f = u * vn[:, None]
    f[:, VX:VZ + 1] -= w[:, BX:BZ + 1] * bn[:, None]
    f[:, VX + d] += pt
    f[:, PR] += pt * vn - bn * vb
    f[:, BX:BZ + 1] -= w[:, VX:VZ + 1] * bn[:, None]
    return f


def _riemann(name, l, r, d, ch):
    N = BX + d
    t = [k for k in range(3) if k != d]
    bn = 0.5 * (l[:, N] + r[:, N]) - (r[:, PSI] - l[:, PSI]) / (2 * ch)
    ps = 0.5 * (l[:, PSI] + r[:, PSI]) - 0.5 * ch * (r[:, N] - l[:, N])
    l, r = l.clone(), r.clone()
    l[:, N], r[:, N] = bn, bn
    ul, ur = _cons(l), _cons(r)
    fl, fr = _physical(l, ul, d), _physical(r, ur, d)
    vl, vr, cl, cr = l[:, VX + d], r[:, VX + d], _fast(l, d), _fast(r, d)
    if name == "hlld":
        cm = torch.maximum(cl, cr)
        sl, sr = torch.minimum(vl, vr) - cm, torch.maximum(vl, vr) + cm
    else:
        sl, sr = torch.minimum(vl - cl, vr - cr), torch.maximum(vl + cl, vr + cr)
    S = lambda x: x[:, None]  # noqa: E731
    if name == "hll":
        f = (S(sr) * fl - S(sl) * fr + S(sl * sr) * (ur - ul)) / S(sr - sl)
    else:
        ptl, ptr = (w[:, PR] + 0.5 * (w[:, BX:BZ + 1] ** 2).sum(1) for w in (l, r))
        dl, dr = l[:, RHO] * (sl - vl), r[:, RHO] * (sr - vr)
        sm = (dr * vr - dl * vl - ptr + ptl) / (dr - dl)
        right = sm < 0
        if name == "hllc":
            pts = dl * (sm - vl) + ptl
            h = (S(sr) * ur - S(sl) * ul - fr + fl) / S(sr - sl)
        else:
            pts = (dr * ptl - dl * ptr + dl * dr * (vr - vl)) / (dr - dl)
        star = []
        for w, u, pt, vn, sa in ((l, ul, ptl, vl, sl), (r, ur, ptr, vr, sr)):
            s = torch.empty_like(u)
            rs = w[:, RHO] * (sa - vn) / (sa - sm)
            vs, bs = w[:, VX:VZ + 1].clone(), w[:, BX:BZ + 1].clone()
            vs[:, d] = sm
            if name == "hllc":
                for k in t:
                    vs[:, k], bs[:, k] = h[:, VX + k] / h[:, RHO], h[:, BX + k]
                vbs = (vs * bs).sum(1)
            else:
                den = w[:, RHO] * (sa - vn) * (sa - sm) - bn * bn
                deg = den.abs() <= 1e-12 * w[:, RHO] * (sa - vn) ** 2
                one = torch.where(deg, 1.0, den)
                for k in t:
                    vs[:, k] -= torch.where(deg, 0.0, bn * (sm - vn) / one) * w[:, BX + k]
                    bs[:, k] *= torch.where(deg, 1.0, (w[:, RHO] * (sa - vn) ** 2 - bn * bn) / one)
                vbs = (vs * bs).sum(1)
            vb = (w[:, VX:VZ + 1] * w[:, BX:BZ + 1]).sum(1)
            s[:, RHO] = rs
            if name == "hllc":  # tangential momentum from the jump across the outer wave
                for k in t:
                    s[:, VX + k] = (u[:, VX + k] * (sa - vn) + bn * (w[:, BX + k] - bs[:, k])) / (sa - sm)
                s[:, VX + d] = rs * sm
            else:
                s[:, VX:VZ + 1] = S(rs) * vs
            s[:, PR] = ((sa - vn) * u[:, PR] - pt * vn + pts * sm + bn * (vb - vbs)) / (sa - sm)
            s[:, BX:BZ + 1] = bs
            s[:, PSI] = u[:, PSI]
            star.append((s, vs, bs, vbs))
        fsl, fsr = fl + S(sl) * (star[0][0] - ul), fr + S(sr) * (star[1][0] - ur)
        if name == "hlld":
            ql, qr = torch.sqrt(star[0][0][:, RHO]), torch.sqrt(star[1][0][:, RHO])
            sg = torch.sign(bn)
            vss, bss = star[0][1].clone(), star[0][2].clone()
            for k in t:
                (a, b), (e, g) = (star[0][1][:, k], star[1][1][:, k]), (star[0][2][:, k], star[1][2][:, k])
                vss[:, k] = (ql * a + qr * b + (g - e) * sg) / (ql + qr)
                bss[:, k] = (ql * g + qr * e + ql * qr * (b - a) * sg) / (ql + qr)
            vbss = (vss * bss).sum(1)
            for side, (f, q, sgn) in enumerate(((fsl, ql, -1.0), (fsr, qr, 1.0))):
                s, _, _, vbs = star[side]
                ss = s.clone()
                ss[:, VX:VZ + 1] = S(s[:, RHO]) * vss
                ss[:, PR] = s[:, PR] + sgn * q * (vbs - vbss) * sg
                ss[:, BX:BZ + 1] = bss
                sa = sm + sgn * bn.abs() / q
                f.copy_(torch.where(S(sgn * sa > 0), f + S(sa) * (ss - s), f))
        f = torch.where(S(right), fsr, fsl)
    f = torch.where(S(sl >= 0), fl, torch.where(S(sr <= 0), fr, f))
    f[:, N], f[:, PSI] = ps, ch * ch * bn
    return f


class _Exact:
    """The scheme on padded blocks [block][var][(z)][y][x]."""

    def __init__(self, case, G):
        self.c, self.G = case, G
        n, ng, nd = G.nx, G.ng, G.ndim
        where = {(int(l),) + tuple(int(v) for v in p): b for b, (l, p) in enumerate(zip(G.level, G.ijk))}
        self.same, self.phys, self.fine, self.coarse = {}, {}, {}, {}
        for b in range(G.nb):
            l, p = int(G.level[b]), [int(v) for v in G.ijk[b]]
            for d in range(nd):
                for side in (0, 1):
                    q = list(p)
                    q[d] += 2 * side - 1
                    nblk = G.base[d] << (l - 1)
                    if not 0 <= q[d] < nblk:
                        bc = (G.bc_hi if side else G.bc_lo)[d]
                        if bc != PERIODIC:
                            self.phys.setdefault((d, side, bc), []).append(b)
                            continue
                        q[d] %= nblk
                    f = (d, side)
                    if (l,) + tuple(q) in where:
                        self.same.setdefault(f, []).append((b, where[(l,) + tuple(q)]))
                    elif (l - 1,) + tuple(v >> 1 for v in q) in where:
                        key = f + tuple(p[a] & 1 for a in range(nd))
                        self.coarse.setdefault(key, []).append((b, where[(l - 1,) + tuple(v >> 1 for v in q)]))
                    else:
                        for k in _children((l,) + tuple(q), nd):
                            o = [k[1 + a] & 1 for a in range(3)]
                            if o[d] == 1 - side:
                                key = f + tuple(o[a] for a in range(nd))
                                self.fine.setdefault(key, []).append((b, where[k]))
        as_idx = lambda v: torch.tensor(v, device=G.dev).T  # noqa: E731
        self.same, self.fine, self.coarse = ({k: as_idx(v) for k, v in t.items()}
                                             for t in (self.same, self.fine, self.coarse))
        self.idx = torch.from_numpy(1.0 / G.dx).to(G.dev)
        finest = G.dx[int(np.argmax(G.level))][:nd]
        self.sum_inv, self.min_dx = float((1 / finest).sum()), float(finest.min())
        self.inner = (slice(ng, ng + n),) * nd

    def at(self, **ax):
        """An index of padded arrays: per axis (0 x, 1 y, 2 z) a slice, the interior elsewhere."""
        G = self.G
        s = [slice(G.ng, G.ng + G.nx)] * G.ndim
        for k, v in ax.items():
            s[G.ndim - 1 - int(k[1:])] = v
        return (slice(None), slice(None)) + tuple(s)

    def pool(self, v, axes):
        """Mean of pairs along the given axes (0 x, ...)."""
        for a in axes:
            dim = v.dim() - 1 - a
            v = 0.5 * (v.narrow(dim, 0, v.shape[dim] - 1)[self.every(v.dim(), dim)]
                       + v.narrow(dim, 1, v.shape[dim] - 1)[self.every(v.dim(), dim)])
        return v

    @staticmethod
    def every(nd, dim):
        return tuple(slice(None, None, 2) if k == dim else slice(None) for k in range(nd))

    def put(self, U, blocks, ix, v):
        part = (blocks,) + ix[1:]
        U[part] = v

    def fill(self, U):
        G, n, ng, nd = self.G, self.G.nx, self.G.ng, self.G.ndim

        def ghost(side):
            return slice(ng + n, ng + n + ng) if side else slice(0, ng)

        for (d, side), (b, m) in self.same.items():
            src = slice(ng, 2 * ng) if side else slice(n, n + ng)
            self.put(U, b, self.at(**{"a%d" % d: ghost(side)}), U[(m,) + self.at(**{"a%d" % d: src})[1:]])
        for (d, side, bc), b in self.phys.items():
            b = torch.tensor(b, device=G.dev)
            if bc == FIXED:
                v = _cons(torch.from_numpy(G.fixed[d, side]).to(G.dev).view(1, NV, 1))[0]
                v = v.view((1, NV) + (1,) * nd)
            elif bc == ZEROGRAD:
                one = slice(ng + n - 1, ng + n) if side else slice(ng, ng + 1)
                v = U[(b,) + self.at(**{"a%d" % d: one})[1:]].repeat_interleave(ng, dim=2 + nd - 1 - d)
            else:
                src = slice(n, n + ng) if side else slice(ng, 2 * ng)
                v = U[(b,) + self.at(**{"a%d" % d: src})[1:]].flip(2 + nd - 1 - d)
                v[:, VX + d] *= -1
                v[:, BX + d] *= -1
            self.put(U, b, self.at(**{"a%d" % d: ghost(side)}), v)
        for key, (b, m) in self.fine.items():  # the mean of the fine cells under a coarse ghost cell
            (d, side), o = key[:2], key[2:]
            src = slice(ng, 3 * ng) if side else slice(ng + n - 2 * ng, ng + n)
            v = self.pool(U[(m,) + self.at(**{"a%d" % d: src})[1:]], range(nd))
            ax = {"a%d" % a: slice(ng + o[a] * n // 2, ng + (o[a] + 1) * n // 2) for a in range(nd)}
            ax["a%d" % d] = ghost(side)
            self.put(U, b, self.at(**ax), v)
        new = []
        for key, (b, m) in self.coarse.items():  # minmod-limited linear values from the coarse leaf
            (d, side), o = key[:2], key[2:]
            lay = (ng + 1) // 2
            lo = [ng + o[a] * n // 2 for a in range(nd)]
            hi = [lo[a] + n // 2 for a in range(nd)]
            lo[d], hi[d] = (ng, ng + lay) if side else (ng + n - lay, ng + n)

            def part(ax=None, s=0):
                return U[(m, slice(None)) + tuple(slice(lo[a] + s * (a == ax), hi[a] + s * (a == ax))
                                                  for a in reversed(range(nd)))]

            v = part()
            slopes = [_minmod(v - part(a, -1), part(a, 1) - v) for a in range(nd)]
            for a in range(nd):
                dim = 2 + nd - 1 - a
                v = v.repeat_interleave(2, dim)
                slopes = [s.repeat_interleave(2, dim) for s in slopes]
            for a in range(nd):
                dim = 2 + nd - 1 - a
                sg = torch.tensor([-0.25, 0.25], device=G.dev, dtype=U.dtype).repeat(v.shape[dim] // 2)
                v = v + slopes[a] * sg.view([-1 if k == dim else 1 for k in range(v.dim())])
            dim = 2 + nd - 1 - d
            v = v.narrow(dim, 0, ng) if side else v.narrow(dim, v.shape[dim] - ng, ng)
            new.append((b, self.at(**{"a%d" % d: ghost(side)}), v))
        for b, ix, v in new:
            self.put(U, b, ix, v)

    def rate(self, U):
        w = _prim(U[self.at()])
        k = self.idx.view((-1, 3) + (1,) * self.G.ndim)
        r = sum((w[:, VX + d].abs() + _fast(w, d)) * k[:, d] for d in range(self.G.ndim))
        dt = CFL / float(r.max())
        ch = CFL / (dt * self.sum_inv)
        return dt, ch, ALPHA * ch / self.min_dx

    def fluxes(self, U, d, ch):
        """Face fluxes along d, [block][var] with nx + 1 faces along that axis."""
        G, n, ng = self.G, self.G.nx, self.G.ng
        dim = 2 + G.ndim - 1 - d
        out = []
        name = self.c["limiter"]
        for b0 in range(0, G.nb, 512):
            u = U[b0:b0 + 512][self.at(**{"a%d" % d: slice(None)})]
            w = _prim(u)
            lam = torch.from_numpy(G.dx[b0:b0 + 512, d] ** (2.0 / 3.0)).to(G.dev).view([-1] + [1] * (w.dim() - 1))
            l, r = _faces(name, [w.narrow(dim, s, n + 1) for s in range(2 * ng)], lam)
            out.append(_riemann(self.c["flux"], l, r, d, ch))
        return torch.cat(out)

    def rhs(self, U, ch, kappa):
        """-(flux differences) - kappa psi on the interior; fills U's ghost cells."""
        G, n, nd = self.G, self.G.nx, self.G.ndim
        self.fill(U)
        L = torch.zeros_like(U[self.at()])
        for d in range(nd):
            dim = 2 + nd - 1 - d
            F = self.fluxes(U, d, ch)
            for key, (b, m) in self.fine.items():
                if key[0] != d:
                    continue
                side, o = key[1], key[2:]
                sub = F[m].narrow(dim, 0 if side else n, 1)
                v = self.pool(sub, [a for a in range(nd) if a != d])
                ix = [slice(o[a] * n // 2, (o[a] + 1) * n // 2) for a in range(nd)]
                ix[d] = slice(n, n + 1) if side else slice(0, 1)
                F[(b, slice(None)) + tuple(reversed(ix))] = v
            k = self.idx[:, d].view([-1] + [1] * (L.dim() - 1))
            L -= (F.narrow(dim, 1, n) - F.narrow(dim, 0, n)) * k
            del F
        L[:, PSI] -= kappa * U[self.at()][:, PSI]
        return L

    def padded(self, u):
        G = self.G
        U = torch.full((G.nb, NV) + (G.nx + 2 * G.ng,) * G.ndim, 1.0, device=G.dev, dtype=torch.float64)
        U[self.at()] = u
        return U

    def step(self, u, stages):
        U = self.padded(u)
        dt, ch, kap = self.rate(U)

        def euler(v, h):
            U[self.at()] = v
            return v + h * dt * self.rhs(U, ch, kap)

        if stages == 2:
            return 0.5 * (u + euler(euler(u, 1.0), 1.0))
        if stages == 3:
            u2 = 0.75 * u + 0.25 * euler(euler(u, 1.0), 1.0)
            return u / 3 + 2.0 / 3.0 * euler(u2, 1.0)
        if stages == 4:
            u2 = euler(euler(u, 0.5), 0.5)
            return euler(2.0 / 3.0 * u + 1.0 / 3.0 * euler(u2, 0.5), 0.5)
        u1 = euler(u, 0.391752226571890)
        u2 = 0.444370493651235 * u + 0.555629506348765 * euler(u1, 0.368410593050371 / 0.555629506348765)
        u3 = 0.620101851488403 * u + 0.379898148511597 * euler(u2, 0.251891774271694 / 0.379898148511597)
        U[self.at()] = u3
        L3 = dt * self.rhs(U, ch, kap)
        u4 = 0.178079954393132 * u + 0.821920045606868 * u3 + 0.544974750228521 * L3
        U[self.at()] = u4
        L4 = dt * self.rhs(U, ch, kap)
        return (0.517231671970585 * u2 + 0.096059710526147 * u3 + 0.063692468666290 * L3
                + 0.386708617503269 * u4 + 0.226007483236906 * L4)


def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "pool":
        out = []
        for n, j in enumerate(_pool_jobs(case)):
            G, p = _initial(j, seed + 1000 * n, dev)
            X, u = _Exact(j, G), _cons(p)
            for _ in range(case["steps"]):
                u = X.step(u, case["stages"])
            out.append(u)
        return torch.cat(out)
    G, p = _initial(case, seed, dev)
    X, u = _Exact(case, G), _cons(p)
    del p
    if case["kind"] == "adapt":
        U = X.padded(u)
        X.fill(U)
        num, den, b = 0.0, 0.0, U[X.at()][:, RHO]
        for d in range(G.ndim):
            a, e = (U[X.at(**{"a%d" % d: slice(G.ng + s, G.ng + G.nx + s)})][:, RHO] for s in (-1, 1))
            num = num + (a - 2 * b + e) ** 2
            den = den + ((e - b).abs() + (b - a).abs() + LOHNER_EPS * (e.abs() + 2 * b.abs() + a.abs())) ** 2
        ind = torch.sqrt(num / den).flatten(1).amax(1)
        return {"indicator": ind.cpu().numpy(), "level": None, "ijk": None, "u": None}
    stages = case["stages"] if case["kind"] == "advance" else (2 if case["stages"] == 2 else 3)
    for _ in range(case["steps"]):
        u = X.step(u, stages)
    return u
