"""The workloads this library's speed is measured on.

listed() names them, draw() gives more of the same ranges, prepare() makes what
a simulation holds before the call (tree, state, plan), run() is one pass
through the Python binding, and exact() computes the same results in plain
torch, in 64 bits and with none of the library's code: its own oct lists,
neighbour search, MUSCL-Hancock/HLLC update and multigrid cycles.

Families ("what"):
  step       one step of a tree, one time step for all levels (DeviceTree.step)
  subcycle   one coarse step with level subcycling (DeviceTree.run_subcycled)
  batch      many boxes advanced by one graph launch (Batch.run)
  refine     flags, closure, new oct list, state gather, hash, lists, schedule
             (DeviceTree.refine)
  poisson    V-cycles on a periodic unigrid (Multigrid)
  levels     V-cycles level by level on an AMR tree (mg_solve_levels)
"""
import functools
import math

import torch

from paper_2607_20704_amd import api

CFL = 0.8
OUT = -(1 << 31)
FORMS = {"fp64": api.RG_FP64, "mixed": api.RG_MIXED}
RHO_MIN, P_MIN = 1e-10, 1e-20


def listed():
    return [
        # the smallest call: a 32^3 shock tube, 4096 octs, time step found first
        {"name": "sod_32_fp64", "what": "step", "tree": "uniform", "base": 5, "lmax": 5, "bc": "outflow",
         "gas": "sod", "form": "fp64", "lists": "kept", "chain": False, "ghost": 0},
        # an ordinary box in a time loop: lists kept, each time step folded into the update before
        {"name": "turbulent_128_mixed", "what": "step", "tree": "uniform", "base": 7, "lmax": 7, "bc": "periodic",
         "gas": "turbulent", "form": "mixed", "lists": "kept", "chain": True, "ghost": 0},
        # the large box of the benchmark, hash table and neighbour lists rebuilt every step, both forms
        {"name": "turbulent_256_fp64", "what": "step", "tree": "uniform", "base": 8, "lmax": 8, "bc": "periodic",
         "gas": "turbulent", "form": "fp64", "lists": "rebuilt", "chain": True, "ghost": 0},
        {"name": "turbulent_256_mixed", "what": "step", "tree": "uniform", "base": 8, "lmax": 8, "bc": "periodic",
         "gas": "turbulent", "form": "mixed", "lists": "rebuilt", "chain": True, "ghost": 0},
        # a blast on a graded tree, levels 6-8, coordinates re-keyed and sorted every step (a tree that moves)
        {"name": "sedov_6_8_fp64", "what": "step", "tree": "sphere", "base": 6, "lmax": 8, "bc": "periodic",
         "gas": "sedov", "form": "fp64", "lists": "rekeyed", "chain": True, "ghost": 0, "fill": 0.0141},
        # the same tree advanced by level subcycling
        {"name": "sedov_6_8_subcycle", "what": "subcycle", "tree": "sphere", "base": 6, "lmax": 8, "bc": "periodic",
         "gas": "sedov", "form": "mixed", "ghost": 0, "fill": 0.0141},
        # clumpy gas on a deep tree, levels 7-11, about 8 M cells
        {"name": "clumps_7_11_fp64", "what": "step", "tree": "clumps", "base": 7, "lmax": 11, "bc": "periodic",
         "gas": "clumps", "form": "fp64", "lists": "kept", "chain": True, "ghost": 0, "fill": 0.0006, "layout": 0},
        # clumpy gas subcycled, coarse ghost cells interpolated
        {"name": "clumps_6_9_subcycle", "what": "subcycle", "tree": "clumps", "base": 6, "lmax": 9, "bc": "periodic",
         "gas": "clumps", "form": "mixed", "ghost": 1, "fill": 0.01, "layout": 0},
        # 64 uneven boxes (16^3-128^3 cells, 0-2 extra levels; tubes, blasts, turbulence), two steps a launch
        {"name": "boxes_64_fp64", "what": "batch", "boxes": 64, "base": 7, "form": "fp64", "lists": "kept",
         "steps": 2},
        # one tree change of a deep tree, as between two steps
        {"name": "refine_7_11", "what": "refine", "tree": "clumps", "base": 7, "lmax": 11, "bc": "periodic",
         "gas": "clumps", "fill": 0.0006, "layout": 0, "blocks": 2},
        # self-gravity on the large box: four V-cycles from zero
        {"name": "poisson_256", "what": "poisson", "base": 8, "cycles": 4},
        # self-gravity level by level on the blast's tree: four V-cycles a level
        {"name": "levels_6_8", "what": "levels", "tree": "sphere", "base": 6, "lmax": 8, "bc": "periodic",
         "fill": 0.0141, "cycles": 4},
    ]


def draw(rng):
    what = rng.choice(["step", "step", "step", "subcycle", "batch", "refine", "poisson", "levels"])
    form = rng.choice(["fp64", "mixed"])
    c = {"what": what}
    if what == "batch":
        return {**c, "boxes": round(math.exp(rng.uniform(math.log(3), math.log(64)))), "base": rng.randint(5, 7),
                "form": form, "lists": rng.choice(["kept", "rebuilt"]), "steps": rng.choice([2, 4])}
    if what == "poisson":
        return {**c, "base": rng.randint(4, 8), "cycles": rng.randint(1, 4)}
    if what == "step" and rng.random() < 0.4:
        gas = rng.choice(["sod", "turbulent"])
        base = rng.randint(4, 8)
        return {**c, "tree": "uniform", "base": base, "lmax": base, "bc": "outflow" if gas == "sod" else "periodic",
                "gas": gas, "form": form, "lists": rng.choice(["kept", "rebuilt", "rekeyed"]),
                "chain": rng.random() < 0.6, "ghost": 0}
    base = rng.randint(4, 7)
    lmax = min(base + rng.randint(1, 4), 9 if what == "levels" else 11)
    if what == "subcycle":
        lmax = min(lmax, base + 3)
    # volume of the finest level: a few thousand to a few million cells
    cells = math.exp(rng.uniform(math.log(2e3), math.log(4e6 if what == "step" else 1e6)))
    fill = round(min(0.05, cells / 8.0 ** lmax), 9)
    c.update(tree=rng.choice(["sphere", "clumps"]), base=base, lmax=lmax, bc="periodic", fill=fill,
             layout=rng.randint(0, 999))
    if what == "levels":
        return {**c, "cycles": rng.randint(1, 4)}
    c["gas"] = "sedov" if c["tree"] == "sphere" else "clumps"
    if what == "refine":
        return {**c, "tree": "clumps", "gas": "clumps", "blocks": rng.choice([2, 2, 4])}
    c.update(form=form, ghost=rng.randint(0, 1))
    if c["tree"] == "sphere" and rng.random() < 0.3:
        c.update(gas="sod", bc="outflow")
    if what == "step":
        c.update(lists=rng.choice(["kept", "rebuilt", "rekeyed"]), chain=rng.random() < 0.6)
    return c


def gamma_of(gas):
    return 1.4 if gas in ("sod", "sedov") else 5.0 / 3.0


# --------------------------------------------------------------------------
# trees and states (plain torch)
# --------------------------------------------------------------------------

def device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def rows(n):
    return torch.arange(n, dtype=torch.int64, device=device())


def code(i, j, k, n):
    return (k * n + j) * n + i


def uncode(c, n):
    return c % n, (c // n) % n, c // (n * n)


def cells_of(octs, level):
    """Coordinates (3 x [n, 8]) of the cells of the octs with these codes."""
    b = rows(8)
    return [2 * p[:, None] + ((b >> a) & 1) for a, p in enumerate(uncode(octs, 1 << (level - 1)))]


def curve_keys(i, j, k, level):
    """Position along Skilling's Hilbert curve of level-1 bits, behind a leading one."""
    nb = level - 1
    x = [i.clone(), j.clone(), k.clone()]
    for b in range(nb - 1, 0, -1):
        q, low = 1 << b, (1 << b) - 1
        for a in range(3):
            up = (x[a] & q) != 0
            d = torch.where(up, torch.zeros_like(x[0]), (x[0] ^ x[a]) & low)
            first = torch.where(up, x[0] ^ low, x[0] ^ d)
            if a:
                x[a] = x[a] ^ d
            x[0] = first
    x[1] ^= x[0]
    x[2] ^= x[1]
    flip = torch.zeros_like(x[0])
    for b in range(nb - 1, 0, -1):
        flip = torch.where((x[2] & (1 << b)) != 0, flip ^ ((1 << b) - 1), flip)
    h = torch.full_like(x[0], 1 << (3 * nb))
    for b in range(nb):
        for a in range(3):
            h += (((x[a] ^ flip) >> b) & 1) << (3 * b + 2 - a)
    return h


def geometry(case):
    """Centres, radii and amplitudes of the refined regions: the case's own, so that every seed has the same tree."""
    g = torch.Generator().manual_seed(case.get("layout", 0) * 7919 + 13)
    n = 1 if case["tree"] == "sphere" else 24
    centre = torch.rand((n, 3), generator=g, dtype=torch.float64)
    size = torch.exp(0.5 * torch.randn(n, generator=g, dtype=torch.float64))
    if case["tree"] == "sphere":
        centre[:] = 0.5
        size[:] = 1.0
    radius = size * (case["fill"] / (4.0 / 3.0 * math.pi * (size ** 3).sum())) ** (1.0 / 3.0)
    amp = 12.0 + 20.0 * torch.rand(n, generator=g, dtype=torch.float64)
    return centre.to(device()), radius.to(device()), amp.to(device())


def distance2(x, centre):
    d = x[:, None, :] - centre[None]
    d = d - torch.round(d)
    return (d * d).sum(-1)


def clump_density(x, geo):
    """Background 1 and Gaussian clumps that reach 8 at their radius."""
    centre, radius, amp = geo
    rho = torch.ones(len(x), dtype=torch.float64, device=x.device)
    for b in range(0, len(x), 1 << 20):
        r2 = distance2(x[b:b + (1 << 20)], centre) / (radius * radius)
        rho[b:b + (1 << 20)] += (amp * torch.exp(-r2 * torch.log(amp / 7.0))).sum(1)
    return rho


class Mesh:
    """Octs of a graded tree in key order with their links, in plain torch."""

    def __init__(self, levels, periodic):
        self.periodic = periodic
        self.lmin, self.lmax = min(levels), max(levels)
        self.begin, self.codes, self.rank, parts = {}, {}, {}, []
        n = 0
        for l in sorted(levels):
            c = levels[l]
            ijk = uncode(c, 1 << (l - 1))
            order = torch.argsort(curve_keys(*ijk, l))
            self.begin[l] = n
            self.codes[l] = c                                  # ascending
            self.rank[l] = torch.empty_like(order)             # code position -> oct
            self.rank[l][order] = n + rows(len(c))
            parts.append(torch.stack([p[order] for p in ijk] + [torch.full_like(c, l)], 1))
            n += len(c)
        self.begin[self.lmax + 1] = n
        self.ijkl = torch.cat(parts)
        self.n = n
        self.split = torch.zeros(8 * n, dtype=torch.bool, device=device())
        self.father = torch.full((n,), -1, dtype=torch.int64, device=device())
        for l in range(self.lmin + 1, self.lmax + 1):
            p = self.ijkl[self.begin[l]:self.begin[l + 1]]
            f = 8 * self.find(l - 1, p[:, 0] >> 1, p[:, 1] >> 1, p[:, 2] >> 1)
            f = f + (p[:, 0] & 1) + 2 * (p[:, 1] & 1) + 4 * (p[:, 2] & 1)
            self.father[self.begin[l]:self.begin[l + 1]] = f
            self.split[f] = True

    def find(self, l, i, j, k):
        """Oct index, -1 where there is none (coordinates inside the box)."""
        want = code(i, j, k, 1 << (l - 1))
        pos = torch.searchsorted(self.codes[l], want).clamp(max=len(self.codes[l]) - 1)
        return torch.where(self.codes[l][pos] == want, self.rank[l][pos], torch.full_like(want, -1))

    def octs(self, l):
        return slice(self.begin[l], self.begin[l + 1])

    def cells(self, l):
        return slice(8 * self.begin[l], 8 * self.begin[l + 1])

    def centres(self):
        b = rows(8)
        sub = torch.stack([(b >> a) & 1 for a in range(3)], 1)
        h = torch.exp2(-self.ijkl[:, 3:].double())
        return ((2 * self.ijkl[:, None, :3] + sub).double() + 0.5).mul(h[:, :, None]).reshape(-1, 3)

    def fill_split(self, u):
        for l in range(self.lmax, self.lmin, -1):
            u[self.father[self.octs(l)]] = u[self.cells(l)].view(-1, 8, u.shape[1]).mean(1)
        return u

    def neighbours(self, l, octs):
        """[m, 27]: oct, -1 - (coarse cell), or OUT outside the box."""
        p = self.ijkl[octs]
        n = 1 << (l - 1)
        out = torch.empty((len(p), 27), dtype=torch.int64, device=p.device)
        for s in range(27):
            q = [p[:, 0] + s % 3 - 1, p[:, 1] + s // 3 % 3 - 1, p[:, 2] + s // 9 - 1]
            outside = torch.zeros(len(p), dtype=torch.bool, device=p.device)
            if not self.periodic:
                for a in range(3):
                    outside |= (q[a] < 0) | (q[a] >= n)
            q = [v % n for v in q]
            e = self.find(l, *q)
            if l > self.lmin:
                f = 8 * self.find(l - 1, *[v >> 1 for v in q])
                f = f + (q[0] & 1) + 2 * (q[1] & 1) + 4 * (q[2] & 1)
                e = torch.where(e < 0, -1 - f, e)
            out[:, s] = torch.where(outside, torch.full_like(e, OUT), e)
        return out


def tree_levels(case):
    base, lmax, periodic = case["base"], case["lmax"], case["bc"] == "periodic"
    levels = {base: rows(8 ** (base - 1))}
    if lmax == base:
        return levels
    geo = geometry(case)
    for _ in range(8):
        before = {l: len(v) for l, v in levels.items()}
        for l in range(base, lmax):
            if l not in levels:
                break
            c = cells_of(levels[l], l)
            flat = [v.reshape(-1) for v in c]
            x = (torch.stack(flat, 1).double() + 0.5) * 0.5 ** l
            if case["tree"] == "sphere":
                inside = (distance2(x, geo[0]) < geo[1] * geo[1]).any(1)
                # the blast's centre is refined whatever the sphere's size
                inside |= ((x - 0.5).abs() < 0.75 * 0.5 ** l).all(1)
            else:
                inside = clump_density(x, geo) > 8.0
            new = code(*[v[inside] for v in flat], 1 << l)
            if len(new) or l + 1 in levels:
                levels[l + 1] = torch.unique(torch.cat([levels.get(l + 1, rows(0)), new]))
        # grading: a split cell has its 26 neighbours at its own level
        for l in range(max(levels) - 1, base, -1):
            f = uncode(levels[l + 1], 1 << l)      # an oct's coordinates are its father cell's
            need = [levels[l]]
            for s in range(27):
                q = [f[0] + s % 3 - 1, f[1] + s // 3 % 3 - 1, f[2] + s // 9 - 1]
                if periodic:
                    q = [v % (1 << l) for v in q]
                else:
                    keep = torch.ones(len(f[0]), dtype=torch.bool, device=f[0].device)
                    for v in q:
                        keep &= (v >= 0) & (v < (1 << l))
                    q = [v[keep] for v in q]
                need.append(torch.unique(code(*[v >> 1 for v in q], 1 << (l - 1))))
            levels[l] = torch.unique(torch.cat(need))
        if {l: len(v) for l, v in levels.items()} == before:
            break
    return levels


def mesh_of(case):
    return Mesh(tree_levels(case), case["bc"] == "periodic")


def noise_fields(n, seed, count):
    """Gaussian fields with |f(k)|^2 ~ k^-4, zero mean, unit variance, [z, y, x]."""
    g = torch.Generator(device=device()).manual_seed(int(seed) * 31 + 5)
    k = torch.fft.fftfreq(n, dtype=torch.float64, device=device()) * n
    kr = torch.fft.rfftfreq(n, dtype=torch.float64, device=device()) * n
    kk = torch.sqrt(k[:, None, None] ** 2 + k[None, :, None] ** 2 + kr[None, None, :] ** 2)
    amp = torch.where((kk >= 1.0) & (kk <= n / 2), kk.clamp(min=1.0) ** -2.0, torch.zeros_like(kk))
    out = []
    for _ in range(count):
        w = torch.randn((n, n, n), generator=g, dtype=torch.float64, device=device())
        f = torch.fft.irfftn(torch.fft.rfftn(w) * amp, s=(n, n, n))
        f = f - f.mean()
        out.append(f / f.std(unbiased=False))
    return out


def conserved(rho, vel, p, gamma):
    e = p / (gamma - 1.0) + 0.5 * rho * (vel[0] ** 2 + vel[1] ** 2 + vel[2] ** 2)
    return torch.stack([rho] + [rho * v for v in vel] + [e], 1)


def state_of(case, mesh, seed):
    """Conserved variables of every cell, key order, split cells averaged."""
    gas, gamma = case["gas"], gamma_of(case["gas"])
    x = mesh.centres()
    g = torch.Generator().manual_seed(int(seed) * 104729 + 17)
    r = torch.rand(12, generator=g, dtype=torch.float64).tolist()
    zero = torch.zeros(len(x), dtype=torch.float64, device=x.device)
    if gas == "sod":       # a tube: the pressures vary a little with the seed
        left = x[:, 0] < 0.5
        rho = torch.where(left, zero + 1.0, zero + 0.125)
        p = torch.where(left, zero + (0.9 + 0.2 * r[0]), zero + (0.09 + 0.02 * r[1]))
        u = conserved(rho, (zero, zero, zero), p, gamma)
    elif gas == "sedov":   # a point blast: energy in the finest cells around the centre
        h = 0.5 ** mesh.lmax
        near = ((x - 0.5).abs() < 0.75 * h).all(1)
        near[:8 * mesh.begin[mesh.lmax]] = False
        u = conserved(zero + 1.0, (zero, zero, zero), zero + 1e-5, gamma)
        u[:, 4] = torch.where(near, zero + (0.8 + 0.4 * r[0]) / 8.0 / h ** 3, u[:, 4])
    elif gas == "turbulent":   # lognormal density, k^-2 velocities at Mach 2
        n = 1 << case["base"]
        f = noise_fields(n, seed, 4)
        rho = torch.exp(0.5 * f[0] - 0.125)
        rms = torch.sqrt((f[1] ** 2 + f[2] ** 2 + f[3] ** 2).mean())
        scale = 2.0 * math.sqrt(gamma) / rms
        c = (x * n).long().clamp(max=n - 1)
        at = (c[:, 2] * n + c[:, 1]) * n + c[:, 0]
        vel = [(v * scale).reshape(-1)[at] for v in f[1:]]
        u = conserved(rho.reshape(-1)[at], vel, zero + 1.0, gamma)
    else:                  # clumps of gas in a slow shear
        rho = clump_density(x, geometry(case))
        two_pi = 2.0 * math.pi
        vel = [0.3 * torch.sin(two_pi * (x[:, (a + 1) % 3] + r[a])) + 0.2 * torch.cos(two_pi * (x[:, a] + r[3 + a]))
               for a in range(3)]
        u = conserved(rho, vel, (0.9 + 0.2 * r[6]) * rho ** gamma, gamma)
    return mesh.fill_split(u).contiguous()


def box_cases(case):
    """The boxes of a batch: uneven levels, three kinds of gas."""
    g = torch.Generator().manual_seed(case["boxes"] * 17 + case["base"])
    out = []
    for b in range(case["boxes"]):
        base = int(torch.randint(4, case["base"] + 1, (1,), generator=g))
        extra = int(torch.randint(0, 3, (1,), generator=g))
        radius = 0.1 + 0.15 * float(torch.rand(1, generator=g))
        gas = ("sod", "sedov", "turbulent")[b % 3]
        if gas == "turbulent":
            extra = 0
        out.append({"tree": "sphere" if extra else "uniform", "base": base, "lmax": base + extra, "gas": gas,
                    "bc": "outflow" if gas == "sod" else "periodic", "fill": 4.0 / 3.0 * math.pi * radius ** 3})
    return out


def right_side(mesh, seed):
    """Right-hand side of the Poisson problem per cell, zero mean on the base."""
    g = torch.Generator(device=device()).manual_seed(int(seed) * 53 + 3)
    f = torch.randn(8 * mesh.n, generator=g, dtype=torch.float64, device=device())
    f[mesh.cells(mesh.lmin)] -= f[mesh.cells(mesh.lmin)].mean()
    return f


def host_octs(mesh):
    """Octs as a program lists them: level by level, x fastest."""
    parts = []
    for l in range(mesh.lmin, mesh.lmax + 1):
        c = mesh.codes[l]
        parts.append(torch.stack(list(uncode(c, 1 << (l - 1))) + [torch.full_like(c, l)], 1))
    return torch.cat(parts).to(torch.int32).cpu().numpy()


# --------------------------------------------------------------------------
# the measured passes
# --------------------------------------------------------------------------

def prepare(case, seed):
    what = case["what"]
    s = {"case": case}
    if what == "poisson":
        mg = api.Multigrid(case["base"])
        mesh = mesh_of({**case, "lmax": case["base"], "bc": "periodic", "tree": "uniform"})
        mg.f[mg.fine] = right_side(mesh, seed)
        return {**s, "mg": mg}
    if what == "batch":
        boxes = box_cases(case)
        meshes = [mesh_of(b) for b in boxes]
        trees = [api.DeviceTree(host_octs(m), bc_of(b)) for b, m in zip(boxes, meshes)]
        states = [state_of(b, m, seed + n) for n, (b, m) in enumerate(zip(boxes, meshes))]
        batch = api.Batch(trees, states, [gamma_of(b["gas"]) for b in boxes], [CFL] * len(boxes), case["steps"],
                          form=FORMS[case["form"]], rebuild=case["lists"] == "rebuilt")
        return {**s, "batch": batch}
    mesh = mesh_of(case)
    tree = api.DeviceTree(host_octs(mesh), bc_of(case), ghost=case.get("ghost", 0),
                          capacity=mesh.n * 5 // 4 if what == "refine" else None)
    s["tree"] = tree
    if what == "levels":
        f = right_side(mesh, seed)
        _, levels = api.mg_solve_levels(tree, f, 0)
        return {**s, "f": f, "levels": levels}
    u = state_of(case, mesh, seed)
    s["gamma"] = gamma_of(case["gas"])
    if what == "refine":
        # the tree its own state asks for: the criterion reads the averages of split cells, so a few passes settle it
        other = torch.empty((8 * tree.capacity, 5), dtype=torch.float64, device=u.device)
        s["spare"] = torch.empty_like(other)
        for _ in range(6):
            n = tree.n
            keys = tree.keys.view(torch.int64).clone()
            u = tree.refine(u, rho_thresh=8.0, lmax=case["lmax"], out=other, nsubgrid=case["blocks"]).clone()
            if tree.n == n and torch.equal(tree.keys.view(torch.int64), keys):
                break
        return {**s, "u": u}
    s["u"] = u
    if what == "step":
        s["out"] = torch.empty_like(u)
        s["dt"] = torch.zeros(2, dtype=torch.float64, device=u.device)
        api.cfl_dt(u, tree.son_mask, tree.level_begin, tree.lmin, tree.lmax, s["gamma"], CFL, s["dt"][:1])
    return s


def bc_of(case):
    return api.RG_BC_OUTFLOW if case["bc"] == "outflow" else api.RG_BC_PERIODIC


def run(s):
    case = s["case"]
    what = case["what"]
    if what == "poisson":
        mg = s["mg"]
        mg.phi.zero_()
        mg.vcycles(case["cycles"])
        return {"phi": mg.phi[mg.fine], "residual": mg.residual()}
    if what == "batch":
        b = s["batch"]
        b.run()
        return {"dt": b.dts(), "u": [b.state(t) for t in range(min(case["boxes"], 60))]}
    tree = s["tree"]
    if what == "levels":
        return api.mg_solve_levels(tree, s["f"], case["cycles"], levels=s["levels"])[0]
    if what == "refine":
        u = tree.refine(s["u"], rho_thresh=8.0, lmax=case["lmax"], out=s["spare"], nsubgrid=case["blocks"])
        return {"u": u, "keys": tree.keys.view(torch.int64), "lists": tree.nbr27, "father": tree.father_cell,
                "son": tree.son_mask}
    if what == "subcycle":
        u, dts = tree.run_subcycled(s["u"], s["gamma"], CFL, 1, form=FORMS[case["form"]])
        return {"u": u, "dt": dts}
    if case["lists"] == "rebuilt":
        tree.prepare(api.RG_STEP_REBUILD)
    tree.step(s["u"], s["out"], s["gamma"], CFL, FORMS[case["form"]], rebuild=case["lists"] == "rekeyed",
              dt=s["dt"], chain=case["chain"])
    return {"u": s["out"], "dt": s["dt"] if case["chain"] else s["dt"][:1]}


@functools.lru_cache(maxsize=None)
def octs_by_level(text):
    case = dict(text)
    return tuple((l, len(v)) for l, v in tree_levels(case).items())


def size_of(case):
    """{level: octs} of the case's tree."""
    keys = ("tree", "base", "lmax", "bc", "fill", "layout")
    return dict(octs_by_level(tuple((k, case[k]) for k in keys if k in case)))


def work(case):
    """State read and written once (80 bytes a cell), the keys where lists are rebuilt; about 650 operations a cell."""
    what = case["what"]
    if what == "poisson":
        n = 8 ** case["base"]   # phi written, f read, residual written; 12 operations a cell and sweep
        return {"bytes": 24 * n, "flops": n * (case["cycles"] * (4 * 9 + 30) * 8 // 7 + 9)}
    if what == "batch":
        n = sum(8 * sum(size_of(b).values()) for b in box_cases(case))
        return {"bytes": 80 * n * case["steps"], "flops": 650 * n * case["steps"]}
    octs = size_of(case)
    n = 8 * sum(octs.values())
    if what == "levels":
        return {"bytes": 16 * n, "flops": n * case["cycles"] * 80}
    if what == "refine":
        return {"bytes": (80 + 14) * n, "flops": 2 * n}
    if what == "subcycle":
        n = sum(8 * m * 2 ** (l - case["base"]) for l, m in octs.items())
        return {"bytes": 80 * n, "flops": 650 * n}
    per_oct = {"kept": 0, "rebuilt": 8, "rekeyed": 16}[case["lists"]]
    return {"bytes": 80 * n + per_oct * n // 8, "flops": 650 * n}


# --------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# --------------------------------------------------------------------------

def exact(case, seed):
    what = case["what"]
    if what == "refine":
        return None     # lists of whole numbers and copied states: nothing is computed
    if what == "poisson":
        return exact_poisson(case, seed)
    if what == "batch":
        us, dts = [], []
        for n, b in enumerate(box_cases(case)):
            mesh = mesh_of(b)
            u = state_of(b, mesh, seed + n)
            gamma, row = gamma_of(b["gas"]), []
            for _ in range(case["steps"]):
                row.append(time_step(mesh, u, gamma))
                u = tree_step(mesh, u, row[-1], gamma, 0)
            us.append(u)
            dts.append(torch.stack(row))
        return {"dt": torch.stack(dts, 1), "u": us[:60]}
    mesh = mesh_of(case)
    if what == "levels":
        return exact_levels(case, mesh, right_side(mesh, seed))
    u = state_of(case, mesh, seed)
    gamma = gamma_of(case["gas"])
    if what == "subcycle":
        dt = time_step(mesh, u, gamma, sub=True)
        return {"u": tree_subcycled(mesh, u, dt, gamma, case["ghost"]), "dt": dt.reshape(1)}
    dt = time_step(mesh, u, gamma)
    new = tree_step(mesh, u, dt, gamma, case["ghost"])
    dts = [dt, time_step(mesh, new, gamma)] if case["chain"] else [dt]
    return {"u": new, "dt": torch.stack(dts)}


def primitive(u, gamma):
    rho = u[..., 0].clamp(min=RHO_MIN)
    v = u[..., 1:4] / rho[..., None]
    p = ((gamma - 1.0) * (u[..., 4] - 0.5 * rho * (v * v).sum(-1))).clamp(min=P_MIN)
    return torch.cat([rho[..., None], v, p[..., None]], -1)


def time_step(mesh, u, gamma, sub=False):
    best = []
    for l in range(mesh.lmin, mesh.lmax + 1):
        c = mesh.cells(l)
        w = primitive(u[c][~mesh.split[c]], gamma)
        if len(w):
            speed = w[:, 1:4].abs().sum(1) + 3.0 * torch.sqrt(gamma * w[:, 4] / w[:, 0])
            best.append(0.5 ** (mesh.lmin if sub else l) / speed.max())
    return CFL * torch.stack(best).min()


def minmod(a, b):
    return torch.where(a * b > 0, torch.where(a.abs() < b.abs(), a, b), torch.zeros_like(a))


def hllc(left, right, ax, gamma):
    cl, cr = (torch.sqrt(gamma * s[..., 4] / s[..., 0]) for s in (left, right))
    ul, ur = left[..., 1 + ax], right[..., 1 + ax]
    sl, sr = torch.minimum(ul - cl, ur - cr), torch.maximum(ul + cl, ur + cr)
    ml, mr = left[..., 0] * (ul - sl), right[..., 0] * (sr - ur)
    star = (mr * ur + ml * ul + left[..., 4] - right[..., 4]) / (ml + mr)
    pstar = (mr * left[..., 4] + ml * right[..., 4] + ml * mr * (ul - ur)) / (ml + mr)
    use_l = (sl > 0) | (star > 0)
    outer = torch.where(use_l, sl > 0, ~(sr > 0))
    s = torch.where(use_l[..., None], left, right)
    rho, p, un = s[..., 0], s[..., 4], s[..., 1 + ax]
    e = p / (gamma - 1.0) + 0.5 * rho * (s[..., 1:4] ** 2).sum(-1)
    edge = torch.where(use_l, sl, sr)
    rs = torch.where(outer, rho, rho * (edge - un) / (edge - star))
    es = torch.where(outer, e, ((edge - un) * e - p * un + pstar * star) / (edge - star))
    ps, ss = torch.where(outer, p, pstar), torch.where(outer, un, star)
    f = [rs * ss] + [rs * ss * s[..., 1 + a] for a in range(3)] + [(es + ps) * ss]
    f[1 + ax] = rs * ss * ss + ps
    return torch.stack(f, -1)


def interpolated(mesh, l, u, cell, sub):
    """Minmod-limited values at a quarter of the width from coarse cells' centres."""
    uc = u[cell]
    out = uc.clone()
    octs, q = cell >> 3, cell & 7
    uniq, back = torch.unique(octs, return_inverse=True)
    nb = mesh.neighbours(l, uniq)[back]
    for a in range(3):
        side = []
        for d in range(2):
            e = nb[:, 13 + (2 * d - 1) * 3 ** a]
            other = q ^ (1 << a)
            far = torch.where(e >= 0, 8 * e + other, torch.where(e == OUT, cell, -1 - e))
            side.append(u[torch.where(((q >> a) & 1) != d, 8 * octs + other, far)])
        out += torch.where(sub[a], 0.25, -0.25)[:, None] * minmod(uc - side[0], side[1] - uc)
    return out


def level_update(mesh, l, u, dt, gamma, ghost):
    """New cells of level l and, per side, the fluxes owed to coarse cells."""
    r = dt * 2.0 ** l
    h = 0.5 * r
    new, owed = torch.empty_like(u[mesh.cells(l)]), [[] for _ in range(6)]
    at = torch.arange(-2, 4, device=u.device)
    first, last = mesh.begin[l], mesh.begin[l + 1]
    for b in range(first, last, 1 << 16):
        octs = torch.arange(b, min(last, b + (1 << 16)), device=u.device)
        nb = mesh.neighbours(l, octs)
        slot, sub, clamped = [], [], []
        for a in range(3):
            lo, hi = nb[:, 13 - 3 ** a] == OUT, nb[:, 13 + 3 ** a] == OUT
            s = torch.div(at, 2, rounding_mode="floor")[None].expand(len(octs), 6)
            out = (lo[:, None] & (s < 0)) | (hi[:, None] & (s > 0))
            slot.append(torch.where(out, torch.zeros_like(s), s) + 1)
            sub.append(torch.where(out, (s > 0).long(), at[None] & 1))
            clamped.append(out)
        each = slice(None)
        full = [(each, None, None), (each, None, each, None), (each, each, None, None)]
        pick = slot[0][full[0]] + 3 * slot[1][full[1]] + 9 * slot[2][full[2]]
        e = nb.gather(1, pick.reshape(len(octs), -1)).view(-1, 6, 6, 6)
        bit = sub[0][full[0]] + 2 * sub[1][full[1]] + 4 * sub[2][full[2]]
        cell = torch.where(e >= 0, 8 * e + bit, -1 - e)
        ut = u[cell]
        coarse = e < 0
        if ghost and bool(coarse.any()):
            subs = [v[f].expand_as(e)[coarse].bool() for v, f in zip(sub, full)]
            ut[coarse] = interpolated(mesh, l - 1, u, cell[coarse], subs)
        clamp = clamped[0][full[0]] | clamped[1][full[1]] | clamped[2][full[2]]
        split = mesh.split[cell] & (e >= 0) & ~clamp
        w = primitive(ut, gamma)
        mid = slice(1, 5)
        w0 = w[:, mid, mid, mid]
        dw = []
        for a in range(3):
            lo, hi = [mid] * 3, [mid] * 3
            lo[2 - a], hi[2 - a] = slice(0, 4), slice(2, 6)
            dw.append(minmod(w0 - w[(slice(None), *lo)], w[(slice(None), *hi)] - w0))
        div = dw[0][..., 1] + dw[1][..., 2] + dw[2][..., 3]
        rate = sum(w0[..., 1 + a, None] * dw[a] for a in range(3))
        rate[..., 0] += w0[..., 0] * div
        for a in range(3):
            rate[..., 1 + a] += dw[a][..., 4] / w0[..., 0]
        rate[..., 4] += gamma * w0[..., 4] * div
        wp = w0 - h * rate
        own = ut[:, 2:4, 2:4, 2:4].clone()
        for a in range(3):
            inner = [slice(1, 3)] * 3

            def along(v, s, a=a, inner=inner):
                q = list(inner)
                q[2 - a] = s
                return v[(slice(None), *q)]

            left = along(wp, slice(0, 3)) + 0.5 * along(dw[a], slice(0, 3))
            right = along(wp, slice(1, 4)) - 0.5 * along(dw[a], slice(1, 4))
            for s in (left, right):
                s[..., 0].clamp_(min=RHO_MIN)
                s[..., 4].clamp_(min=P_MIN)
            g = hllc(left, right, a, gamma) * r
            sp = split[:, mid, mid, mid]
            g = torch.where((along(sp, slice(0, 3)) | along(sp, slice(1, 4)))[..., None], torch.zeros_like(g), g)
            lo, hi = [slice(None)] * 3, [slice(None)] * 3
            lo[2 - a], hi[2 - a] = slice(0, 2), slice(1, 3)
            own += g[(slice(None), *lo)] - g[(slice(None), *hi)]
            for d in range(2):
                n = nb[:, 13 + (2 * d - 1) * 3 ** a]
                sel = (n < 0) & (n != OUT)
                face = g[sel].select(3 - a, 2 * d).sum((1, 2)) * 0.125
                owed[2 * a + d].append((-1 - n[sel], face if d else -face))
        new[8 * (b - first):8 * (b - first) + 8 * len(octs)] = own.reshape(-1, 5)
    return new, [[(torch.cat([p[k] for p in s])) for k in range(2)] for s in owed]


def tree_step(mesh, u, dt, gamma, ghost):
    new, owed = torch.empty_like(u), []
    for l in range(mesh.lmin, mesh.lmax + 1):
        new[mesh.cells(l)], o = level_update(mesh, l, u, dt, gamma, ghost)
        owed.append(o)
    for side in range(6):
        for o in owed:
            new.index_add_(0, o[side][0], o[side][1])
    return mesh.fill_split(new)


def tree_subcycled(mesh, u, dt, gamma, ghost):
    cur = u.clone()

    def advance(l, step):
        new, owed = level_update(mesh, l, cur, step, gamma, ghost)
        if l < mesh.lmax:
            first = 8 * mesh.begin[l]
            subs = [advance(l + 1, 0.5 * step) for _ in range(2)]
            for side in range(6):
                for o in subs:
                    new.index_add_(0, o[side][0] - first, o[side][1])
            new[mesh.father[mesh.octs(l + 1)] - first] = cur[mesh.cells(l + 1)].view(-1, 8, 5).mean(1)
        cur[mesh.cells(l)] = new
        return owed

    advance(mesh.lmin, dt)
    return cur


# multigrid on dense grids [z, y, x] -----------------------------------------

def sides(p):
    return [torch.roll(p, s, d) for d in (2, 1, 0) for s in (1, -1)]


def checker(n):
    a = torch.arange(n, device=device())
    return (a[:, None, None] + a[None, :, None] + a[None, None, :]) % 2 == 0


def mean8(v):
    n = v.shape[0] // 2
    return v.view(n, 2, n, 2, n, 2).mean((1, 3, 5))


def trilinear(c):
    """Values at the fine cells' centres: a quarter of a coarse cell to either side per axis."""
    for d in range(3):
        lo, hi = 0.75 * c + 0.25 * torch.roll(c, 1, d), 0.75 * c + 0.25 * torch.roll(c, -1, d)
        c = torch.stack([lo, hi], d + 1).flatten(d, d + 1)
    return c


def laplacian_parts(p, mask, wall, inside):
    """Sum of the six neighbours (outside ones from `wall`, or with the mask's cut diagonal) and the diagonal."""
    total, diag = torch.zeros_like(p), torch.full_like(p, 6.0)
    if inside is None:
        return sum(sides(p)), diag
    for q, m, i in zip(sides(p), sides(mask), sides(inside)):
        if wall is None:
            total += torch.where(i, q, torch.zeros_like(q))
            diag += torch.where(i, torch.zeros_like(q), (mask - m) / mask - 1.0)
        else:
            total += q
    return total, diag


def grid_cycle(e, f, l, stop, mask=None, wall=None):
    """One V-cycle on level l (in place on a copy); mask None: every cell inside."""
    h2, n = 4.0 ** -l, e.shape[0]
    red = checker(n)
    inside = None if mask is None else mask[l] > 0
    m = None if mask is None else mask[l]

    def field(e):
        return e if wall is None else torch.where(inside, e, wall)

    def sweeps(e, count):
        for _ in range(count):
            for colour in (red, ~red):
                total, diag = laplacian_parts(field(e), m, wall, inside)
                on = colour if inside is None else colour & inside
                e = torch.where(on, (total - h2 * f) / diag, e)
        return e

    if l == stop:
        return sweeps(e, 50)
    e = sweeps(e, 2)
    total, diag = laplacian_parts(field(e), m, wall, inside)
    res = f - (total - diag * e) / h2
    if inside is not None:
        res = torch.where(inside, res, torch.zeros_like(res))
    c = mean8(res)
    add = trilinear(grid_cycle(torch.zeros_like(c), c, l - 1, stop, mask))
    e = e + (add if inside is None else torch.where(inside, add, torch.zeros_like(add)))
    return sweeps(e, 2)


def places(mesh, l):
    """Positions in a dense [z, y, x] grid of level l's cells, key order."""
    p = mesh.ijkl[mesh.octs(l)]
    b = rows(8)
    c = [2 * p[:, a, None] + ((b >> a) & 1) for a in range(3)]
    return code(*c, 1 << l).reshape(-1)


def exact_poisson(case, seed):
    l = case["base"]
    mesh = mesh_of({**case, "lmax": l, "bc": "periodic", "tree": "uniform"})
    n, at = 1 << l, places(mesh, l)
    f = torch.zeros(n ** 3, dtype=torch.float64, device=device())
    f[at] = right_side(mesh, seed)
    f = f.view(n, n, n)
    e = torch.zeros_like(f)
    for _ in range(case["cycles"]):
        e = grid_cycle(e, f, l, 1)
    res = f - (sum(sides(e)) - 6.0 * e) * 4.0 ** l
    return {"phi": e.reshape(-1)[at], "residual": res.reshape(-1)[at]}


def exact_levels(case, mesh, f):
    phi = torch.zeros_like(f)
    coarse = None
    for l in range(mesh.lmin, mesh.lmax + 1):
        n, at = 1 << l, places(mesh, l)
        here = torch.zeros(n ** 3, dtype=torch.float64, device=f.device)
        here[at] = f[mesh.cells(l)]
        mask = {l: torch.full((n ** 3,), -1.0, dtype=torch.float64, device=f.device)}
        mask[l][at] = 1.0
        mask[l] = mask[l].view(n, n, n)
        for m in range(l - 1, 0, -1):
            mask[m] = mean8(mask[m + 1])
        wall = torch.zeros((n, n, n), dtype=torch.float64, device=f.device) if coarse is None else trilinear(coarse)
        e = torch.zeros((n, n, n), dtype=torch.float64, device=f.device)
        for _ in range(case["cycles"]):
            e = grid_cycle(e, here.view(n, n, n), l, 1, mask, wall)
        e = torch.where(mask[l] > 0, e, torch.zeros_like(e))
        phi[mesh.cells(l)] = e.reshape(-1)[at]
        coarse = e
    return phi
