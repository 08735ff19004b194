"""Cases for timing the DEM library as its users call it.

Every case is a simulation (or a batch of them) that a program holds on the
GPU and advances: one pass is ``step(n)`` followed by a state read-out, or,
for the stateless search, one search of device arrays.  The inputs are made
here, vectorised and from the seed alone: rigid aggregates of 1-8 spheres cut
out of a jittered lattice, so that neighbours overlap by about 1e-3 as in a
settled pile, listed in random order as a random placement would leave them.
The physical constants are those of ``workloads.py``.
"""
import math

import numpy as np
import torch

from paper_2311_11322_amd import dem
from paper_2311_11322_amd import workloads as W

# a connected path through the 8 sites of a 2 x 2 x 2 block
_PATH = np.array([[0, 0, 0], [1, 0, 0], [1, 1, 0], [0, 1, 0],
                  [0, 1, 1], [1, 1, 1], [1, 0, 1], [0, 0, 1]])


def listed():
    return [
        # a system small enough for one workgroup: parameter scans over a few bodies
        dict(name="gas_97", kind="gas", n=97, precision=0, steps=100),
        # the contact-only periodic box of the benchmark (500 aggregates)
        dict(name="gas_2350", kind="gas", n=2350, precision=0, steps=100),
        # box filling under a uniform field, five walls (the paper's profiling runs)
        dict(name="fill_6400", kind="fill", n=6400, precision=0, steps=100),
        # Brazil-nut run: one large intruder among grains, shaken walls
        dict(name="nut_4001", kind="nut", n=4001, precision=0, steps=100),
        # served request, small: a pile in a tidal flyby, FP32-force
        dict(name="flyby_3000", kind="pile", n=3000, precision=1, steps=40, flyby=True),
        # served request, ordinary: one pile spun up, plain FP64
        dict(name="spin_13001", kind="pile", n=13001, precision=0, steps=20, spin=True),
        # batched spin-up campaign: many piles of 500-20,000 spheres in one engine, FP32-force
        dict(name="batch_48", kind="batch", n=48, precision=1, steps=12, nmin=500, nmax=20000),
        # stateless search on device arrays, as a tight loop of another program calls it
        dict(name="search_20011", kind="search", n=20011, periodic=False),
        # the headline: collapse of 25,000 aggregates, exact gravity, plain FP64
        dict(name="cloud_125k", kind="cloud", n=124958, precision=0, steps=4),
        # the same form of run in the FP32-force form, larger
        dict(name="cloud_180k_f32", kind="cloud", n=180001, precision=1, steps=3),
        # tree gravity (hexadecapole, opening angle 0.5, leaves of 32)
        dict(name="tree_125k", kind="cloud", n=124958, precision=0, steps=6, tree=4, theta=0.5),
        # the contact path alone at 1M spheres (memory bound)
        dict(name="lattice_1M", kind="lattice", n=1000000, precision=0, steps=60,
             order="slices"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gas", "fill", "nut", "pile", "pile", "batch", "search", "cloud", "tree",
                       "lattice"])
    prec = rng.randrange(2)
    if kind == "gas":
        return dict(kind="gas", n=_log(rng, 40, 60000), precision=prec, steps=60)
    if kind == "fill":
        return dict(kind="fill", n=_log(rng, 400, 20000), precision=prec, steps=60)
    if kind == "nut":
        return dict(kind="nut", n=_log(rng, 2000, 12000), precision=prec, steps=60)
    if kind == "pile":
        form = rng.choice(["still", "spin", "flyby"])
        return dict(kind="pile", n=_log(rng, 200, 50000), precision=prec, steps=16,
                    spin=form == "spin", flyby=form == "flyby")
    if kind == "batch":
        return dict(kind="batch", n=rng.randrange(4, 64), precision=prec, steps=10, nmin=500,
                    nmax=_log(rng, 2000, 16000))
    if kind == "search":
        return dict(kind="search", n=_log(rng, 100, 65536), periodic=rng.random() < 0.5)
    if kind == "cloud":
        return dict(kind="cloud", n=_log(rng, 50000, 124000 if prec == 0 else 180000),
                    precision=prec, steps=3)
    if kind == "tree":
        return dict(kind="cloud", n=_log(rng, 20000, 400000), precision=prec, steps=4,
                    tree=rng.choice([2, 4]), theta=rng.choice([0.5, 0.7]))
    side = 2 * rng.randrange(15, 50) + rng.randrange(2)
    return dict(kind="lattice", n=side ** 3, precision=prec, steps=30,
                order=rng.choice(["slices", "morton"]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _aggregates(rng, blocks, n, cmin, dense, spread, overlap=0.0, noise=1e-3, spacing=2.0):
    """Spheres of the first n sites of 2 x 2 x 2 blocks (given in order of
    preference), grouped into rigid aggregates: dense blocks are cut into runs
    along the path, others hold one aggregate of cmin..8 sites (the cuts
    depend on n alone, so that every seed gives as many aggregates).  Radii
    alternate between 1 + spread and 1 - spread, so that neighbours touch:
    about half of them, or, with an overlap above the noise, all of them."""
    nb = blocks.shape[0]
    cuts = np.random.default_rng(n)
    if dense:
        start = cuts.random((nb, 8)) < 0.12
        start[:, 0] = True
        keep = np.ones((nb, 8), bool)
    else:
        c = cuts.integers(cmin, 9, nb)
        keep = np.arange(8)[None, :] < c[:, None]
        start = np.zeros((nb, 8), bool)
        start[:, 0] = True
    site = (2 * blocks[:, None, :] + _PATH[None]).reshape(-1, 3)[keep.ravel()][:n]
    start = start.ravel()[keep.ravel()][:n]
    agg = np.cumsum(start) - 1
    pos = spacing * (site + 0.5) + rng.uniform(-2e-4, 2e-4, site.shape)
    rad = 1.0 + spread * (1 - 2 * (site.sum(1) & 1)) + rng.uniform(-noise, noise, len(site))
    rad += 0.5 * overlap
    # aggregates in random order, members kept together
    rank = rng.permutation(agg[-1] + 1)
    order = np.argsort(rank[agg], kind="stable")
    counts = np.bincount(rank[agg]).astype(np.int32)
    return counts, pos[order], rad[order]


def _cube_blocks(nx, ny, nz):
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1)
    return g.reshape(-1, 3)


def _ball_blocks(rng, n, fraction, mean):
    """Blocks in a ball about the origin, nearest first, each kept with
    probability `fraction`, enough for n spheres of `mean` per block."""
    want = int(n / mean / fraction * 1.1) + 64
    r = int(math.ceil((want * 0.75 / math.pi) ** (1.0 / 3.0))) + 2
    g = _cube_blocks(2 * r, 2 * r, 2 * r) - r
    d = ((g + 0.5) ** 2).sum(1)
    g = g[np.argsort(d, kind="stable")]
    return g[rng.random(g.shape[0]) < fraction]


def _inputs(case, seed):
    """One system: dict of arrays and parameters."""
    rng = np.random.default_rng(seed)
    kind, n = case["kind"], int(case["n"])
    prm = dict(W.CONTACT_PARAMS, dt=5e-4, G=0.0, soft_frac=0.5, periodic=0, box=(0.0, 0.0, 0.0))
    vel, spin = 0.05, 0.05
    if kind == "lattice":
        w = W.dense_lattice(seed=seed, n_side=int(round(n ** (1.0 / 3.0))), order=case["order"])
        return dict(counts=w.counts, pos=w.pos, radius=w.radius, mass=w.mass, vel=w.agg_vel,
                    spin=w.agg_spin, params=w.params)
    if kind in ("gas", "search"):
        # packing 0.2 in a periodic cube
        m = max(2, int(math.ceil((n / 4.5 / 0.68) ** (1.0 / 3.0))) + 1)
        blocks = rng.permutation(_cube_blocks(m, m, m))
        counts, pos, rad = _aggregates(rng, blocks, n, 1, False, 0.2)
        prm.update(dt=1e-4, periodic=1, box=(4.0 * m,) * 3)
    elif kind in ("fill", "nut"):
        # unit spheres settled in a box of base 40 x 40
        layers = int(math.ceil(n / 400.0 / 2)) + (4 if kind == "nut" else 1)
        blocks = _cube_blocks(10, 10, layers)
        blocks = blocks[np.argsort(blocks[:, 2], kind="stable")]
        n_grain = n
        if kind == "nut":
            n_grain = n - 1
            c = 4.0 * blocks + 2.0
            blocks = blocks[np.linalg.norm(c - np.array([20.0, 20.0, 6.0]), axis=1) > 9.0]
        counts, pos, rad = _aggregates(rng, blocks, n_grain, 1, True, 0.0)
        prm.update(g=(0.0, 0.0, -2.0), walls=W.open_box_walls(40.0, 40.0))
        vel, spin = 0.01, 0.01
        if kind == "nut":
            counts = np.concatenate([[1], counts]).astype(np.int32)
            pos = np.concatenate([[[20.0, 20.0, 5.9995]], pos])
            rad = np.concatenate([[6.0], rad])
            walls = list(prm["walls"])
            walls[0] = (0.0, 0.0, 1.0, 4.0)          # lowest point of the shaking at t = 0
            prm.update(walls=walls, shake_amp=[(0.0, 0.0, 4.0)] * 5,
                       shake_omega=math.sqrt(3.0 * 2.0 / 4.0), shake_phase=-0.5 * math.pi)
    else:
        # every neighbour pair overlaps from the start, as in a settled pile,
        # so no contact's first step hangs on the last bits of the FP32 forces
        prm.update(G=1.0)
        vel, spin, over = 0.02, 0.02, dict(overlap=1e-3, noise=1e-4)
        if kind == "pile":
            blocks = _ball_blocks(rng, n, 1.0, 8.0)
            counts, pos, rad = _aggregates(rng, blocks, n, 1, True, 0.2, **over)
        else:
            blocks = _ball_blocks(rng, n, 0.46, 5.0)
            counts, pos, rad = _aggregates(rng, blocks, n, 2, False, 0.2, **over)
        if case.get("tree"):
            prm.update(gravity_tree=1, theta=float(case["theta"]), tree_leaf=32,
                       tree_order=int(case["tree"]))
    na = counts.shape[0]
    mass = W.sphere_mass(rad)
    out = dict(counts=counts, pos=pos, radius=rad, mass=mass, vel=rng.normal(0.0, vel, (na, 3)),
               spin=rng.normal(0.0, spin, (na, 3)), params=prm)
    if case.get("spin"):
        out["spin_dw"] = 1e-6 / prm["dt"]
    if case.get("flyby"):
        M = float(mass.sum())
        com = (mass[:, None] * pos).sum(0) / M
        R = math.sqrt(5.0 / 3.0 * float((mass * ((pos - com) ** 2).sum(1)).sum()) / M)
        p, v = W.flyby_orbit(M, 1000.0 * M, 3.0 * R, start_factor=3.0)
        out["pert"] = (1000.0 * M, p + com, v)
    return out


def _sizes(case):
    """Sphere counts of a batch, log-uniform (stratified), in random order."""
    k = int(case["n"])
    rng = np.random.default_rng(k)
    lo, hi = math.log(case["nmin"]), math.log(case["nmax"])
    x = lo + (np.arange(k) + rng.random(k)) / k * (hi - lo)
    return [int(v) for v in rng.permutation(np.exp(x))]


def _piles(case, seed):
    return [_inputs(dict(kind="pile", n=m, spin=True), seed * 1009 + k)
            for k, m in enumerate(_sizes(case))]


# ---------------------------------------------------------------------------
# the library's side
# ---------------------------------------------------------------------------

def _sim(x, precision):
    sim = dem.Sim(x["params"], precision=precision)
    if "pert" in x:
        sim.set_forcing(0.0, *x["pert"])
    elif "spin_dw" in x:
        sim.set_forcing(x["spin_dw"])
    return sim.add_aggregates(x["counts"], x["pos"], x["radius"], x["mass"], x["vel"], x["spin"])


def prepare(case, seed):
    if case["kind"] == "search":
        x = _inputs(case, seed)
        agg = np.repeat(np.arange(len(x["counts"]), dtype=np.int32), x["counts"])
        return dict(case=case, pos=torch.from_numpy(x["pos"]).cuda(),
                    radius=torch.from_numpy(x["radius"]).cuda(), agg=torch.from_numpy(agg).cuda(),
                    box=x["params"]["box"] if case["periodic"] else None,
                    out=torch.zeros(8 * len(agg), dtype=torch.int64, device="cuda"))
    if case["kind"] == "batch":
        sims = [_sim(x, case["precision"]) for x in _piles(case, seed)]
        eng = dem.Engine(1 << 40)
        for s in sims:
            eng.attach(s)
        return dict(case=case, eng=eng, sims=sims)
    return dict(case=case, sim=_sim(_inputs(case, seed), case["precision"]))


_FIELDS = ("agg_pos", "agg_vel", "agg_spin", "agg_acc")


def _typed(st, precision):
    """In the FP32-force form everything but the positions is as good as its
    FP32 forces, and is handed on as FP32."""
    if precision == 1:
        for k in st:
            if isinstance(st[k], np.ndarray) and st[k].dtype == np.float64 and k != "agg_pos":
                st[k] = st[k].astype(np.float32)
    return st


def _padded(st, n):
    """Contact arrays brought to a length that does not depend on the seed."""
    for k in ("pair_keys", "pair_hist"):
        if k in st:
            a = np.zeros((4 * n,) + st[k].shape[1:], np.int64 if k == "pair_keys" else st[k].dtype)
            m = min(4 * n, len(st[k]))
            a[:m] = st[k][:m]
            st[k] = a
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "search":
        n = dem.find_contacts_noalloc(state["pos"], state["radius"], state["agg"],
                                      box=state["box"], out=state["out"])
        return {"n": n, "keys": state["out"]}
    if case["kind"] == "batch":
        code = state["eng"].step(case["steps"])
        sts = [s.read_state(("agg_pos", "agg_vel")) for s in state["sims"]]
        return {"code": code, "n_pairs": np.array([s["n_pairs"] for s in sts]),
                **_typed({k: np.concatenate([s[k] for s in sts]) for k in ("agg_pos", "agg_vel")},
                         case["precision"])}
    sim = state["sim"]
    sim.step(case["steps"])
    # contacts and their history are read where a run is small enough to keep them
    pairs = case["n"] <= 30000
    st = sim.read_state(_FIELDS if case["n"] <= 500000 else _FIELDS[:2], pairs=pairs)
    if case.get("flyby"):
        f = sim.get_forcing()
        st.update(pert_pos=f["pert_pos"], pert_vel=f["pert_vel"])
    st.pop("step")
    return _typed(_padded(st, case["n"]), case["precision"])


def work(case):
    """Per sphere and step about 390 B for the body update, binning and search
    and 64 B for each contact; exact gravity 20 flops per ordered pair; the
    hexadecapole tree about 3e5 flops per sphere."""
    if case["kind"] == "search":
        return {"bytes": 36.0 * case["n"] + 8.0 * case["n"], "flops": 27.0 * 10 * case["n"]}
    z = {"lattice": 5.0, "fill": 2.5, "nut": 2.5, "pile": 3.5, "batch": 3.5}.get(case["kind"], 0.7)
    if case["kind"] == "batch":
        n = np.array(_sizes(case), float)
        g, n = 20.0 * float((n * n).sum()), float(n.sum())
    else:
        n = float(case["n"])
        g = 0.0
        if case["kind"] in ("pile", "cloud"):
            g = 20.0 * n * (n - 1)
        if case.get("tree"):
            g = {(2, 0.5): 1.8e5, (4, 0.5): 3.0e5, (2, 0.7): 0.9e5, (4, 0.7): 1.5e5}[
                (int(case["tree"]), float(case["theta"]))] * n
    s = float(case["steps"])
    return {"bytes": s * n * (390.0 + 64.0 * z), "flops": s * (g + n * (200.0 + 300.0 * z))}


# ---------------------------------------------------------------------------
# the method in plain float64
# ---------------------------------------------------------------------------

def _quat_rot(q):
    w, x, y, z = q.unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                       1).reshape(-1, 3, 3)


def _mv(R, v):
    return (R * v[:, None, :]).sum(2)


def _cross(a, b):
    return torch.linalg.cross(a, b)


def _dot(a, b):
    return (a * b).sum(1, keepdim=True)


_CK_A = [[], [1 / 5], [3 / 40, 9 / 40], [3 / 10, -9 / 10, 6 / 5],
         [-11 / 54, 5 / 2, -70 / 27, 35 / 27],
         [1631 / 55296, 175 / 512, 575 / 13824, 44275 / 110592, 253 / 4096]]
_CK_B = [37 / 378, 0, 250 / 621, 125 / 594, 0, 512 / 1771]


class _Exact:
    """The step in float64 torch operations.  Orientations start at the
    identity with the inertia tensor in space axes: the Runge-Kutta step does
    not depend on the choice of the body axes."""

    def __init__(self, x, device):
        t = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=device)
        self.p, self.x = x["params"], x
        self.dev = device
        counts = torch.as_tensor(x["counts"].astype(np.int64), device=device)
        self.na, self.ns = counts.numel(), len(x["radius"])
        self.agg = torch.repeat_interleave(torch.arange(self.na, device=device), counts)
        self.s, self.m = t(x["radius"]), t(x["mass"])
        pos = t(x["pos"])
        self.M = self._sum(self.m[:, None])
        com = self._sum(self.m[:, None] * pos) / self.M
        self.b = pos - com[self.agg]
        tr = (self.b ** 2).sum(1) + 0.4 * self.s ** 2
        eye = torch.eye(3, dtype=torch.float64, device=device)
        I = self.m[:, None, None] * (tr[:, None, None] * eye
                                     - self.b[:, :, None] * self.b[:, None, :])
        self.I = self._sum(I.reshape(-1, 9)).reshape(-1, 3, 3)
        self.Iinv = torch.linalg.inv(self.I)
        self.L = float(self.p["box"][0]) if self.p["periodic"] else 0.0
        self.r = torch.remainder(com, self.L) if self.L else com
        self.v, self.wb = t(x["vel"]), t(x["spin"])
        self.q = torch.zeros(self.na, 4, dtype=torch.float64, device=device)
        self.q[:, 0] = 1.0
        self.h = float(self.p["dt"])
        self.step_no = 0
        self.keys = torch.zeros(0, dtype=torch.int64, device=device)
        self.hist = torch.zeros(0, 7, dtype=torch.float64, device=device)
        self.pert = None
        if "pert" in x:
            self.pert = [float(x["pert"][0]), t(x["pert"][1]), t(x["pert"][2]), None]
        self._evaluate(self.v, 0)

    def _sum(self, v):
        return torch.zeros(self.na, v.shape[1], dtype=v.dtype, device=v.device).index_add_(
            0, self.agg, v)

    def _image(self, d):
        if self.L:
            d = torch.where(d > 0.5 * self.L, d - self.L,
                            torch.where(d < -0.5 * self.L, d + self.L, d))
        return d

    def _touch(self, i, j, rs):
        d = self._image(rs[j] - rs[i])
        S = self.s[i] + self.s[j]
        d2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        return (d2 < S * S) & (self.agg[i] != self.agg[j])

    def _pairs(self, rs):
        """Canonical keys of all touching pairs i < j of other aggregates."""
        n, found = self.ns, []
        if n <= 9000:
            ids = torch.arange(n, device=self.dev)
            for a in range(0, n, 1024):
                i = ids[a:a + 1024]
                hit = self._touch(i[:, None], ids[None, :], rs) & (ids[None, :] > i[:, None])
                ii, jj = hit.nonzero(as_tuple=True)
                found.append((i[ii] << 32) | jj)
            return torch.cat(found).sort().values
        cell = 2.0 * float(self.s.max()) * (1 + 1e-9)
        if self.L:
            nc = max(1, int(self.L / cell))
            c = (torch.remainder(rs, self.L) * (nc / self.L)).long().clamp(0, nc - 1)
            dims = (nc, nc, nc)
        else:
            c = ((rs - rs.min(0).values) / cell).long()
            dims = tuple(int(v) + 1 for v in c.max(0).values)
        key = (c[:, 0] * dims[1] + c[:, 1]) * dims[2] + c[:, 2]
        skey, order = key.sort()
        ids = torch.arange(n, device=self.dev)
        for ox in (-1, 0, 1):
            for oy in (-1, 0, 1):
                for oz in (-1, 0, 1):
                    o = c + torch.tensor([ox, oy, oz], device=self.dev)
                    ok = torch.ones(n, dtype=torch.bool, device=self.dev)
                    for k in range(3):
                        if self.L:
                            o[:, k] %= dims[k]
                        else:
                            ok &= (o[:, k] >= 0) & (o[:, k] < dims[k])
                    nk = (o[:, 0] * dims[1] + o[:, 1]) * dims[2] + o[:, 2]
                    lo = torch.searchsorted(skey, nk)
                    hi = torch.where(ok, torch.searchsorted(skey, nk, right=True), lo)
                    for u in range(int((hi - lo).max())):
                        i = ids[lo + u < hi]
                        j = order[(lo + u)[i]]
                        i, j = i[j > i], j[j > i]
                        hit = self._touch(i, j, rs)
                        found.append((i[hit] << 32) | j[hit])
        return torch.unique(torch.cat(found))

    def _gravity(self, rs):
        n, p = self.ns, self.p
        e = 0.5 * float(p["soft_frac"]) * self.s
        out = torch.empty_like(rs)
        rows = max(1, int(6e7) // n)
        for a in range(0, n, rows):
            d = [rs[None, :, k] - rs[a:a + rows, None, k] for k in range(3)]
            r2 = e[None, :] + e[a:a + rows, None]
            r2 = r2.mul_(r2)
            for k in range(3):
                r2.addcmul_(d[k], d[k])
            w = r2.pow_(-1.5).mul_(self.m[None, :])
            for k in range(3):
                out[a:a + rows, k] = d[k].mul_(w).sum(1)
        return out * (float(p["G"]) * self.m)[:, None]

    def _model(self, n, delta, la, lb, mu, Rab, va, wa, vb, wb, hs):
        p, h = self.p, self.h
        damp = [-2 * math.log(p[k]) / math.sqrt(math.pi ** 2 + math.log(p[k]) ** 2)
                for k in ("eps_n", "eps_t")]
        kn, kt, kr, kq = (float(p[k]) for k in ("k_n", "k_t", "k_r", "k_q"))
        arm_a, arm_b = la * n, -lb * n
        u = (vb + _cross(wb, arm_b)) - (va + _cross(wa, arm_a))
        un = _dot(u, n)
        ut = u - un * n
        Cn, Ct = damp[0] * torch.sqrt(kn * mu), damp[1] * torch.sqrt(kt * mu)
        fn = -kn * delta + Cn * un
        load = (-fn).clamp(min=0.0)

        def cap(xi, k, lim):
            mag = k * xi.norm(dim=1, keepdim=True)
            over = mag > lim
            return torch.where(over, xi * (lim / torch.where(over, mag, torch.ones_like(mag))),
                               xi), over

        xt = hs[:, 0:3]
        xt, slid = cap(xt - _dot(xt, n) * n + h * ut, kt, p["mu_s"] * load)
        F = fn * n + kt * xt + torch.where(slid, torch.zeros_like(ut), Ct * ut)
        dw = wb - wa
        xr = hs[:, 3:6]
        xr, _ = cap(xr - _dot(xr, n) * n + h * Rab * _cross(dw, n), kr, p["mu_r"] * load)
        xq, _ = cap(hs[:, 6:7] + h * Rab * _dot(dw, n), kq, p["mu_t"] * load)
        couple = Rab * kr * _cross(n, xr) + Rab * kq * xq * n
        return (F, _cross(arm_a, F) + couple, -_cross(arm_b, F) - couple,
                torch.cat([xt, xr, xq], 1))

    def _evaluate(self, vpred, at):
        p, ns, agg = self.p, self.ns, self.agg
        R = _quat_rot(self.q)
        d = _mv(R[agg], self.b)
        wA = _mv(R, self.wb)
        rs = self.r[agg] + d
        vs = vpred[agg] + _cross(wA[agg], d)
        keys = self._pairs(rs)
        walls, t = p.get("walls", ()), at * self.h
        gaps = []
        for w, wl in enumerate(walls):
            nrm = torch.tensor(wl[:3], dtype=torch.float64, device=self.dev)
            A = torch.tensor(p["shake_amp"][w] if "shake_amp" in p else (0.0, 0.0, 0.0),
                             dtype=torch.float64, device=self.dev)
            ph = p.get("shake_omega", 0.0) * t + p.get("shake_phase", 0.0)
            gap = (rs * nrm).sum(1) - (wl[3] + float((nrm * A).sum()) * math.sin(ph))
            gaps.append((gap, nrm, A * p.get("shake_omega", 0.0) * math.cos(ph)))
            hit = (gap < self.s).nonzero()[:, 0]
            keys = torch.cat([keys, (hit << 32) | (ns + w)])
        keys = keys.sort().values
        i, j = keys >> 32, keys & 0xffffffff
        hs = torch.zeros(keys.numel(), 7, dtype=torch.float64, device=self.dev)
        if self.keys.numel():
            at_old = torch.searchsorted(self.keys, keys).clamp(max=self.keys.numel() - 1)
            same = self.keys[at_old] == keys
            hs[same] = self.hist[at_old[same]]
        F = torch.zeros(ns, 3, dtype=torch.float64, device=self.dev)
        T = torch.zeros_like(F)
        hist = torch.zeros_like(hs)
        sp = j < ns
        a, b = i[sp], j[sp]
        dd = self._image(rs[b] - rs[a])
        dist = dd.norm(dim=1, keepdim=True)
        sa, sb = self.s[a][:, None], self.s[b][:, None]
        la = (sa * sa - sb * sb + dist * dist) / (2 * dist)
        Ma, Mb = self.M[agg[a]], self.M[agg[b]]
        f, ta, tb, hist[sp] = self._model(dd / dist, sa + sb - dist, la, dist - la,
                                          Ma * Mb / (Ma + Mb), sa * sb / (sa + sb), vs[a],
                                          wA[agg[a]], vs[b], wA[agg[b]], hs[sp])
        F.index_add_(0, a, f).index_add_(0, b, -f)
        T.index_add_(0, a, ta).index_add_(0, b, tb)
        for w, (gap, nrm, vw) in enumerate(gaps):
            at_w = j == ns + w
            a = i[at_w]
            g = gap[a][:, None]
            z = torch.zeros(a.numel(), 3, dtype=torch.float64, device=self.dev)
            sa = self.s[a][:, None]
            f, ta, _, hist[at_w] = self._model((-nrm).expand_as(z), sa - g, g, torch.zeros_like(g),
                                               self.M[agg[a]], sa, vs[a], wA[agg[a]],
                                               vw.expand_as(z), z, hs[at_w])
            F.index_add_(0, a, f)
            T.index_add_(0, a, ta)
        self.keys, self.hist = keys, hist
        if p["G"] != 0.0:
            F = F + self._gravity(rs)
            if self.pert is not None:
                M, pr = self.pert[0], self.pert[1]
                dp = pr - rs
                pull = (float(p["G"]) * self.m)[:, None] * M * dp / dp.norm(dim=1,
                                                                            keepdim=True) ** 3
                F = F + pull
                self.pert[3] = -pull.sum(0) / M
        g = torch.tensor(p.get("g", (0.0, 0.0, 0.0)), dtype=torch.float64, device=self.dev)
        self.a = self._sum(F) / self.M + g
        self.N = self._sum(_cross(d, F) + T)
        self.rs = rs

    def _rotate(self, h):
        y = torch.cat([self.q, self.wb], 1)

        def f(y):
            q, w = y[:, :4], y[:, 4:]
            Nb = _mv(_quat_rot(q).transpose(1, 2), self.N)
            dq = 0.5 * torch.cat([-_dot(q[:, 1:], w), q[:, :1] * w + _cross(q[:, 1:], w)], 1)
            return torch.cat([dq, _mv(self.Iinv, Nb - _cross(w, _mv(self.I, w)))], 1)

        k = []
        for row in _CK_A:
            k.append(f(y + h * sum((c * kk for c, kk in zip(row, k)), torch.zeros_like(y))))
        y = y + h * sum(c * kk for c, kk in zip(_CK_B, k))
        self.q, self.wb = y[:, :4] / y[:, :4].norm(dim=1, keepdim=True), y[:, 4:]

    def step(self):
        h = self.h
        self.v = self.v + 0.5 * h * self.a
        self.r = self.r + h * self.v
        if self.L:
            self.r = torch.where(self.r >= self.L, self.r - self.L, self.r)
            self.r = torch.where(self.r < 0, self.r + self.L, self.r)
        if self.pert is not None:
            self.pert[2] = self.pert[2] + 0.5 * h * self.pert[3]
            self.pert[1] = self.pert[1] + h * self.pert[2]
        self._rotate(h)
        self._evaluate(self.v + 0.5 * h * self.a, self.step_no + 1)
        self.v = self.v + 0.5 * h * self.a
        if self.pert is not None:
            self.pert[2] = self.pert[2] + 0.5 * h * self.pert[3]
        if "spin_dw" in self.x:
            z = torch.tensor([0.0, 0.0, self.x["spin_dw"]], dtype=torch.float64, device=self.dev)
            com = (self.m[:, None] * self.rs).sum(0) / self.m.sum()
            self.v = self.v + _cross(z.expand_as(self.r), self.r - com)
            self.wb = self.wb + _mv(_quat_rot(self.q).transpose(1, 2), z.expand_as(self.r))
        self.step_no += 1

    def state(self):
        return dict(agg_pos=self.r, agg_vel=self.v, agg_spin=_mv(_quat_rot(self.q), self.wb),
                    agg_acc=self.a)


def exact(case, seed):
    if case["kind"] == "search":
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    cpu = lambda d: {k: v.cpu().numpy() for k, v in d.items()}
    if case["kind"] == "batch":
        if sum(float(m) ** 2 for m in _sizes(case)) * (case["steps"] + 1) > 8e10:
            return None
        piles = []
        for x in _piles(case, seed):
            o = _Exact(x, dev)
            for _ in range(case["steps"]):
                o.step()
            piles.append(cpu({k: v for k, v in o.state().items() if k in ("agg_pos", "agg_vel")}))
        return {k: np.concatenate([p[k] for p in piles]) for k in piles[0]}
    n, ev = float(case["n"]), case["steps"] + 1
    if case["kind"] in ("pile", "cloud") and ev * n * n > 1.6e11:
        return None
    o = _Exact(_inputs(case, seed), dev)
    for _ in range(case["steps"]):
        o.step()
    st = o.state()
    if case["n"] > 500000:
        st = {k: st[k] for k in _FIELDS[:2]}
    if case["n"] <= 30000:
        st["pair_hist"] = o.hist
    if case.get("flyby"):
        st.update(pert_pos=o.pert[1], pert_vel=o.pert[2])
    return _padded(cpu(st), case["n"])
