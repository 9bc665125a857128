"""The work that users of the engine have it do, as measurable cases.

Kinds of case
  chain     strained glasses: every replica is loaded, minimised to its
            inherent structure and strained by a few fine AQS steps (Eqs. 12,
            19), all in one batched call.  From one 2D replica of 256 atoms
            (bound by latency) to batches; plain, extrapolated or learned start,
            simple or pure shear.
  step      one affine increment of every replica and at most max_iter
            iterations of the minimiser (FIRE or conjugate gradients), replicas
            loaded one by one or, as level I of Algorithm 1 does, copied from
            the first and sheared further apart.  The large sizes are here: how
            a large glass rearranges on the way to its minimum depends on the
            last bit, a bounded number of iterations does not.
  round     one round of Algorithm 1: P chains of K steps and their checks,
            batched or with live checks.
  evaluate  energy, forces and stress of one configuration.
  learned   descriptors of a configuration and the network's prediction.
  train     the network's training (forward and backward).

The inputs do not come from the engine: `relax` below is a plain torch FIRE
that takes seeded random configurations near to their inherent structures, so
both sides of a comparison start from the same bits.  `exact` continues with
it in FP64 to max |F| < 1e-11.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_20802_amd import (AQS_START_EXTRAPOLATED, AQS_START_LEARNED, AQS_START_PLAIN, Cg, Engine, Fire,
                                  LJParams, learned, parallel)
from paper_2507_20802_amd.speedup import paper_potential

STARTS = {"plain": AQS_START_PLAIN, "extrapolated": AQS_START_EXTRAPOLATED, "learned": AQS_START_LEARNED}
DENSITY = {"kob_andersen": 1.2, "paper": 1.0}
FRACTION_A = {("kob_andersen", 2): 0.65, ("kob_andersen", 3): 0.80, ("paper", 2): 1.0 / (1.0 + (1.0 + 5.0 ** 0.5) / 4.0)}


def chain(name, **kw):
    c = {"name": name, "kind": "chain", "glass": "kob_andersen", "dim": 2, "n": 256, "n_max": 0, "replicas": 1,
         "steps": 1, "dgamma": 1e-4, "pure": False, "minimizer": "fire", "start": "plain", "tuning": "auto"}
    c.update(kw)
    return c


def step(name, **kw):
    c = {"name": name, "kind": "step", "glass": "kob_andersen", "dim": 3, "n": 32768, "n_max": 0, "replicas": 1,
         "copies": False, "dgamma": 5e-5, "pure": False, "minimizer": "fire", "max_iter": 300, "tuning": "auto"}
    c.update(kw)
    return c


def round_(name, **kw):
    c = {"name": name, "kind": "round", "glass": "kob_andersen", "dim": 2, "n": 4096, "glasses": 1, "P": 8, "K": 2,
         "dgamma": 1e-4, "live": False, "start": "plain"}
    c.update(kw)
    return c


def listed():
    return [
        # one small 2D glass strained step by step: the smallest call, bound by latency
        chain("chain_2d_256", n=256, steps=2),
        # the paper's benchmark problem (Sec. 2.2), many samples in one batch
        chain("paper_2d_400_x128", glass="paper", n=400, replicas=128, dgamma=1.0 / 200.0, tuning="default"),
        # a small odd 3D glass whose steps start from the extrapolated displacement
        chain("extrap_3d_1501", dim=3, n=1501, steps=3, dgamma=2e-5, start="extrapolated"),
        # the paper's minimiser under the pure shear of Eq. (17)
        step("cg_pure_2d_1000", dim=2, n=1000, replicas=2, pure=True, minimizer="cg", max_iter=60),
        # sequential AQS at the benchmark's size: one replica alone
        step("seq_3d_32768"),
        # the benchmark's level II: 16 chains of one glass in one launch
        step("batch_3d_32768_x16", replicas=16, copies=True, max_iter=150),
        # replicas of very different sizes in one batch
        step("uneven_3d", n=2048, n_max=16000, replicas=5, dgamma=1e-4),
        # several 2D glasses in one batched round of Algorithm 1
        round_("round_2d_2100_x4", n=2100, glasses=4, P=8, K=1),
        # the benchmark's form: learned start, live checks (the network's starts are mostly rejected there)
        round_("live_3d_3001", dim=3, n=3001, P=6, K=1, dgamma=5e-5, live=True, start="learned"),
        # one evaluation of a large configuration: energy, forces and stress
        {"name": "evaluate_3d_132651", "kind": "evaluate", "dim": 3, "m": 51, "strain": 37},
        # descriptors and the network's prediction for one configuration
        {"name": "learned_3d_29791", "kind": "learned", "dim": 3, "m": 31},
        # the training of the learned start
        {"name": "train_32768", "kind": "train", "dim": 3, "samples": 32768, "batch": 4096, "epochs": 4},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["small", "small", "paper", "middle", "middle", "large", "copies", "round", "live", "evaluate",
                       "learned", "train"])
    if kind == "small":
        dim = rng.choice([2, 2, 3])
        c = chain("", dim=dim, n=size(256, 1100) if dim == 2 else size(900, 2000), replicas=rng.randint(1, 4),
                  steps=rng.randint(1, 3), dgamma=rng.choice([2e-5, 5e-5, 1e-4]), pure=rng.random() < 0.2,
                  start=rng.choice(["plain", "plain", "extrapolated", "learned"]))
    elif kind == "paper":
        c = chain("", glass="paper", n=400, replicas=size(16, 160), dgamma=1.0 / 200.0, tuning="default")
    elif kind == "middle":
        cg = rng.random() < 0.25
        c = step("", dim=rng.choice([2, 3]), n=size(1000, 9000), replicas=rng.randint(1, 4),
                 dgamma=rng.choice([5e-5, 1e-4]), pure=rng.random() < 0.2, minimizer="cg" if cg else "fire",
                 max_iter=rng.randint(30, 60) if cg else rng.randint(100, 300), tuning=rng.choice(["auto", "default"]))
    elif kind == "large":
        c = step("", n=size(9000, 32768), max_iter=rng.randint(100, 300))
    elif kind == "copies":
        c = step("", n=size(4000, 32768), replicas=rng.randint(2, 12), copies=True, max_iter=rng.randint(60, 150))
    elif kind == "round":
        c = round_("", dim=2, n=size(500, 2100), glasses=rng.randint(1, 4), P=rng.choice([4, 6, 8]), K=1)
    elif kind == "live":
        c = round_("", dim=3, n=size(1200, 3000), P=rng.randint(3, 6), K=1, dgamma=5e-5, live=True,
                   start=rng.choice(["plain", "learned"]))
    elif kind == "evaluate":
        dim = rng.choice([2, 3])
        c = {"kind": "evaluate", "dim": dim, "m": size(12, 50) if dim == 3 else size(20, 300), "strain": rng.randint(0, 80)}
    elif kind == "learned":
        dim = rng.choice([2, 3])
        c = {"kind": "learned", "dim": dim, "m": size(12, 30) if dim == 3 else size(20, 150)}
    else:
        c = {"kind": "train", "dim": rng.choice([2, 3]), "samples": size(3000, 32768), "batch": rng.choice([1024, 2048, 4096]),
             "epochs": rng.randint(1, 4)}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# Plain torch FP64 Lennard-Jones (Eq. 13) and FIRE, for inputs and exact().


def potential_of(glass):
    return paper_potential() if glass == "paper" else LJParams()


class Pairs:
    """Neighbours of replicas of equal size in one box, padded: x (S, n, d), H (d, d)."""

    def __init__(self, x, types, H, pot, skin=0.4):
        S, n, d = x.shape
        Hi = torch.linalg.inv(H)
        self.H, self.Hi, self.shape, self.x0 = H.tolist(), Hi, x.shape, x.clone()
        f = x @ Hi.T
        f = f - f.floor()
        cells = [int(1.0 / float(Hi[a].norm()) / (pot.rc_max + skin)) for a in range(d)]
        by_cell = n > 3000 and min(cells) >= 3
        near, span = self.cell_table(f, cells) if by_cell else (None, n)
        rows, cols = [], []
        slots = max(1, (1 << 25) // (n * span))
        chunk = min(n, max(1, (1 << 25) // span))
        for s0 in range(0, S, slots):
            fs = f[s0:s0 + slots]
            for r0 in range(0, n, chunk):
                me = fs[:, r0:r0 + chunk]
                if by_cell:
                    j = near[s0, r0:r0 + chunk][None]
                    u = [fs[0][:, a][j.clamp(min=0)] - me[..., a, None] for a in range(d)]
                else:
                    u = [fs[:, None, :, a] - me[..., a, None] for a in range(d)]
                r2 = sum(q * q for q in self.cartesian([q - q.round() for q in u]))
                inside = (r2 < (pot.rc_max + skin) ** 2) & (j >= 0) if by_cell else r2 < (pot.rc_max + skin) ** 2
                s, i, k = inside.nonzero(as_tuple=True)
                k = j[0][i, k] if by_cell else k
                i = i + r0
                keep = i != k
                rows.append((s[keep] + s0) * n + i[keep])
                cols.append((s[keep] + s0) * n + k[keep])
        row, col = torch.cat(rows), torch.cat(cols)
        count = torch.bincount(row, minlength=S * n)
        first = count.cumsum(0) - count
        width = max(1, int(count.max()))
        self.nb = torch.arange(S * n, device=x.device)[:, None].repeat(1, width)
        self.nb[row, torch.arange(row.numel(), device=x.device) - first[row]] = col
        self.live = torch.arange(width, device=x.device)[None, :] < count[:, None]
        sig = torch.tensor(pot.sigma, dtype=torch.float64, device=x.device)
        eps = torch.tensor(pot.eps, dtype=torch.float64, device=x.device)
        t = types.long().repeat(S)
        ti, tj = t[:, None].expand_as(self.nb), t[self.nb]
        self.tj = tj
        self.s2, self.e4 = sig[ti, tj] ** 2, 4.0 * eps[ti, tj]
        self.rc2 = torch.where(self.live, self.s2 * pot.rc_factor ** 2, torch.zeros((), dtype=torch.float64, device=x.device))
        c6 = pot.rc_factor ** -6
        self.cut = c6 * c6 - c6

    def cell_table(self, f, cells):
        """Per atom the atoms of its cell and the cells around it (-1 where there is none): (S, n, width)."""
        S, n, d = f.shape
        dev = f.device
        total = math.prod(cells)
        c = [(f[..., a] * cells[a]).long().clamp(0, cells[a] - 1) for a in range(d)]
        flat = c[0]
        for a in range(1, d):
            flat = flat * cells[a] + c[a]
        flat = flat + total * torch.arange(S, device=dev)[:, None]
        order = flat.reshape(-1).sort(stable=True)
        count = torch.bincount(order.values, minlength=S * total)
        first = count.cumsum(0) - count
        cap = int(count.max())
        table = torch.full((S * total, cap), -1, dtype=torch.long, device=dev)
        table[order.values, torch.arange(S * n, device=dev) - first[order.values]] = order.indices % n
        near = []
        for off in range(3 ** d):
            q, rest = None, off
            for a in range(d):
                t = (c[a] + rest % 3 - 1) % cells[a]
                q = t if q is None else q * cells[a] + t
                rest //= 3
            near.append(table[q + total * torch.arange(S, device=dev)[:, None]])
        near = torch.cat(near, -1)
        return near, near.shape[-1]

    def cartesian(self, u):
        """H u of fractional components u, one array per axis."""
        out = []
        for row in self.H:
            t = None
            for h, q in zip(row, u):
                if h != 0.0:
                    t = h * q if t is None else t.add_(q, alpha=h)
            out.append(t)
        return out

    def separations(self, x):
        """Minimum-image r_j - r_i of every pair, one (rows, width) array per axis."""
        d = self.shape[2]
        f = (x.reshape(-1, d) @ self.Hi.T).T.contiguous()
        u = []
        for b in range(d):
            q = f[b][self.nb].sub_(f[b][:, None])
            u.append(q.sub_(q.round()))
        return self.cartesian(u)

    def forces(self, x, energy=False):
        dr = self.separations(x)
        r2 = sum(q * q for q in dr)
        inside = r2 < self.rc2
        inv = torch.where(inside, r2.reciprocal_(), 0.0)
        s6 = (self.s2 * inv) ** 3
        g = s6 * (6.0 - 12.0 * s6) * inv * self.e4
        F = torch.stack([(g * q).sum(1) for q in dr], -1).reshape(self.shape)
        if not energy:
            return F
        e = torch.where(inside, self.e4 * (s6 * s6 - s6 - self.cut), 0.0)
        S, n, d = self.shape
        W = torch.stack([(0.5 * g * p * q).sum(1) for p in dr for q in dr], -1)
        return F, 0.5 * e.sum(1).reshape(S, n).sum(1), W.reshape(S, n, d, d).sum(1)


def relax(x, types, H, pot, ftol, max_iter):
    """FIRE of every replica of x (S, n, d) in the box H, to max |F| < ftol."""
    S = x.shape[0]
    x, v = x.clone(), torch.zeros_like(x)

    def scalar(value):
        return torch.full((S, 1, 1), value, dtype=torch.float64, device=x.device)

    dt, alpha, npos = scalar(0.01), scalar(0.2), scalar(0.0)
    pairs = Pairs(x, types, H, pot)
    for it in range(max_iter):
        if it and it % 3 == 0 and float((x - pairs.x0).square().sum(-1).max()) > 0.17 ** 2:
            pairs = Pairs(x, types, H, pot)
        F = pairs.forces(x)
        if it % 20 == 0 and float(F.square().sum(-1).max()) < ftol * ftol:
            break
        up = (F * v).sum((1, 2), keepdim=True) > 0.0
        npos = torch.where(up, npos + 1.0, torch.zeros_like(npos))
        grow = up & (npos > 5.0)
        dt = torch.where(grow, (1.2 * dt).clamp(max=0.03), torch.where(up, dt, (0.9 * dt).clamp(min=2e-4)))
        alpha = torch.where(grow, 0.95 * alpha, torch.where(up, alpha, torch.full_like(alpha, 0.2)))
        x = torch.where(up, x, x - 0.5 * dt * v)
        v = torch.where(up, v, torch.zeros_like(v)) + dt * F
        vn = v.square().sum((1, 2), keepdim=True).sqrt()
        fn = F.square().sum((1, 2), keepdim=True).sqrt().clamp(min=1e-300)
        v = (1.0 - alpha) * v + (alpha * vn / fn) * F
        step = dt * v.square().sum(-1, keepdim=True).sqrt()
        v = v * (0.1 / step.clamp(min=1e-300)).clamp(max=1.0)
        x = x + dt * v
    return x


def box_of(dim, L, shear=((0.0, 0.0), (0.0, 0.0)), k=0):
    """H = F^k diag(L), F = [[1, a], [b, 1]] on (x, y)."""
    F = np.eye(dim)
    F[0, 1], F[1, 0] = shear[0][1], shear[1][0]
    if F[1, 0] == 0.0:
        F[0, 1] *= k
    else:
        F = np.linalg.matrix_power(F, k)
    return F @ np.diag([L] * dim)


def types_of(n, x_a, gen):
    t = torch.ones(n, dtype=torch.uint8, device="cuda")
    t[torch.randperm(n, generator=gen, device="cuda")[: int(math.floor(x_a * n + 0.5))]] = 0
    return t


def glass_inputs(glass, dim, n, replicas, seed):
    """Seeded random configurations taken near to their inherent structures: x (S, n, d), types (n), L."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    L = float((n / DENSITY[glass]) ** (1.0 / dim))
    types = types_of(n, FRACTION_A[(glass, dim)], gen)
    x = L * torch.rand((replicas, n, dim), generator=gen, dtype=torch.float64, device="cuda")
    H = torch.tensor(box_of(dim, L), dtype=torch.float64, device="cuda")
    x = relax(x, types, H, potential_of(glass), 1e-7, 2000 if n <= 4096 else 700)
    return torch.remainder(x, L), types, L


def lattice_inputs(dim, m, seed, strain=0.0):
    """A jittered simple lattice with random types: an evaluation's configuration, sheared by `strain`."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    n = m ** dim
    L = float((n / 1.2) ** (1.0 / dim))
    grid = torch.stack(torch.meshgrid(*[torch.arange(m, device="cuda", dtype=torch.float64)] * dim, indexing="ij"), -1)
    jit = torch.rand((n, dim), generator=gen, dtype=torch.float64, device="cuda") * 0.2 - 0.1
    x = (grid.reshape(n, dim) + 0.5 + jit) * (L / m)
    x[:, 0] += strain * x[:, 1]
    return x, types_of(n, FRACTION_A[("kob_andersen", dim)], gen), L


def network(dim, seed, **standard):
    """A network of random weights (the initialisation that training starts from)."""
    rng = np.random.default_rng(seed)
    w = {}
    for name, fi, fo in (("1", 64, 128), ("2", 128, 128), ("3", 128, dim)):
        k = 1.0 / math.sqrt(fi)
        w["w" + name] = rng.uniform(-k, k, size=(fi, fo)).astype(np.float32)
        w["b" + name] = rng.uniform(-k, k, size=fo).astype(np.float32)
    return learned.make_mlp(dim, w, **standard), w


def descriptors(x, types, L, dim):
    """The 64 descriptors of every atom (radial by species, angular), FP64."""
    pot = LJParams()
    H = torch.tensor(box_of(dim, L), dtype=torch.float64, device="cuda")
    p = Pairs(x[None], types, H, pot, skin=0.0)
    out = []
    w = (2.5 - 0.6) / 23.0
    mu = 0.6 + w * torch.arange(24, dtype=torch.float64, device="cuda")
    if dim == 2:
        an = 2.0 * math.pi * torch.arange(16, dtype=torch.float64, device="cuda") / 16.0
        dirs = torch.stack([an.cos(), an.sin()], -1)
    else:
        k = torch.arange(16, dtype=torch.float64, device="cuda")
        z = 1.0 - (2.0 * k + 1.0) / 16.0
        phi = k * math.pi * (3.0 - math.sqrt(5.0))
        dirs = torch.stack([(1 - z * z).sqrt() * phi.cos(), (1 - z * z).sqrt() * phi.sin(), z], -1)
    dr = p.separations(x[None])
    r2 = sum(q * q for q in dr)
    inside = r2 < p.rc2
    r = torch.where(inside, r2, torch.ones_like(r2)).sqrt()
    fc = torch.where(inside, 0.5 * ((math.pi * r / p.rc2.clamp(min=1e-9).sqrt()).cos() + 1.0), torch.zeros_like(r))
    for s in (0, 1):
        fs = torch.where(p.tj == s, fc, torch.zeros_like(fc))
        for b in range(24):
            out.append(((-(r - mu[b]) ** 2 / (2.0 * w * w)).exp() * fs).sum(1))
    for k in range(16):
        c = (sum(q * float(dirs[k, a]) for a, q in enumerate(dr)) / r).clamp(min=0.0)
        out.append((fc * c * c).sum(1))
    return torch.stack(out, -1)


# ---------------------------------------------------------------------------
# Cases


def sizes_of(case):
    """Atoms of every replica: equal, or spread over their logarithm up to n_max."""
    R, n, top = case["replicas"], case["n"], case["n_max"]
    if not top:
        return [n] * R
    return [int(round(n * (top / n) ** (i / (R - 1)))) for i in range(R)]


def chain_inputs(case, seed):
    """Per group of equal replicas: (x (S, n, d), types, L)."""
    if case.get("copies"):
        return [glass_inputs(case["glass"], case["dim"], case["n"], 1, 100 * seed)]
    if case["n_max"]:
        return [glass_inputs(case["glass"], case["dim"], n, 1, 100 * seed + i) for i, n in enumerate(sizes_of(case))]
    return [glass_inputs(case["glass"], case["dim"], case["n"], case["replicas"], 100 * seed)]


def shear_of(case):
    return ((0.0, case["dgamma"]), (0.5 * case["dgamma"] if case.get("pure") else 0.0, 0.0))


def wrapped(eng, slot):
    """The slot's positions in its cell, as a program stores them."""
    H = eng.box(slot)
    s = eng.positions(slot) @ np.linalg.inv(H).T
    return (s - np.floor(s)) @ H.T


def padded(values, length, fill):
    """The values of the accepted steps (or the decisions) of a round, in an array of the most there can be."""
    return np.array(list(values) + [fill] * (length - len(values)))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("chain", "step", "round"):
        if kind != "round":
            groups, slots = chain_inputs(case, seed), case["replicas"]
            atoms, edges = sizes_of(case), [L for x, _, L in groups for _ in range(x.shape[0])]
            edges = edges * slots if case.get("copies") else edges
            where = list(range(slots))
        else:
            groups = [glass_inputs(case["glass"], case["dim"], case["n"], case["glasses"], 100 * seed)]
            slots = parallel.slots_needed(case["glasses"], case["P"])
            atoms, edges = [case["n"]] * slots, [groups[0][2]] * slots
            where = [g.star for g in parallel.layout(case["glasses"], case["P"])]
        tuning = None if case.get("tuning") == "default" else "auto"
        eng = Engine(case["dim"], atoms, np.array([[L] * case["dim"] for L in edges]), case["dgamma"],
                     pot=potential_of(case["glass"]), fire=Fire(max_iter=case.get("max_iter", 1_000_000)), tuning=tuning)
        if case.get("pure"):
            eng.set_pure_shear(list(range(slots)), 0.5 * case["dgamma"])
        if case.get("minimizer") == "cg":
            eng.set_minimizer("cg", Cg(max_iter=case["max_iter"]))
        if case.get("start") == "learned":
            eng.learned_load(network(case["dim"], seed)[0])
        loads = [(t.cpu().numpy(), x[s].cpu().numpy()) for x, t, _ in groups for s in range(x.shape[0])]
        return {"case": case, "eng": eng, "loads": list(zip(where, loads))}
    if kind == "evaluate":
        x, types, L = lattice_inputs(case["dim"], case["m"], seed, 1e-3 * case["strain"])
        eng = Engine(case["dim"], [x.shape[0]], L, 1e-3, tuning="auto")
        return {"case": case, "eng": eng, "types": types.cpu().numpy(), "x": x.cpu().numpy()}
    if kind == "learned":
        x, types, L = lattice_inputs(case["dim"], case["m"], seed)
        f = descriptors(x, types, L, case["dim"])
        eng = Engine(case["dim"], [x.shape[0]], L, 1e-4, tuning="auto")
        eng.learned_load(network(case["dim"], seed, feat_mean=f.mean(0).cpu().numpy(),
                                 feat_std=f.std(0).clamp(min=1e-3).cpu().numpy())[0])
        n = x.shape[0]
        return {"case": case, "eng": eng, "types": types.cpu().numpy(), "x": x.cpu().numpy(),
                "features": torch.empty((n, 64), dtype=torch.float32, device="cuda"),
                "u": torch.empty((n, case["dim"]), dtype=torch.float32, device="cuda")}
    feat, target, orders = train_inputs(case, seed)
    return {"case": case, "feat": feat, "target": target, "orders": orders, "init": network(case["dim"], seed)[1]}


def train_inputs(case, seed):
    """Features of the descriptors' spread and a smooth displacement field of them with a few plastic outliers."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    n, d = case["samples"], case["dim"]
    base = torch.randn((n, 12), generator=gen, device="cuda")
    mix = torch.randn((12, 64), generator=gen, device="cuda")
    feat = 3.0 + 0.4 * (base @ mix) + 0.3 * torch.randn((n, 64), generator=gen, device="cuda")
    target = torch.tanh(base[:, :d] + 0.5 * base[:, d:2 * d] * base[:, 2 * d:3 * d]) \
        + 0.1 * torch.randn((n, d), generator=gen, device="cuda")
    target[:: 997] *= 40.0
    orders = torch.stack([torch.randperm(n, generator=gen, device="cuda") for _ in range(case["epochs"])]).to(torch.int32)
    return feat.contiguous(), target.contiguous(), orders.contiguous()


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "chain":
        eng = state["eng"]
        for slot, (types, x) in state["loads"]:
            eng.set_replica(slot, types, x)
        slots = [slot for slot, _ in state["loads"]]
        rec = eng.minimize(slots, n_steps=[case["steps"]] * len(slots), start=STARTS[case["start"]])
        end = [wrapped(eng, s) for s in slots]
        return {"energy": rec["energy"], "sigma_xy": rec["sigma_xy"], "converged": rec["status"],
                "positions": end if case["n_max"] else np.stack(end)}
    if kind == "step":
        eng = state["eng"]
        for slot, (types, x) in state["loads"]:
            eng.set_replica(slot, types, x)
        slots = list(range(case["replicas"]))
        if case["copies"]:
            for s in slots[1:]:
                eng.copy_replica(0, s)
        eng.affine_shear(slots, [1 + (20 * s if case["copies"] else 0) for s in slots])
        rec = eng.minimize(slots)
        end = [wrapped(eng, s) for s in slots]
        return {"energy": rec["energy"], "sigma_xy": rec["sigma_xy"], "status": rec["status"],
                "positions": end if case["n_max"] else np.stack(end)}
    if kind == "round":
        eng = state["eng"]
        for slot, (types, x) in state["loads"]:
            eng.set_replica(slot, types, x)
        glasses = parallel.layout(case["glasses"], case["P"])
        parallel.run(eng, glasses, case["P"] * case["K"], case["K"], case["P"], start=STARTS[case["start"]], max_rounds=1,
                     live=case["live"])
        return {"accepted": [g.n_current for g in glasses],
                "equal": np.stack([padded([int(d.equal) for d in g.decisions], case["P"], -1) for g in glasses]),
                "energy": np.stack([padded(g.energies, case["P"] * case["K"], 0.0) for g in glasses]),
                "sigma_xy": np.stack([padded(g.sigma_xy, case["P"] * case["K"], 0.0) for g in glasses]),
                "positions": np.stack([wrapped(eng, g.star) for g in glasses])}
    if kind == "evaluate":
        eng = state["eng"]
        eng.set_replica(0, state["types"], state["x"], case["strain"])
        energy, forces = eng.energy_forces(0)
        sigma, energy2 = eng.stress(0)
        return {"energy": energy, "forces": forces, "sigma": sigma, "energy2": energy2}
    if kind == "learned":
        eng = state["eng"]
        eng.set_replica(0, state["types"], state["x"])
        return {"features": eng.learned_features(0, out=state["features"]), "u": eng.learned_predict(0, out=state["u"])}
    model = learned.make_mlp(case["dim"], state["init"])
    loss = learned.train(model, state["feat"], state["target"], state["orders"],
                         learned.TrainParams(batch=case["batch"], epochs=case["epochs"]))
    return {"loss": loss, **learned.mlp_arrays(model)}


def work(case):
    """Per force evaluation and atom: positions, velocities and types read, forces, velocities and positions written
    (145 B in 3D, 97 B in 2D), and each pair in the cutoff once (about 1100 and 310 flops); the evaluations are the
    typical ones of these glasses."""
    kind, dim = case["kind"], case.get("dim", 3)
    per_b, per_f = (145.0, 1100.0) if dim == 3 else (97.0, 310.0)
    if kind in ("chain", "step", "round"):
        def iters(n):
            return 300.0 * (n / 1500.0) ** 0.35 if dim == 3 else 400.0 * (n / 256.0) ** 0.44
        if kind == "chain":
            evals = sum(n * iters(n) for n in sizes_of(case)) * (0.5 + case["steps"])
        elif kind == "step":
            evals = sum(sizes_of(case)) * float(case["max_iter"])
        else:
            evals = case["glasses"] * case["P"] * (1 + case["K"]) * case["n"] * iters(case["n"])
        if case["glass"] == "paper":
            evals *= 2.0
        return {"bytes": per_b * evals, "flops": per_f * evals}
    if kind == "evaluate":
        n = case["m"] ** dim
        return {"bytes": n * (16.0 * dim + 1.0) + n * (8.0 * dim + 1.0), "flops": 2.0 * n * per_f}
    if kind == "learned":
        n = case["m"] ** dim
        pairs = 64.0 if dim == 3 else 18.0
        return {"bytes": n * (2.0 * (8.0 * dim + 1.0) + 256.0 + 4.0 * dim),
                "flops": n * (pairs * 2.0 * 64.0 * 3.0 + 2.0 * (64 * 128 + 128 * 128 + 128 * dim))}
    n = float(case["samples"])
    return {"bytes": n * (256.0 + 4.0 * dim) + case["epochs"] * n * (128.0 + 16.0 + 4.0),
            "flops": 6.0 * case["epochs"] * n * (64 * 128 + 128 * 128 + 128 * dim)}


# ---------------------------------------------------------------------------
# The same in 64 bits


def exact(case, seed):
    kind = case["kind"]
    if kind == "chain":
        return exact_chain(case, seed)
    if kind == "evaluate":
        x, types, L = lattice_inputs(case["dim"], case["m"], seed, 1e-3 * case["strain"])
        H = torch.tensor(box_of(case["dim"], L, ((0.0, 1e-3), (0.0, 0.0)), case["strain"]), dtype=torch.float64, device="cuda")
        F, e, W = Pairs(x[None], types, H, LJParams(), skin=0.0).forces(x[None], energy=True)
        return {"energy": float(e), "forces": F[0], "sigma": W[0] / float(L ** case["dim"]), "energy2": float(e)}
    if kind == "learned":
        x, types, L = lattice_inputs(case["dim"], case["m"], seed)
        f = descriptors(x, types, L, case["dim"])
        mean, std = f.mean(0).float().double(), f.std(0).clamp(min=1e-3).float().double()
        w = {k: torch.tensor(v, dtype=torch.float64, device="cuda") for k, v in network(case["dim"], seed)[1].items()}
        return {"features": f, "u": forward((f - mean) / std, w)}
    if kind == "train":
        return exact_train(case, seed)
    return None  # a step: cut at a number of iterations; a round: as many minimisations as its chains, and which of them stay follows from their checks


def exact_chain(case, seed):
    """Energies, stresses and positions of the inherent structures."""
    if sum(sizes_of(case)) * (1 + case["steps"]) > 120000:
        return None  # over 20 seconds of FIRE in torch
    pot, dim = potential_of(case["glass"]), case["dim"]
    shear = shear_of(case)
    F = torch.eye(dim, dtype=torch.float64, device="cuda")
    F[0, 1], F[1, 0] = shear[0][1], shear[1][0]
    energy, sigma, end = [], [], []
    for x, types, L in chain_inputs(case, seed):
        es, ss = [], []
        for k in range(case["steps"] + 1):
            if k:
                x = x @ F.T
            Hn = box_of(dim, L, shear, k)
            H = torch.tensor(Hn, dtype=torch.float64, device="cuda")
            x = relax(x, types, H, pot, 1e-10, 6000)
            _, e, W = Pairs(x, types, H, pot, skin=0.0).forces(x, energy=True)
            es.append(e)
            ss.append(W[:, 0, 1] / float(abs(np.linalg.det(Hn))))
        energy.append(torch.stack(es, 1))
        sigma.append(torch.stack(ss, 1))
        f = x @ torch.linalg.inv(H).T
        end.append((f - f.floor()) @ H.T)
    return {"energy": torch.cat(energy), "sigma_xy": torch.cat(sigma), "converged": None, "positions": torch.cat(end)}


def forward(z, w):
    h = torch.nn.functional.silu(z @ w["w1"] + w["b1"])
    h = torch.nn.functional.silu(h @ w["w2"] + w["b2"])
    return h @ w["w3"] + w["b3"]


def exact_train(case, seed):
    """Adam on the Huber loss of the samples within five deviations of the targets' trimmed mean."""
    feat, target, orders = (t.double() if t.is_floating_point() else t.long() for t in train_inputs(case, seed))
    w = {k: torch.tensor(v, dtype=torch.float64, device="cuda", requires_grad=True)
         for k, v in network(case["dim"], seed)[1].items()}

    def spread(t):
        return t.mean(0), t.std(0, unbiased=False)

    fm, fs = spread(feat)
    keep = torch.ones(feat.shape[0], dtype=torch.bool, device="cuda")
    tm, ts = spread(target)
    for _ in range(3):
        keep = ((target - tm).abs() <= 5.0 * ts).all(1)
        tm, ts = spread(target[keep])
    keep = ((target - tm).abs() <= 5.0 * ts).all(1)
    z, t = (feat - fm) / fs, (target - tm) / ts
    p = learned.TrainParams()
    state = {k: [torch.zeros_like(v), torch.zeros_like(v)] for k, v in w.items()}
    losses, step = [], 0
    for e in range(case["epochs"]):
        got = []
        for b in range(0, z.shape[0], case["batch"]):
            i = orders[e, b:b + case["batch"]]
            err = (forward(z[i], w) - t[i])[keep[i]]
            loss = torch.where(err.abs() <= 1.0, 0.5 * err * err, err.abs() - 0.5).sum() / (i.numel() * case["dim"])
            grads = torch.autograd.grad(loss, list(w.values()))
            got.append(float(loss))
            step += 1
            with torch.no_grad():
                for (k, v), g in zip(w.items(), grads):
                    m = state[k]
                    m[0] = p.beta1 * m[0] + (1.0 - p.beta1) * g
                    m[1] = p.beta2 * m[1] + (1.0 - p.beta2) * g * g
                    v -= p.lr * (m[0] / (1.0 - p.beta1 ** step)) / ((m[1] / (1.0 - p.beta2 ** step)).sqrt() + p.eps)
        losses.append(sum(got) / len(got))
    return {"loss": np.array(losses), **{k: v.detach() for k, v in w.items()}, "feat_mean": fm, "feat_std": fs,
            "tgt_mean": tm, "tgt_std": ts}
