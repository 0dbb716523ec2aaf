"""What a user of the MD library has it do, as cases that can be timed.

Every case goes through the public Python entry points (paper_0912_3824_amd.mdx
and .serve) and ends with the frames (positions, velocities, image counters)
or curves that the program asked for.  The kinds of pass:

  run      advance one or more replicas, `reads` observations on the way (0 =
           none), then read every replica's frame
  bath     the same through the Andersen heat bath, a thermostat call every
           `every` steps
  curves   a production run with time-correlation functions sampled every
           `every` steps
  forces   the library as a force engine: attach a configuration, evaluate its
           forces and energies, detach it
  serve    trajectory jobs through the continuous-batching server

Inputs are made from the seed alone: jittered face-centred lattices (a random
subset of the sites where N is not 4 n^3) with Maxwell-Boltzmann velocities,
the Kob-Andersen 80/20 mixture at density 1.2 or the one-species Lennard-Jones
fluid.  A pass continues the trajectory of the one before, as a program's next
chunk of steps does.
"""
import math
import types

import numpy as np
import torch

from paper_0912_3824_amd import mdx, serve, tune

DT = 0.001
# aligned-rebuild policy of replica ensembles (every, fraction of skin/2)
ALIGNED = (12, 0.5)


def listed():
    def case(name, kind, **kw):
        c = {"name": name, "kind": kind, "model": "ka", "precision": "ds", "n": 0, "n_hi": 0, "replicas": 1,
             "temperature": 0.7, "steps": 0, "reads": 0, "every": 0, "skin": 0.3, "smooth": 0.0, "lanes": 0,
             "order": "row", "aligned": False}
        c.update(kw)
        return c

    return [
        # the smallest replica that is of use: one cell, a handful of steps between
        # two frames, so launches and latency are all there is
        case("single_cell_ds", "run", n=600, temperature=0.6, steps=20),
        # a small one-species fluid in double precision: 1 ms of reference trajectory
        case("lj4000_fp64", "run", model="lj", n=4000, temperature=1.5, precision="fp64", steps=200, lanes=4),
        # an energy-conservation study: the smoothed fluid, energies read every 10 steps
        case("energies_10k_fp32", "run", model="fluid", n=10000, temperature=1.12, precision="fp32", steps=200,
             reads=20, smooth=0.005),
        # equilibration in the heat bath, odd size, single precision
        case("bath_37k_fp32", "bath", n=37111, temperature=0.6, precision="fp32", steps=400, every=100),
        # the mixture at the size its glassy dynamics are studied at: frames 500 steps apart
        case("ka64k_ds", "run", n=64000, steps=500),
        # drift measurement: eight replicas advanced together, energies every 100 steps
        case("drift_8x64k_mixed64", "run", n=64000, replicas=8, precision="mixed64", steps=300, reads=3),
        # a large double-precision run along the Hilbert curve
        case("ka200k_fp64_hilbert", "run", n=200000, temperature=0.5, precision="fp64", steps=200, order="hilbert"),
        # the headline system
        case("ka1m_ds", "run", n=1000000, temperature=0.5, steps=400),
        # an ensemble of replicas of many sizes and temperatures, rebuilding together
        case("ensemble256_ds", "run", n=500, n_hi=8000, replicas=256, temperature=0.0, steps=240, skin=0.4,
             aligned=True),
        # production run: mean-square displacement, velocity autocorrelation and F_s(q, t)
        case("curves_250k_ds", "curves", n=250000, temperature=0.5, steps=200, every=10),
        # forces and energies of configurations that come from outside
        case("forces_120k_ds", "forces", n=120011, temperature=0.5),
        # jobs of many sizes served from one pool
        case("serve_ds", "serve", n=1000, n_hi=64000, replicas=12, temperature=0.0, steps=600),
    ]


def draw(rng):
    """Sizes spread over their logarithm, every kind, precision and option."""
    kind = rng.choice(["run", "run", "run", "run", "bath", "curves", "forces", "ensemble", "serve"])
    log_uniform = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    c = {"kind": kind, "model": rng.choice(["ka", "ka", "lj", "fluid"]), "precision": "ds", "n": 0, "n_hi": 0,
         "replicas": 1, "temperature": round(rng.uniform(0.45, 1.0), 3), "steps": 0, "reads": 0, "every": 0,
         "skin": rng.choice([0.25, 0.3, 0.3, 0.3, 0.4]), "smooth": 0.0, "lanes": 0, "order": "row",
         "aligned": False}
    c["precision"] = rng.choice(["ds", "ds", "fp32", "mixed64", "fp64"])
    if kind in ("ensemble", "serve"):
        c["model"], c["temperature"] = "ka", 0.0
        c["n"] = log_uniform(500, 1500)
        c["n_hi"] = c["n"] * rng.choice([4, 16, 32])
        if kind == "ensemble":
            c["kind"] = "run"
            c["n_hi"] = min(c["n_hi"], 8000)
            c["replicas"] = log_uniform(8, 256)
            c["steps"] = log_uniform(60, 240)
            c["aligned"] = rng.random() < 0.5
        else:
            c["replicas"] = rng.randint(4, 12)
            c["steps"] = log_uniform(200, 600)
        return c
    c["n"] = log_uniform(500, 900000)
    if kind == "run":
        c["lanes"] = rng.choice([0, 0, 0, 1, 4])
        c["order"] = rng.choice(["row", "row", "row", "morton", "hilbert"])
        c["steps"] = log_uniform(20, min(500.0, (1.2e8 if c["precision"] == "fp64" else 2.5e8) / c["n"]))
        c["reads"] = rng.choice([0, 0, 2, 5]) if c["steps"] >= 40 else 0
        c["smooth"] = 0.005 if c["model"] == "fluid" else rng.choice([0.0, 0.0, 0.01])
        if c["n"] < 40000 and rng.random() < 0.3:
            c["replicas"] = rng.randint(2, 8)
    elif kind == "bath":
        c["n"] = log_uniform(500, 300000)
        c["every"] = rng.choice([20, 50, 100])
        c["steps"] = c["every"] * rng.randint(2, 4)
    elif kind == "curves":
        c["n"] = log_uniform(1000, 250000)
        c["every"] = rng.choice([5, 10, 20])
        c["steps"] = c["every"] * rng.randint(10, 15)
    else:
        c["n"] = log_uniform(500, 300000)
    return c


# ------------------------------------------------------------------- inputs
def _table(case):
    """Pair parameters: the Kob-Andersen mixture, or one species with the
    Lennard-Jones cutoff 2.5 ("lj", and "fluid" at the lower density)."""
    if case["model"] == "ka":
        sig = np.array([[1.0, 0.8], [0.8, 0.88]])
        return types.SimpleNamespace(n_species=2, eps=np.array([[1.0, 1.5], [1.5, 0.5]]), sigma=sig,
                                     rcut=2.5 * sig, smooth=case["smooth"])
    one = np.ones((2, 2))
    return types.SimpleNamespace(n_species=1, eps=one, sigma=one, rcut=2.5 * one, smooth=case["smooth"])


def _system(case, n, temperature, rng):
    """One replica: jittered lattice sites, species by a random permutation,
    velocities of zero sum rescaled to the temperature."""
    rho = {"ka": 1.2, "lj": 0.8442, "fluid": 0.75}[case["model"]]
    box = float(np.float32((n / rho) ** (1.0 / 3.0)))
    nc = int(math.ceil((n / 4.0) ** (1.0 / 3.0) - 1e-9))
    basis = np.array([[0.25, 0.25, 0.25], [0.75, 0.75, 0.25], [0.75, 0.25, 0.75], [0.25, 0.75, 0.75]])
    g = np.arange(nc)
    cells = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 1, 3)
    sites = (cells + basis).reshape(-1, 3) * (box / nc)
    if len(sites) > n:
        keep = np.ones(len(sites), dtype=bool)
        keep[rng.permutation(len(sites))[n:]] = False
        sites = sites[keep]
    pos = np.mod(sites + rng.uniform(-0.06, 0.06, size=sites.shape), box)
    pos[pos >= box] = 0.0
    vel = rng.normal(size=(n, 3))
    vel -= vel.mean(axis=0)
    vel *= math.sqrt(3.0 * n * temperature / float(np.sum(vel * vel)))
    species = np.zeros(n, dtype=np.int32)
    if case["model"] == "ka":
        species[rng.permutation(n)[int(round(0.8 * n)):]] = 1
    return types.SimpleNamespace(n=n, box=box, pos=pos, vel=vel, species=species, temperature=temperature)


def _systems(case, seed):
    """The replicas (or jobs) of a case: one size, or sizes spread over the
    logarithm of [n, n_hi] with temperatures of their own."""
    rng = np.random.default_rng([int(seed), 912])
    out = []
    for k in range(case["replicas"]):
        n, t = case["n"], case["temperature"]
        if case["n_hi"]:
            # the sizes are the case's, so that every seed has the same work
            n = int(round(math.exp(math.log(n) + (k + 0.5) / case["replicas"] * math.log(case["n_hi"] / n))))
            t = (0.45, 0.5, 0.6, 0.8)[k % 4]
        out.append(_system(case, n, t, rng))
    if case["n_hi"]:  # large and small ones mixed, for every seed alike
        out = [out[k] for k in np.random.default_rng(5).permutation(len(out))]
    return out


def _job_steps(case, k):
    """Steps of the k-th job of a served case: half to all of `steps`."""
    return case["steps"] * (case["replicas"] + k) // (2 * case["replicas"])


# ----------------------------------------------------------------- the passes
def prepare(case, seed):
    systems = _systems(case, seed)
    total = sum(s.n for s in systems)
    every, early = ALIGNED if case["aligned"] else (0, 0.0)
    st = {"case": case, "systems": systems, "call": 0}
    if case["kind"] == "serve":
        # the arena holds about half of the jobs at a time
        st["server"] = serve.Server(_table(case), case["precision"], skin=case["skin"],
                                    max_slots=max(2, case["replicas"] // 2),
                                    max_particles=max(max(s.n for s in systems), total // 2),
                                    make_system=lambda job: systems[job.job_id])
        return st
    cfg = mdx.make_config(_table(case), case["precision"], DT, case["skin"], len(systems), total,
                          lanes_per_particle=case["lanes"], cell_order=case["order"], rebuild_every=every,
                          rebuild_early=early)
    st["pool"] = pool = mdx.MdSystem(cfg)
    if case["kind"] != "forces":
        for k, s in enumerate(systems):
            pool.attach_system(k, s)
        tune.apply_cached(pool)
    if case["kind"] == "curves":
        # wave number of the first peak of the structure factor, on the box's grid
        q = 2 * math.pi * max(1, round(7.25 * systems[0].box / (2 * math.pi))) / systems[0].box
        st["tcf"] = pool.tcf(0, 4, 10, q)
    return st


def _frames(pool, count):
    frames = [pool.get_state(k) for k in range(count)]
    if count == 1:
        return dict(zip(("pos", "vel", "image"), frames[0]))
    return {key: np.concatenate([f[i] for f in frames]) for i, key in enumerate(("pos", "vel", "image"))}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        jobs = [types.SimpleNamespace(job_id=k, arrival=0.0, steps=_job_steps(case, k), tcf_every=0)
                for k in range(case["replicas"])]
        results = state["server"].run(jobs)["results"]
        return {key: np.concatenate([getattr(r, key) for r in results]) for key in ("pos", "vel", "image")}
    pool = state["pool"]
    if kind == "forces":
        s = state["systems"][0]
        pool.attach_system(0, s)
        f, e = pool.forces(0)
        pool.detach(0)
        return {"forces": f, "energies": e}
    if kind == "bath":
        state["call"] = pool.andersen(0, case["temperature"], 1.0 / (case["every"] * DT), case["steps"], 4711,
                                      first_call=state["call"])
        return _frames(pool, 1)
    if kind == "curves":
        for _ in range(case["steps"] // case["every"]):
            state["tcf"].sample()
            pool.step(case["every"])
        lags, values, terms = state["tcf"].read()
        return {"lags": lags, "curves": values, "terms": terms, **_frames(pool, 1)}
    reads, out = [], {}
    if case["reads"]:
        for _ in range(case["reads"]):
            pool.step(case["steps"] // case["reads"])
            reads.append(pool.observables())
        for key in ("epot", "ekin", "virial", "pressure"):
            out[key] = np.array([[o[key] for o in r] for r in reads])
    else:
        pool.step(case["steps"])
    out.update(_frames(pool, case["replicas"]))
    return out


def work(case):
    """Per step: the state read and written once, and one evaluation of every
    pair inside the cutoff (about 20 flops for the separation and the test and
    20 for the pair term, by Newton's third law once per pair); per frame: the
    state read and 60 bytes a particle written; per correlation sample: the
    pass over the stored lags."""
    rho = {"ka": 1.2, "lj": 0.8442, "fluid": 0.75}[case["model"]]
    sizes = [case["n"]] * case["replicas"]
    if case["n_hi"]:
        sizes = [case["n"] * math.exp((k + 0.5) / case["replicas"] * math.log(case["n_hi"] / case["n"]))
                 for k in range(case["replicas"])]
    # neighbours inside the cutoff: for the mixture the mean of 2.5 sigma_ab over species
    mean_rc3 = (0.64 + 0.32 * 0.8 ** 3 + 0.04 * 0.88 ** 3 if case["model"] == "ka" else 1.0) * 2.5 ** 3
    pairs = 0.5 * 4.0 / 3.0 * math.pi * mean_rc3 * rho
    word = 24 if case["precision"] == "fp32" else 48
    if case["kind"] == "forces":
        return {"bytes": sizes[0] * (52 + 32), "flops": sizes[0] * pairs * 40}
    steps = [_job_steps(case, k) if case["kind"] == "serve" else case["steps"] for k in range(case["replicas"])]
    moved = sum(n * k for n, k in zip(sizes, steps))
    byts = moved * 2 * word + sum(sizes) * (word + 60)
    flops = moved * pairs * 40
    if case["kind"] == "curves":
        samples = case["steps"] // case["every"]
        byts += sizes[0] * 48 * (samples + 10 * max(0, samples - 9))
        flops += sizes[0] * 60 * 9 * max(0, samples - 9)
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------------- the same in 64 bits
class _Reference:
    """Velocity Verlet in double precision over padded neighbour tables, in
    plain torch: all replicas of a case as one flat set of particles."""

    LIST_SKIN = 0.55

    def __init__(self, case, systems):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t = _table(case)
        dev64 = dict(dtype=torch.float64, device=self.dev)
        self.eps, self.sig, self.rc = (torch.as_tensor(np.ascontiguousarray(x), **dev64).reshape(4)
                                       for x in (t.eps, t.sigma, t.rcut))
        s2 = (self.sig / self.rc) ** 2
        self.shift = 4 * self.eps * (s2 ** 6 - s2 ** 3)
        self.rc_max = float(np.max(t.rcut[:t.n_species, :t.n_species]))
        self.h = float(case["smooth"])
        self.sizes = [s.n for s in systems]
        self.boxes = [s.box for s in systems]
        cat = lambda key: torch.as_tensor(np.concatenate([getattr(s, key) for s in systems]), device=self.dev)  # noqa: E731
        self.x, self.v, self.sp = cat("pos").double(), cat("vel").double(), cat("species").long()
        self.box = torch.cat([torch.full((n,), b, **dev64) for n, b in zip(self.sizes, self.boxes)])[:, None]
        self.ref = None

    def _pairs_brute(self, x, L, r):
        rows = max(1, int(4e7) // len(x))
        for a in range(0, len(x), rows):
            d = x[a:a + rows, None, :] - x[None, :, :]
            d -= L * torch.round(d / L)
            i, j = torch.nonzero((d * d).sum(-1) < r * r, as_tuple=True)
            yield i + a, j

    def _pairs_cells(self, x, L, r):
        nd = int(L / r)
        w = torch.remainder(x, L)
        c = (w * (nd / L)).long().clamp_(0, nd - 1)
        key = c[:, 0] + nd * (c[:, 1] + nd * c[:, 2])
        order = torch.argsort(key)
        count = torch.bincount(key, minlength=nd ** 3)
        start = torch.cumsum(count, 0) - count
        m = int(count.max())
        table = torch.full((nd ** 3, m), -1, dtype=torch.long, device=x.device)
        sk = key[order]
        table[sk, torch.arange(len(x), device=x.device) - start[sk]] = order
        cell = torch.arange(nd ** 3, device=x.device)
        cx, cy, cz = cell % nd, (cell // nd) % nd, cell // (nd * nd)
        rows = max(1, int(4e7) // (m * m))
        for k in range(27):
            o = (cx + k % 3 - 1) % nd + nd * ((cy + k // 3 % 3 - 1) % nd + nd * ((cz + k // 9 - 1) % nd))
            for a in range(0, nd ** 3, rows):
                i, j = table[a:a + rows, :, None], table[o[a:a + rows]][:, None, :]
                d = x[i.clamp(min=0)] - x[j.clamp(min=0)]
                d -= L * torch.round(d / L)
                near = ((d * d).sum(-1) < r * r) & (i >= 0) & (j >= 0)
                p, q, s = torch.nonzero(near, as_tuple=True)
                yield i[p, q, 0], j[p, 0, s]

    def _lists(self):
        """nbr[k, i]: the k-th neighbour of i within the cutoff plus the
        list's skin, itself where there is none."""
        r, off, ii, jj = self.rc_max + self.LIST_SKIN, 0, [], []
        for n, L in zip(self.sizes, self.boxes):
            x = self.x[off:off + n]
            for i, j in (self._pairs_cells if n > 3000 and L / r >= 3 else self._pairs_brute)(x, L, r):
                keep = i != j
                ii.append(i[keep] + off)
                jj.append(j[keep] + off)
            off += n
        i, j = torch.cat(ii), torch.cat(jj)
        i, by = torch.sort(i)
        j = j[by]
        count = torch.bincount(i, minlength=off)
        start = torch.cumsum(count, 0) - count
        self.nbr = torch.arange(off, device=self.dev).repeat(int(count.max()), 1)
        self.nbr[torch.arange(len(i), device=self.dev) - start[i], i] = j
        self.ref = self.x.clone()

    def forces(self, energies=False):
        """Forces, and energies and virials per particle when asked for."""
        n = len(self.x)
        f = torch.empty_like(self.x)
        e = torch.zeros(n, dtype=torch.float64, device=self.dev)
        w = torch.zeros_like(e)
        cols = max(1, int(3e7) // len(self.nbr))
        me = torch.arange(n, device=self.dev)
        for a in range(0, n, cols):
            b = min(n, a + cols)
            j = self.nbr[:, a:b]
            L = self.box[a:b, 0]
            d = [self.x[a:b, c] - self.x[:, c][j] for c in range(3)]
            d = [u - L * torch.round(u / L) for u in d]
            r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
            t = 2 * self.sp[a:b] + self.sp[j]
            rc = self.rc[t]
            inside = (r2 < rc * rc) & (j != me[a:b])
            r2 = torch.where(inside, r2, torch.ones_like(r2))
            sig, eps = self.sig[t], self.eps[t]
            s6 = (sig * sig / r2) ** 3
            ff = 24 * eps * s6 * (2 * s6 - 1) / r2
            if energies or self.h > 0:
                v = 4 * eps * s6 * (s6 - 1) - self.shift[t]
                if self.h > 0:
                    r = torch.sqrt(r2)
                    x = (r - rc) / (self.h * sig)
                    g = x ** 4 / (1 + x ** 4)
                    ff = ff * g - v * 4 * x ** 3 / (1 + x ** 4) ** 2 / (self.h * sig) / r
                    v = v * g
            ff = torch.where(inside, ff, torch.zeros_like(ff))
            for c in range(3):
                f[a:b, c] = (ff * d[c]).sum(0)
            if energies:
                e[a:b] = 0.5 * torch.where(inside, v, torch.zeros_like(v)).sum(0)
                w[a:b] = 0.5 * (ff * r2).sum(0)
        return (f, e, w) if energies else f

    def step(self, count):
        if self.ref is None:
            self._lists()
        f = self.forces()
        for k in range(count):
            self.v += 0.5 * DT * f
            self.x += DT * self.v
            # between two looks no particle moves more than 0.08
            if k % 8 == 0 and float(((self.x - self.ref) ** 2).sum(-1).max()) > (0.5 * self.LIST_SKIN - 0.08) ** 2:
                self._lists()
            f = self.forces()
            self.v += 0.5 * DT * f

    def frames(self):
        x = torch.remainder(self.x, self.box)
        return {"pos": x.cpu().numpy(), "vel": self.v.cpu().numpy(), "image": None}

    def observe(self):
        _, e, w = self.forces(energies=True)
        out, off = [], 0
        for n, L in zip(self.sizes, self.boxes):
            ekin = 0.5 * float((self.v[off:off + n] ** 2).sum())
            vir = float(w[off:off + n].sum())
            out.append((float(e[off:off + n].sum()), ekin, vir, (2 * ekin + vir) / (3 * L ** 3)))
            off += n
        return out

    def heat_bath(self, temperature, seed, call):
        """Velocities of the thermostat: rand48 elements i + n (4 call + r),
        Box-Muller, zero sum, rescaled to the temperature."""
        n = self.sizes[0]
        mask = np.uint64((1 << 48) - 1)
        u = []
        for r in range(4):
            j = np.arange(n, dtype=np.uint64) + np.uint64(n * (4 * call + r))
            A, C = np.ones(n, dtype=np.uint64), np.zeros(n, dtype=np.uint64)
            a, c = 0x5DEECE66D, 0xB
            while j.any():
                odd = (j & np.uint64(1)).astype(bool)
                A[odd] = (A[odd] * np.uint64(a)) & mask
                C[odd] = (C[odd] * np.uint64(a) + np.uint64(c)) & mask
                a, c = (a * a) & int(mask), (a * c + c) & int(mask)
                j >>= np.uint64(1)
            x0 = np.uint64(((seed & 0xFFFFFFFF) << 16) | 0x330E)
            u.append(((A * x0 + C) & mask).astype(np.float64) / 2.0 ** 48)
        ra, rb = np.sqrt(-2 * np.log(1 - u[0])), np.sqrt(-2 * np.log(1 - u[2]))
        v = np.stack([ra * np.cos(2 * np.pi * u[1]), ra * np.sin(2 * np.pi * u[1]), rb * np.cos(2 * np.pi * u[3])], 1)
        v -= v.mean(axis=0)
        v *= math.sqrt(3.0 * n * temperature / float(np.sum(v * v)))
        self.v = torch.as_tensor(v, device=self.dev)


def _exact_curves(ref, case):
    """Blocking scheme of 4 levels of 10 entries over the trajectory."""
    q = 2 * math.pi * max(1, round(7.25 * ref.boxes[0] / (2 * math.pi))) / ref.boxes[0]
    ring, sums, passes = [[] for _ in range(4)], np.zeros((4, 9, 2, 3)), np.zeros((4, 9, 1, 1))
    masks = [ref.sp == s for s in range(2)]
    for m in range(case["steps"] // case["every"]):
        for lev in range(4):
            if m % 10 ** lev:
                break
            ring[lev] = ring[lev][-9:] + [(ref.x.clone(), ref.v.clone())]
            if len(ring[lev]) == 10:
                x0, v0 = ring[lev][0]
                for j in range(1, 10):
                    x, v = ring[lev][j]
                    d = x - x0
                    val = ((d * d).sum(-1), (v * v0).sum(-1), torch.cos(q * d).mean(-1))
                    for s in range(2):
                        if bool(masks[s].any()):
                            sums[lev, j - 1, s] += [float(z[masks[s]].mean()) for z in val]
                passes[lev] += 1
        ref.step(case["every"])
    with np.errstate(invalid="ignore", divide="ignore"):
        return sums / passes


def exact(case, seed):
    systems = _systems(case, seed)
    if case["kind"] == "serve":
        parts = []
        for k, s in enumerate(systems):
            ref = _Reference(case, [s])
            ref.step(_job_steps(case, k))
            parts.append(ref.frames())
        return {key: np.concatenate([p[key] for p in parts]) if key != "image" else None
                for key in ("pos", "vel", "image")}
    ref = _Reference(case, systems)
    if case["kind"] == "forces":
        ref._lists()
        f, e, _ = ref.forces(energies=True)
        return {"forces": f.cpu().numpy(), "energies": e.cpu().numpy()}
    if case["kind"] == "bath":
        for call in range(case["steps"] // case["every"]):
            ref.heat_bath(case["temperature"], 4711, call)
            ref.step(case["every"])
        return ref.frames()
    if case["kind"] == "curves":
        curves = _exact_curves(ref, case)
        return {"lags": None, "curves": curves, "terms": None, **ref.frames()}
    out = {}
    if case["reads"]:
        reads = []
        for _ in range(case["reads"]):
            ref.step(case["steps"] // case["reads"])
            reads.append(ref.observe())
        for k, key in enumerate(("epot", "ekin", "virial", "pressure")):
            out[key] = np.array([[o[k] for o in r] for r in reads])
    else:
        ref.step(case["steps"])
    out.update(ref.frames())
    return out
