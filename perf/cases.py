"""The work that programs have this library do, as cases to be timed.

A case is a dict of plain values.  prepare() makes a program's state for it
(a context with its topology, workspace and start coordinates, or particle
arrays) from a seed; run() is one pass through the public entry points, and
exact() what that pass returns, in 64 bits.

Kinds of case:
  md        one system stepped on the plain schedule, a frame (and, with
            `energy_every`, the energy record) read back after the pass
  ensemble  many independent chains stepped on the batched schedule
  exchange  the same with replica exchange over a temperature ladder
  score     forces and energies of a new conformation
  ramp      harmonic Brownian particles under a force ramp, with moments

A frame is kept as the displacement from the start, in single precision, as
a diffusion or unfolding analysis stores it; forces are the single-precision
numbers that the device computes.
"""
import math

import numpy as np
import torch

import paper_1003_1148_amd as sop

BOND, MIN_DIST, NATIVE = 3.8, 4.0, 8.0
KB = 0.0019872043  # kcal/mol/K
CANTILEVER = 0.05 * 6.02214076e23 / 4184.0 * 1e-20  # 0.05 N/m in kcal/mol/A^2


class Params:
    """Force field, thermostat and list (kcal/mol, A, reduced time)."""
    k_fene, R0, eps_h, eps_l, sigma, r_list = 14.0, 2.0, 1.0, 1.0, 3.8, 20.0
    kBT, zeta, h, list_every, list_capacity = KB * 300.0, 50.0, 0.08, 10, 0

    def __init__(self, seed):
        self.seed = 0x5EED0000 + seed


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _md(name, shape, n, steps, **kw):
    case = {"kind": "md", "shape": shape, "n": n, "steps": steps, "energy_every": 0, "skin": 4.0,
            "integrator": "overdamped", "pull": False, "tip": False}
    case.update(kw)
    return dict(case, name=name) if name else case


def listed():
    return [
        # a peptide-sized chain in a script's loop: the smallest call, launches and latency
        _md("chain 56", "chain", 56, 500),
        # a single protein domain stretched by a cantilever, force and energies logged
        _md("pulled globule 1000", "globule", 1000, 500, pull=True, energy_every=100),
        # one protein at folded density (over 100 list pairs a residue), ragged size
        _md("dense 4801", "dense", 4801, 100),
        # a medium complex with inertia
        _md("underdamped shell 20k", "shell", 80, 100, integrator="underdamped"),
        # the shell assembly under an indentation tip, as the benchmark steps it
        _md("shell 75k tip", "shell", 300, 500, tip=True, energy_every=1000, skin=6.0),
        # the largest single system: a long fibre, far from the origin
        _md("fibre 250k", "fibre", 1000, 200),
        # a cluster of short runs of one study: too few chains to fill the chip twice
        {"kind": "ensemble", "name": "ensemble 200", "traj": 200, "lmin": 50, "lmax": 500, "steps": 500,
         "energy_every": 0},
        # the many-runs-per-GPU ensemble of the benchmark
        {"kind": "ensemble", "name": "ensemble 4096", "traj": 4096, "lmin": 50, "lmax": 500, "steps": 500,
         "energy_every": 1000},
        # parallel tempering: 16 temperatures, 24 groups of a 137-residue chain
        {"kind": "exchange", "name": "tempering 24x16", "groups": 24, "reps": 16, "length": 137,
         "every": 50, "steps": 200},
        # rescoring conformations of a complex: new coordinates, then forces and energies
        {"kind": "score", "name": "score shell 10k", "shape": "shell", "n": 40},
        # the integrator-accuracy ensemble: 1e5 noisy particles with their moments
        {"kind": "ramp", "name": "ramp 100k", "n": 100_000, "steps": 1000, "order": 1, "noise": True,
         "compensated": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["md", "md", "md", "ensemble", "exchange", "score", "ramp"])
    if kind == "md":
        shape = rng.choice(["chain", "globule", "dense", "shell", "fibre"])
        n = {"chain": lambda: _log(rng, 20, 400), "globule": lambda: _log(rng, 200, 2000),
             "dense": lambda: _log(rng, 400, 12000), "shell": lambda: _log(rng, 12, 300),
             "fibre": lambda: _log(rng, 4, 1000)}[shape]()
        extra = {"energy_every": rng.choice([0, 0, 100, 1000]), "skin": rng.choice([4.0, 4.0, 6.0]),
                 "integrator": rng.choice(["overdamped"] * 3 + ["underdamped"])}
        if shape in ("chain", "globule"):
            extra["pull"] = rng.random() < 0.5
        if shape == "shell":
            extra["tip"] = rng.random() < 0.5
        return _md(None, shape, n, rng.choice([50, 100, 130, 200]), **extra)
    if kind == "ensemble":
        lmin = rng.randint(20, 200)
        return {"kind": kind, "traj": _log(rng, 16, 4000), "lmin": lmin, "lmax": rng.randint(lmin, 500),
                "steps": rng.choice([50, 100, 170, 200]), "energy_every": rng.choice([0, 100, 1000])}
    if kind == "exchange":
        return {"kind": kind, "groups": _log(rng, 2, 64), "reps": rng.randint(4, 24),
                "length": _log(rng, 30, 400), "every": rng.choice([20, 50]), "steps": 200}
    if kind == "score":
        shape = rng.choice(["globule", "dense", "shell", "fibre"])
        return {"kind": kind, "shape": shape,
                "n": {"globule": lambda: _log(rng, 100, 2000), "dense": lambda: _log(rng, 400, 12000),
                      "shell": lambda: _log(rng, 12, 200), "fibre": lambda: _log(rng, 4, 200)}[shape]()}
    return {"kind": "ramp", "n": _log(rng, 1000, 1_000_000), "steps": _log(rng, 100, 1000),
            "order": rng.choice([1, 2]), "noise": rng.random() < 0.8, "compensated": rng.random() < 0.8}


# ---------------------------------------------------------------------------
# structures
# ---------------------------------------------------------------------------

def _unit(rng, m):
    v = rng.standard_normal((m, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def _walk(n, rng, axes=None, batch=24):
    """A self-avoiding chain of n residues, inside an ellipsoid when axes are given."""
    X = np.zeros((n, 3))
    k, fails = 1, 0
    while k < n:
        c = X[k - 1] + BOND * _unit(rng, batch)
        ok = np.ones(batch, bool) if axes is None else ((c / axes) ** 2).sum(1) <= 1.0
        if k > 1:
            d = X[None, :k - 1] - c[:, None]
            ok &= ((d * d).sum(-1) >= MIN_DIST * MIN_DIST).all(1)
        if ok.any():
            X[k] = c[int(np.argmax(ok))]
            k, fails = k + 1, 0
        else:  # a dead end: back off and grow again
            fails += 1
            k = max(1, k - 2 ** min(fails, 6))
    return X


def _walks(m, n, rng):
    """m unconfined self-avoiding chains of n residues, grown together."""
    X = np.zeros((m, n, 3))
    X[:, 1] = BOND * _unit(rng, m)
    stuck = np.zeros(m, bool)
    for k in range(2, n):
        left, tries = np.nonzero(~stuck)[0], 0
        while left.size:
            c = X[left, k - 1] + BOND * _unit(rng, left.size)
            d = X[left, :k - 1] - c[:, None]
            ok = ((d * d).sum(-1) >= MIN_DIST * MIN_DIST).all(1)
            X[left[ok], k] = c[ok]
            left, tries = left[~ok], tries + 1
            if tries > 100:
                stuck[left] = True
                break
    for t in np.nonzero(stuck)[0]:
        X[t] = _walk(n, rng)
    return X


def _dense(n, rng):
    """A chain folded into antiparallel strands at 116 A^3 a residue."""
    lat = math.sqrt(116.0 / BOND)
    rows = max(2, round((n * 116.0) ** (1.0 / 3.0) / lat))
    per = max(4, math.ceil(n / (rows * rows)))
    k = np.arange(n)
    strand, at = k // per, k % per
    at = np.where(strand % 2 == 0, at, per - 1 - at)
    col, row = strand // rows, strand % rows
    row = np.where(col % 2 == 0, row, rows - 1 - row)
    X = np.stack([at * BOND, row * lat, col * lat], 1)
    return X + rng.uniform(-0.25, 0.25, X.shape)


def _turn(rng, m):
    """m random rotations."""
    q = rng.standard_normal((m, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                     2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                     2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(m, 3, 3)


def _contacts(X, apart=2):
    """Pairs i < j of one chain closer than the native cutoff, more than `apart` apart."""
    out = []
    for a in range(0, len(X), 512):
        d2 = np.full((min(512, len(X) - a), len(X)), 1e9)
        for ax in range(3):
            d = X[a:a + 512, ax, None] - X[None, :, ax]
            d2 = d * d if ax == 0 else d2 + d * d
        i, j = np.nonzero(d2 < NATIVE * NATIVE)
        keep = j > i + a + apart
        out.append(np.stack([i[keep] + a, j[keep]], 1))
    return np.concatenate(out)


class System:
    """Chains of one or more trajectories: x, res_offsets, stream_ids, bonds, natives, protocols."""

    def __init__(self, x, offsets, bonds, natives):
        self.x, self.res_offsets = x, np.asarray(offsets, np.int64)
        self.stream_ids = np.arange(len(offsets) - 1, dtype=np.uint32)
        self.bonds = np.asarray(bonds, np.int32).reshape(-1, 2)
        self.natives = np.asarray(natives, np.int32).reshape(-1, 2)
        self.bond_r0 = np.linalg.norm(x[self.bonds[:, 0]] - x[self.bonds[:, 1]], axis=1)
        self.native_r0 = np.linalg.norm(x[self.natives[:, 0]] - x[self.natives[:, 1]], axis=1)
        self.fixed, self.pulls, self.tip = None, [], None


class Pull:
    def __init__(self, traj, residue, kappa, anchor0, v):
        self.traj, self.residue, self.kappa, self.anchor0, self.v = traj, residue, kappa, anchor0, v


class Tip:
    def __init__(self, c0, v):
        self.radius, self.eps, self.sigma, self.c0, self.v = 50.0, 1.0, 1.0, c0, v


def _one_chain(X):
    k = np.arange(len(X) - 1)
    return System(X - X.mean(0), [0, len(X)], np.stack([k, k + 1], 1), _contacts(X))


def _copies(m, rng, shell):
    """m copies of a 250-residue subunit inside an oblate 27 x 27 x 18 A
    ellipsoid, on a shell (short axis outwards) or stacked along x (short axis
    along x); no two copies come closer than 4 A, neighbours share contacts."""
    axes = np.array([27.0, 27.0, 18.0])
    sub = _walk(250, rng, axes)
    spin = rng.uniform(0.0, 2.0 * np.pi, m)
    c, s, o = np.cos(spin), np.sin(spin), np.zeros(m)
    R = np.stack([c, -s, o, s, c, o, o, o, o + 1.0], 1).reshape(m, 3, 3)
    if shell:
        k = np.arange(m) + 0.5
        phi, th = np.arccos(1.0 - 2.0 * k / m), np.pi * (1.0 + 5.0 ** 0.5) * k
        z = np.stack([np.cos(th) * np.sin(phi), np.sin(th) * np.sin(phi), np.cos(phi)], 1)
        t = np.where(np.abs(z[:, :1]) < 0.9, [[1.0, 0.0, 0.0]], [[0.0, 1.0, 0.0]])
        u = np.cross(t, z)
        u /= np.linalg.norm(u, axis=1, keepdims=True)
        R = np.stack([u, np.cross(z, u), z], 2) @ R
        d = np.linalg.norm(z[:, None] - z[None], axis=2) + 10.0 * np.eye(m)
        centre = z * (58.1 / d.min())
        near = np.argwhere(np.triu(d * 58.1 / d.min() < 54.0 + NATIVE))
    else:
        R = np.array([[0.0, 0.0, 1.0], [0.0, 1.0, 0.0], [-1.0, 0.0, 0.0]]) @ R
        x = 40.1 * (np.arange(m) - 0.5 * (m - 1))
        centre = np.stack([x, 0 * x, 0 * x], 1)
        near = np.stack([np.arange(m - 1), np.arange(1, m)], 1)
    y = np.einsum("mij,nj->mni", R, sub) + centre[:, None]
    first = 250 * np.arange(m)[:, None, None]
    k = np.arange(249)
    bonds = (first + np.stack([k, k + 1], 1)).reshape(-1, 2)
    natives = [(first + _contacts(sub)).reshape(-1, 2)]
    g = torch.from_numpy(y).cuda()  # contacts between neighbouring copies
    for a in range(0, len(near), 128):
        p = near[a:a + 128]
        d2 = sum((g[p[:, 0], :, None, ax] - g[p[:, 1], None, :, ax]) ** 2 for ax in range(3))
        h = torch.nonzero(d2 < NATIVE * NATIVE).cpu().numpy()
        natives.append(np.stack([250 * p[h[:, 0], 0] + h[:, 1], 250 * p[h[:, 0], 1] + h[:, 2]], 1))
    return System(y.reshape(-1, 3), [0, 250 * m], bonds, np.concatenate(natives))


def _system(case, rng):
    shape, n = case["shape"], case["n"]
    if shape == "chain":
        s = _one_chain(_walk(n, rng))
    elif shape == "globule":
        r = (3.0 * n * 300.0 / (4.0 * math.pi)) ** (1.0 / 3.0)
        s = _one_chain(_walk(n, rng, np.array([r, r, r])))
    elif shape == "dense":
        s = _one_chain(_dense(n, rng))
    else:
        s = _copies(n, rng, shape == "shell")
    if case.get("pull"):  # one end held, the other on a cantilever
        s.fixed = np.zeros(len(s.x), np.uint8)
        s.fixed[0] = 1
        e = s.x[-1] - s.x[0]
        s.pulls = [Pull(0, len(s.x) - 1, CANTILEVER, s.x[-1].copy(), 5e-6 * e / np.linalg.norm(e))]
    if case.get("tip"):  # a tip above the top, the bottom held
        z = s.x[:, 2]
        s.fixed = (z < z.min() + 10.0).astype(np.uint8)
        s.tip = Tip(np.array([0.0, 0.0, z.max() + 52.0]), np.array([0.0, 0.0, -1e-4]))
    return s


def _ensemble(lengths, rng, same=1):
    """Chains cut at random from a library of self-avoiding walks and turned at
    random; every `same` consecutive trajectories start from one chain."""
    lib = _walks(24, max(int(max(lengths)), 4), rng)
    pairs = [_contacts(X) for X in lib]
    T = len(lengths)
    R = _turn(rng, T)
    xs, bonds, natives, off = [], [], [], [0]
    for t, m in enumerate(lengths):
        if t % same == 0:
            w, a = rng.integers(len(lib)), rng.integers(lib.shape[1] - m + 1)
            p = pairs[w]
            p = p[(p[:, 0] >= a) & (p[:, 1] < a + m)] - a
            X = lib[w, a:a + m] - lib[w, a:a + m].mean(0)
            k = np.arange(m - 1)
        xs.append(X @ R[t].T)
        bonds.append(np.stack([k, k + 1], 1) + off[-1])
        natives.append(p + off[-1])
        off.append(off[-1] + int(m))
    return System(np.concatenate(xs), off, np.concatenate(bonds), np.concatenate(natives))


def _start(s, rng):
    """A thermal displacement of the structure (fixed residues stay)."""
    x = s.x + 0.1 * rng.standard_normal(s.x.shape)
    return x if s.fixed is None else np.where(s.fixed[:, None] != 0, s.x, x)


def _ladder(case):
    return KB * np.geomspace(280.0, 420.0, case["reps"])


def _made(case, seed):
    """(system, parameters, start coordinates) of a case and a seed."""
    rng = np.random.default_rng([seed, 1003])
    if case["kind"] == "ensemble":
        # the lengths belong to the case, the conformations to the seed
        m = np.random.default_rng([case["traj"], case["lmin"], case["lmax"]])
        s = _ensemble(m.integers(case["lmin"], case["lmax"] + 1, case["traj"]), rng)
    elif case["kind"] == "exchange":
        s = _ensemble([case["length"]] * (case["groups"] * case["reps"]), rng, same=case["reps"])
    else:
        s = _system(case, rng)
    return s, Params(seed % 65536), _start(s, rng)


def _ramp_made(case, seed):
    rng = np.random.default_rng([seed, 41])
    x = np.zeros((case["n"], 2), np.float32)
    x[:, 0] = rng.normal(0.0, 0.3, case["n"])
    # pN, nm, ps: K_sp = 40 pN/nm, kB T = 4.14 pN nm, D = 1.5e-11 cm^2/s
    p = {"rf": 1e-8, "xi": 4.14 / 1.5e-9, "k_sp": 40.0, "kBT": 4.14 if case["noise"] else 0.0, "h": 25.0,
         "order": case["order"], "seed": 77 + seed % 65536, "stream": 3}
    return x, p


# ---------------------------------------------------------------------------
# a pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "ramp":
        x, p = _ramp_made(case, seed)
        return {"case": case, "rp": sop.ramp_params(compensated=case["compensated"], **p),
                "x": torch.from_numpy(x).cuda(), "step": 0}
    s, p, x = _made(case, seed)
    batched = case["kind"] in ("ensemble", "exchange")
    ctx = sop.from_system(s, p, schedule="batched" if batched else "plain",
                          energy_every=case.get("energy_every", 0), coordinates=x)
    if case["kind"] == "md":
        ctx.set_list_skin(case["skin"])
        if case["integrator"] != "overdamped":
            ctx.set_integrator(case["integrator"], 5.0)
    if case["kind"] == "exchange":
        ctx.set_tempering(_ladder(case), case["every"])
    return {"case": case, "ctx": ctx, "x0": x}


def run(state):
    case = state["case"]
    if case["kind"] == "ramp":
        mean, var = sop.ramp_run(state["rp"], state["x"], state["step"], case["steps"])
        state["step"] += case["steps"]
        return {"x": state["x"], "mean": mean, "variance": var}
    ctx = state["ctx"]
    if case["kind"] == "score":
        ctx.set_coordinates(state["x0"])
        F, E, _ = ctx.compute_forces()
        return {"forces": F.astype(np.float32), "energies": E.astype(np.float32)}
    ctx.step(case["steps"])
    out = {"moved": (ctx.get_coordinates() - state["x0"]).astype(np.float32)}
    if case["kind"] == "exchange":
        out["rung"], out["accepted"], out["attempted"] = ctx.get_tempering()
    elif case.get("energy_every"):
        out["energies"] = ctx.get_energies()[0].astype(np.float32)
        if case.get("pull"):
            out["force"] = ctx.get_external_force().astype(np.float32)
    if case.get("integrator") == "underdamped":
        out["velocities"] = ctx.get_velocities().astype(np.float32)
    return out


def work(case):
    """Every position, topology entry and result once; each unordered pair's
    term once a step (about 20 operations; 35 to 140 list pairs a residue by
    density), 12 Gaussians' worth of operations a residue and step."""
    if case["kind"] == "ramp":
        return {"bytes": 16 * case["n"], "flops": case["n"] * case["steps"] * (60 if case["noise"] else 10)}
    if case["kind"] == "ensemble":
        n, pairs = case["traj"] * (case["lmin"] + case["lmax"]) / 2, 20
    elif case["kind"] == "exchange":
        n, pairs = case["groups"] * case["reps"] * case["length"], 20
    else:
        n = case["n"] * (250 if case["shape"] in ("shell", "fibre") else 1)
        pairs = {"chain": 18, "globule": 55, "dense": 110, "shell": 45, "fibre": 50}[case["shape"]]
    pairs = min(pairs, n / 2)
    steps = case.get("steps", 1)
    return {"bytes": n * (64 + 12 + 8 * 4 + 24), "flops": n * steps * (20 * (pairs + 4) + 150)}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 over int64 tensors of 32-bit words."""
    m = 0xFFFFFFFF
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # modulo 2^64
        c0, c1, c2, c3 = ((b >> 32) & m) ^ c1 ^ k0, b & m, ((a >> 32) & m) ^ c3 ^ k1, a & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _gauss(local, stream, step, seed):
    step = torch.full_like(local, step & 0xFFFFFFFF)
    w = _philox(local, stream, step, torch.zeros_like(local), seed & 0xFFFFFFFF, seed >> 32)
    u = [((v >> 9).double() + 0.5) * 2.0 ** -23 for v in w]
    r, s = torch.sqrt(-2.0 * torch.log(u[0])), torch.sqrt(-2.0 * torch.log(u[2]))
    t = 2.0 * math.pi
    return torch.stack([r * torch.cos(t * u[1]), r * torch.sin(t * u[1]), s * torch.cos(t * u[3])], 1)


class _Exact:
    """The model in double precision: forces, list, noise and steps."""
    MARGIN = 8.0

    def __init__(self, case, seed):
        self.case = case
        self.s, self.p, x = _made(case, seed)
        d = _dev()
        s = self.s
        self.x = torch.from_numpy(x).to(d)
        self.v = torch.zeros_like(self.x)
        self.bonds, self.natives = (torch.from_numpy(v.astype(np.int64)).to(d) for v in (s.bonds, s.natives))
        self.r0b, self.r0n = (torch.from_numpy(np.float32(v).astype(float)).to(d) for v in (s.bond_r0, s.native_r0))
        off = s.res_offsets
        n = len(x)
        T = len(off) - 1
        traj = np.repeat(np.arange(T), np.diff(off))
        self.traj = torch.from_numpy(traj).to(d)
        self.local = torch.from_numpy(np.arange(n) - off[traj]).to(d)
        self.off, self.T, self.n = off, T, n
        self.free = torch.ones(n, 1, dtype=torch.float64, device=d)
        if s.fixed is not None:
            self.free[torch.from_numpy(s.fixed != 0).to(d)] = 0.0
        pr = torch.cat([self.bonds, self.natives])
        self.known = torch.sort(pr.min(1).values * n + pr.max(1).values).values
        self.cand_at = None

    def candidates(self):
        """Pairs of one trajectory within the list cutoff and a margin, neither bonded nor native."""
        xf, out, rc = self.x.float(), [], self.p.r_list + self.MARGIN
        many = self.T > 1
        block = 4096 if not many else 1 << 62
        if many:  # all pairs of each trajectory
            for t in range(self.T):
                a, m = int(self.off[t]), int(self.off[t + 1] - self.off[t])
                out.append(torch.triu_indices(m, m, 1, device=xf.device).T + a)
            ij = torch.cat(out)
            out = [ij[((xf[ij[:, 0]] - xf[ij[:, 1]]) ** 2).sum(1) < rc * rc]]
        else:
            order = torch.argsort(xf[:, 0])
            sx = xf[order, 0].contiguous()
            for a in range(0, self.n, block):
                i = order[a:a + block]
                hi = int(torch.searchsorted(sx, sx[min(a + block, self.n) - 1] + rc))
                j = order[a:hi]
                d2 = sum((xf[i, k, None] - xf[None, j, k]) ** 2 for k in range(3))
                q = torch.nonzero(d2 < rc * rc)
                q = q[q[:, 1] > q[:, 0]]
                pr = torch.stack([i[q[:, 0]], j[q[:, 1]]], 1)
                out.append(torch.stack([pr.min(1).values, pr.max(1).values], 1))
        ij = torch.cat(out)
        if len(self.known):
            key = ij[:, 0] * self.n + ij[:, 1]
            at = torch.searchsorted(self.known, key).clamp(max=len(self.known) - 1)
            ij = ij[self.known[at] != key]
        self.cand, self.cand_at = ij, self.x.clone()

    def rebuild(self):
        if self.cand_at is None or float(((self.x - self.cand_at) ** 2).sum(1).max()) > (0.4 * self.MARGIN) ** 2:
            self.candidates()
        xf = self.x.float()  # the predicate is in single precision
        d = xf[self.cand[:, 0]] - xf[self.cand[:, 1]]
        d = d * d
        self.list = self.cand[(d[:, 0] + d[:, 1]) + d[:, 2] < np.float32(self.p.r_list ** 2)]

    def forces(self, step, energies=False):
        p, F, E = self.p, torch.zeros_like(self.x), None
        if energies:
            E = torch.zeros(self.T, 5, dtype=torch.float64, device=self.x.device)

        def add(ij, coef, d, e, k):
            f = coef[:, None] * d
            F.index_add_(0, ij[:, 0], f)
            F.index_add_(0, ij[:, 1], -f)
            if E is not None:
                t = self.traj[ij[:, 0]]
                E[:, k].index_add_(0, t, e)
                E[:, 4].index_add_(0, t, coef * (d * d).sum(1))

        d = self.x[self.bonds[:, 0]] - self.x[self.bonds[:, 1]]
        r = d.norm(dim=1)
        dl = r - self.r0b
        q = 1.0 - (dl / p.R0) ** 2
        add(self.bonds, -p.k_fene * dl / (q * r), d, -0.5 * p.k_fene * p.R0 ** 2 * torch.log(q), 0)
        d = self.x[self.natives[:, 0]] - self.x[self.natives[:, 1]]
        r2 = (d * d).sum(1)
        q = (self.r0n * self.r0n / r2) ** 3
        add(self.natives, 12.0 * p.eps_h * (q * q - q) / r2, d, p.eps_h * (q * q - 2.0 * q), 1)
        for a in range(0, len(self.list), 1 << 23):
            ij = self.list[a:a + (1 << 23)]
            d = self.x[ij[:, 0]] - self.x[ij[:, 1]]
            r2 = (d * d).sum(1)
            q = (p.sigma * p.sigma / r2) ** 3
            add(ij, 6.0 * p.eps_l * q / r2, d, p.eps_l * q, 2)
        report = torch.zeros(self.T, dtype=torch.float64, device=self.x.device)
        t = step * p.h
        like = lambda v: torch.tensor(np.asarray(v, float), device=self.x.device)  # noqa: E731
        for w in self.s.pulls:
            d = like(w.anchor0 + w.v * t) - self.x[w.residue]
            F[w.residue] += w.kappa * d
            report[w.traj] += w.kappa * (d @ like(w.v / np.linalg.norm(w.v)))
            if E is not None:
                E[w.traj, 3] += 0.5 * w.kappa * (d * d).sum()
        tip = self.s.tip
        if tip is not None:
            d = self.x - like(tip.c0 + tip.v * t)
            r = d.norm(dim=1)
            q = (tip.sigma / (r - tip.radius)) ** 6
            F += (6.0 * tip.eps * q / ((r - tip.radius) * r))[:, None] * d
            if E is not None:
                E[:, 3].index_add_(0, self.traj, tip.eps * q)
        return F, E, report

    def steps(self, n, kbt=None):
        """n steps from step 0; (energies, reports) of the last record; kbt: per-trajectory
        temperatures by step (a function of self and the step)."""
        p, c, rec = self.p, self.case, None
        under = c.get("integrator") == "underdamped"
        mass, every = 5.0, c.get("energy_every", 0)
        c1 = math.exp(-p.zeta / mass * p.h)
        c2 = math.sqrt((1.0 - c1 * c1) * p.kBT / mass)
        stream = self.traj
        for k in range(n):
            if k % p.list_every == 0:
                self.rebuild()
            want = bool(every) and k % every == 0
            F, E, rep = self.forces(k, want)
            if want:
                rec = (E, rep)
            g = _gauss(self.local, stream, k, p.seed)
            if under:
                w0 = self.v + (0.5 if k == 0 else 1.0) * p.h / mass * F
                w1 = c1 * w0 + c2 * g
                dx, self.v = 0.5 * p.h * (w0 + w1), w1 * self.free
            else:
                T = p.kBT if kbt is None else kbt(self, k)[self.traj][:, None]
                amp = math.sqrt(2.0 * p.h / p.zeta) * (math.sqrt(T) if kbt is None else torch.sqrt(T))
                dx = F * (p.h / p.zeta) + g * amp
            self.x = self.x + dx * self.free
        if under:  # the last half kick
            if n % p.list_every == 0:
                self.rebuild()
            self.v = (self.v + 0.5 * p.h / mass * self.forces(n)[0]) * self.free
        return rec


def _exact_exchange(case, seed):
    e = _Exact(case, seed)
    R, G = case["reps"], case["groups"]
    ladder = _ladder(case)
    rung = np.tile(np.arange(R), G)
    acc, att = np.zeros(R - 1, np.int64), np.zeros(R - 1, np.int64)

    def kbt(self, k):
        if k % case["every"] == 0:
            E = self.forces(k, True)[1][:, :4].sum(1).cpu().numpy()
            r = k // case["every"]
            for lo in range(r % 2, R - 1, 2):
                word = _philox(torch.arange(G), torch.full((G,), lo), torch.full((G,), r),
                               torch.zeros(G, dtype=torch.int64), (self.p.seed & 0xFFFFFFFF) ^ 0x52455843,
                               self.p.seed >> 32)[0].numpy()
                for g in range(G):
                    a, b = (g * R + int(np.nonzero(rung[g * R:(g + 1) * R] == q)[0][0]) for q in (lo, lo + 1))
                    d = (1.0 / ladder[lo] - 1.0 / ladder[lo + 1]) * (E[a] - E[b])
                    att[lo] += 1
                    if d >= 0.0 or ((int(word[g]) >> 9) + 0.5) * 2.0 ** -23 < math.exp(d):
                        acc[lo] += 1
                        rung[a], rung[b] = lo + 1, lo
        return torch.from_numpy(ladder[rung]).to(self.x.device)

    x0 = e.x.clone()
    e.steps(case["steps"], kbt)
    return {"moved": (e.x - x0).cpu().numpy(), "rung": rung.astype(np.int32), "accepted": acc, "attempted": att}


def _exact_ramp(case, seed):
    x, p = _ramp_made(case, seed)
    X = torch.from_numpy(x[:, 0].astype(float)).to(_dev())
    i = torch.arange(case["n"], device=X.device)
    stream = torch.full_like(i, p["stream"])
    c = p["h"] / p["xi"] * (1.0 - 0.5 * p["h"] * p["k_sp"] / p["xi"] if p["order"] == 2 else 1.0)
    amp = math.sqrt(2.0 * p["kBT"] * p["h"] / p["xi"])
    for k in range(case["steps"]):
        dx = c * (p["rf"] * p["h"] * k - p["k_sp"] * X)
        if case["noise"]:
            dx = dx + amp * _gauss(i, stream, k, p["seed"])[:, 0]
        X = X + dx
    # the split of X into its two single-precision parts has no one value
    return {"x": None, "mean": float(X.mean()), "variance": float(X.var(unbiased=False))}


def exact(case, seed):
    if case["kind"] == "ramp":
        return _exact_ramp(case, seed)
    if case["kind"] == "exchange":
        return _exact_exchange(case, seed)
    e = _Exact(case, seed)
    if case["kind"] == "score":
        e.rebuild()
        F, E, _ = e.forces(0, True)
        return {"forces": F.cpu().numpy(), "energies": E.cpu().numpy()}
    x0 = e.x.clone()
    rec = e.steps(case["steps"])
    out = {"moved": (e.x - x0).cpu().numpy()}
    if case.get("energy_every"):
        out["energies"] = rec[0].cpu().numpy()
        if case.get("pull"):
            out["force"] = rec[1].cpu().numpy()
    if case.get("integrator") == "underdamped":
        out["velocities"] = e.v.cpu().numpy()
    return out
