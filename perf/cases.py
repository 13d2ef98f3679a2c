"""What users of this framework have it compute, as cases that can be timed and checked.

Four kinds of call, each through the package's entry points:

* ``step``    new angles for a set of chains, then some KCM iterations
              (kcm_set_theta_batch, kcm_step), the angles and records read back;
* ``fold``    the same with kcm_fold, which stops each chain at its tolerance;
* ``scan``    energies over a grid of dihedrals (landscape.EnergyScanner);
* ``search``  Monte Carlo minimization (kcm_mc_minimize).

Every pass begins from the same angles, so a pass can be repeated on one state
and gives the same results each time.  ``exact`` follows the method of the
paper in 64 bits with numpy and torch alone.
"""
import math

import numpy as np
import torch

import synth
from paper_1712_05012_amd import kcm, landscape, polyala

APR = 10          # atoms per residue
N_ORBITS = 14     # samples of the offset spheres: 14 orbits, 250 directions
COULOMB = 332.0636


def listed():
    return [
        # the helix experiment between two trace points, a hundred iterations of two short chains: launches and latency
        _case("helix_vacuum_fp64", "step", chains=2, lo=15, hi=15, start="coiled", ala=True, terms="vacuum",
              precision="fp64", iters=100),
        # one such chain in water and in mixed precision, ten iterations: the smallest call
        _case("helix_water_mixed", "step", chains=1, lo=15, hi=15, start="coiled", ala=True, iters=10),
        # a Ramachandran map of a residue pair at 5 degree steps: thousands of tiny chains, one evaluation each
        _case("map_pair_mixed", "scan", lo=2, hi=2, start="flat", points=5184, batch=1024),
        # a hinge scan of a 40-residue chain, in FP64
        _case("hinge_40_fp64", "scan", lo=40, hi=40, start="coiled", points=64, batch=64, precision="fp64"),
        # folding statistics: many short chains from random starts, in vacuum
        _case("fold_vacuum_fp64", "fold", chains=256, lo=10, hi=20, start="ramachandran", ala=True, terms="vacuum",
              precision="fp64", iters=200, check_every=50),
        # and in water
        _case("fold_water_mixed", "fold", chains=500, lo=10, hi=20, start="ramachandran", ala=True, iters=100,
              check_every=50),
        # Monte Carlo minimization of short chains
        _case("search_vacuum_fp64", "search", chains=128, lo=10, hi=20, start="ramachandran", ala=True,
              terms="vacuum", precision="fp64", trials=4, iters=20),
        # one chain of 1,000 residues from a compact globule: the single-chain fold
        _case("globule_1000_mixed", "step", chains=1, lo=1000, hi=1000, start="globule", iters=8),
        # one evaluation and step of the same chain in FP64, as an outer optimiser asks for it
        _case("globule_1000_fp64", "step", chains=1, lo=1000, hi=1000, start="globule", precision="fp64", iters=1,
              whole=True),
        # one chain of 10,000 residues (100,000 atoms)
        _case("globule_10000_mixed", "step", chains=1, lo=10000, hi=10000, start="globule", iters=4),
        # what a serving tick holds: chains of very different lengths, here with side-chain joints
        _case("ragged_chi_mixed", "step", chains=61, lo=30, hi=2000, start="coil", side_chains=True, iters=2),
        # the ragged batch of the benchmark: 256 random coils of 50 to 600 residues, the largest call
        _case("batch_256_mixed", "step", chains=256, lo=50, hi=600, start="coil", cell_size=3.6, iters=8),
    ]


def _case(name, kind, **over):
    """chains of lo..hi residues; start: how the angles are drawn (_start); iters: iterations (per trial in a
    search); points, batch: grid points of a scan and chains of its pool; whole: positions, forces and torques are
    read back too."""
    case = {"name": name, "kind": kind, "chains": 1, "lo": 15, "hi": 15, "start": "coil", "ala": False,
            "terms": "all", "precision": "mixed", "side_chains": False, "cell_size": 0.0, "iters": 1,
            "check_every": 10, "points": 0, "batch": 0, "trials": 0, "whole": False}
    case.update(over)
    return case


def draw(rng):
    """One more case of the same kinds: chain counts, lengths, grids and iterations over the listed ones' ranges."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "fold", "scan", "search"])
    over = {"precision": rng.choice(["mixed", "mixed", "fp64"])}
    if kind == "step" and rng.random() < 0.5:
        m = logint(2, 10000)
        over.update(chains=1, lo=m, hi=m, start="coil" if m <= 600 and rng.random() < 0.5 else "globule",
                    iters=rng.randint(1, 4), whole=rng.random() < 0.25, side_chains=rng.random() < 0.25)
    elif kind == "step":
        n = logint(2, 256)
        hi = logint(20, min(2000, 150000 // n))
        lo = max(1, logint(max(1, hi // 20), hi))
        over.update(chains=n, lo=lo, hi=hi, iters=rng.randint(1, 4), side_chains=rng.random() < 0.25,
                    cell_size=rng.choice([0.0, 0.0, 3.6, 4.4]))
    elif kind == "fold":
        hi = rng.randint(8, 24)
        over.update(chains=logint(1, 500), lo=max(2, hi // 2), hi=hi, start="ramachandran", ala=True,
                    terms=rng.choice(["all", "vacuum"]), iters=logint(10, 100), check_every=rng.randint(5, 50))
    elif kind == "scan":
        m = logint(1, 60)
        pts = logint(16, max(17, min(5184, 40000 // m)))
        over.update(lo=m, hi=m, start="coiled" if m > 2 else "flat", points=pts, batch=logint(16, min(1024, pts)))
    else:
        over.update(chains=logint(1, 128), lo=rng.randint(3, 10), hi=rng.randint(11, 24), start="ramachandran",
                    ala=True, terms=rng.choice(["all", "vacuum"]), trials=rng.randint(1, 4), iters=rng.randint(2, 12))
    case = _case("", kind, **over)
    del case["name"]
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _types(case):
    return synth.alanine_like_types() if case["ala"] else synth.residue_types()


def _lengths(case):
    """Residues of each chain: the same for every seed, so that the seeds of a case have outputs of one shape."""
    n, lo, hi = case["chains"], case["lo"], case["hi"]
    rng = np.random.default_rng([n, lo, hi])
    if hi > 600:
        # served jobs: lognormal lengths, median 200
        return np.clip(np.rint(np.exp(rng.normal(math.log(200.0), 0.6, n))), lo, hi).astype(int)
    return rng.integers(lo, hi + 1, n)


def _start(case, m, rng):
    """Angles of one chain: random coil, the stored compact globules (their
    first m residues), a slightly pre-coiled chain, the statistics' starts
    within 90 degrees, or the zero position."""
    kind = case["start"]
    if kind == "coil":
        th = rng.uniform(-math.pi, math.pi, 2 * m)
    elif kind == "globule":
        th = synth.load_globule(1000 if m <= 1000 else 10000)[:2 * m]
    elif kind == "coiled":
        th = math.radians(rng.choice([10.0, -10.0])) + rng.uniform(-0.02, 0.02, 2 * m)
    elif kind == "ramachandran":
        th = rng.uniform(-0.5 * math.pi, 0.5 * math.pi, 2 * m)
    else:
        th = np.full(2 * m, math.pi)
    if case["side_chains"]:
        th = np.concatenate([th, rng.uniform(-math.pi, math.pi, m)])
    return th


def _inputs(case, seed):
    """Sequences, start angles and, by kind, the scan's grid or the search's moves: host arrays, from the seed alone."""
    rng = np.random.default_rng(seed)
    T = _types(case)
    out = {"types": T}
    if case["kind"] == "scan":
        m = case["lo"]
        out["seq"] = [rng.integers(0, len(T.hydro), m).astype(np.int32)]
        base = _start(case, m, rng)
        # two joints of one residue turn through a square grid, in grid order
        j = 2 * (m // 2)
        side = math.isqrt(case["points"] - 1) + 1
        vals = np.linspace(-math.pi, math.pi, side, endpoint=False) + rng.uniform(0.0, 2.0 * math.pi / side)
        grid = landscape.grid_thetas(base, [j, j + 1], [vals, vals])
        out["thetas"] = np.ascontiguousarray(grid[:case["points"]])
        return out
    lens = _lengths(case)
    out["seq"] = [rng.integers(0, len(T.hydro), int(m)).astype(np.int32) for m in lens]
    out["thetas"] = [_start(case, int(m), rng) for m in lens]
    if case["kind"] == "search":
        moves = [synth.mc_moves(case["trials"], th.size, int(rng.integers(1 << 30))) for th in out["thetas"]]
        out["delta"] = [d for d, _ in moves]
        out["u"] = np.stack([u for _, u in moves])
    return out


def _params(case):
    prec = kcm.KCM_MIXED if case["precision"] == "mixed" else kcm.KCM_FP64
    if case["ala"]:
        p = polyala.experiment_params(case["terms"] == "all", prec)
    else:
        p = kcm.kcm_default_params(precision=prec)
    p.cell_size = case["cell_size"]
    return p


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    p = _params(case)
    if case["kind"] == "scan":
        state["scanner"] = landscape.EnergyScanner(state["seq"][0], state["types"], p, batch=case["batch"])
    else:
        state["chains"] = [kcm.Chain(s, state["types"], p, theta0=th, side_chains=case["side_chains"])
                           for s, th in zip(state["seq"], state["thetas"])]
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "scan":
        return {"energies": state["scanner"].energies(state["thetas"])}
    chains = state["chains"]
    held = kcm.kcm_set_theta_batch(chains, state["thetas"])
    out = {}
    if kind == "search":
        _, res = kcm.kcm_mc_minimize(chains, state["delta"], state["u"], case["iters"], 1.0, check=False)
        out["energies"] = np.array([[r.e_start, r.e_accepted, r.e_best] for r in res])
        out["accepted"] = np.array([r.accepted for r in res])
        out["best"] = np.concatenate([c.mc_best_theta() for c in chains])
    else:
        if kind == "fold":
            _, res = kcm.kcm_fold(chains, 1e-4, case["iters"], case["check_every"], check=False)
            out["iterations"] = np.array([r.iterations for r in res])
            _, reps = kcm.kcm_step(chains, 0, report="array", check=False)
        else:
            _, reps = kcm.kcm_step(chains, case["iters"], report="array", check=False)
        out["energies"] = np.stack([reps["e_elec"], reps["e_vdw"], reps["e_cav"]], axis=1)
        out["max_tau"] = np.array(reps["max_tau"])
        out["max_dtheta"] = np.array(reps["max_dtheta"])
        out["status"] = np.array(reps["status"])
    if case["whole"]:
        states = [c.state() for c in chains]
        for k in ("theta", "xyz", "force", "tau", "dtheta"):
            out[k] = np.concatenate([st[k] for st in states])
    else:
        out["theta"] = np.concatenate([c.theta() for c in chains])
    del held
    return out


def work(case):
    """Per evaluation of a conformation: 40 flops per unordered pair within the
    cutoff, 9 per test of a sample against a solvation neighbour and 9 per
    exposed sample and neighbour.  Pairs and neighbours per atom are estimates
    from the shape of the start; the bytes are the angles, axes, template
    positions and parameters read and the angles written, once per pass."""
    m = 0.5 * (case["lo"] + case["hi"]) if case["hi"] <= 600 or case["lo"] == case["hi"] else 236.0
    if case["kind"] == "scan":
        evals, sets = case["points"], 1
    else:
        evals = case["chains"] * (1 + case["trials"] * (case["iters"] + 1) if case["kind"] == "search" else case["iters"])
        sets = case["chains"]
    atoms = APR * m
    dense = case["start"] in ("globule", "coil")
    pairs = min(0.5 * (atoms - 1), 80.0 if dense else 60.0)       # unordered pairs within 10 A, per atom
    nbr = min(atoms - 1, 62.0 if dense else 45.0)                  # solvation neighbours of an atom
    flops = 40.0 * pairs
    if case["terms"] == "all":
        flops += 9.0 * 250 * nbr + 9.0 * 25.0 * nbr
    joints = (3 if case["side_chains"] else 2) * m
    conf = case["points"] if case["kind"] == "scan" else sets
    return {"bytes": sets * (64.0 * 2 * m + 72.0 * atoms) + conf * 16.0 * joints, "flops": evals * atoms * flops}


# ---------------------------------------------------------------------------
# the same in 64 bits, without the framework
# ---------------------------------------------------------------------------
def exact(case, seed):
    evals = 1 + case["trials"] * (case["iters"] + 1) if case["kind"] == "search" else max(1, case["iters"])
    # The first steps out of the contacts of random and compact starts multiply
    # every rounding by orders of magnitude: past these many evaluations two
    # programs have no value in common.
    if evals > {"coil": 1, "globule": 1, "ramachandran": 4 if case["precision"] == "mixed" else 100}.get(case["start"], 1000):
        return None
    inp = _inputs(case, seed)
    scan = case["kind"] == "scan"
    m_all = np.array([len(s) for s in inp["seq"]] * (len(inp["thetas"]) if scan else 1))
    if float(np.sum((APR * m_all) ** 1.5)) * evals > 1.5e8:
        return None
    seqs = inp["seq"] * len(inp["thetas"]) if scan else inp["seq"]
    # conformations evaluated together in groups of about equal length
    order = np.argsort(m_all, kind="stable")
    groups, at = [], 0
    while at < len(order):
        take = max(1, int(2e6 // (APR * m_all[order[min(at + 999, len(order) - 1)]]) ** 2 * 5))
        groups.append(order[at:at + take])
        at += take
    parts = {}
    for g in groups:
        ens = _Chains(case, inp["types"], [seqs[i] for i in g])
        th0 = [np.asarray(inp["thetas"][i]) for i in g]
        if scan:
            got = {"energies": ens.evaluate(ens.pad(th0))[0]}
        elif case["kind"] == "search":
            got = ens.search(th0, [inp["delta"][i] for i in g], inp["u"][g])
        else:
            got = ens.descend(th0, case["iters"], 1e-4 if case["kind"] == "fold" else 0.0)
        for k, i in enumerate(g):
            for name, v in got.items():
                parts.setdefault(name, {})[i] = v[k]
    out = {}
    for name, by in parts.items():
        rows = [by[i] for i in range(len(m_all))]
        out[name] = np.concatenate(rows) if name not in ("energies", "max_tau", "max_dtheta") else np.array(rows)
    return out


def _wrap(t):
    t = t - 2.0 * math.pi * np.floor((t + math.pi) / (2.0 * math.pi))
    return np.where(t <= -math.pi, t + 2.0 * math.pi, t)


def _directions():
    q = []
    for o in range(N_ORBITS):
        polar = math.pi * (o + 0.5) / N_ORBITS
        cnt = max(1, int(math.floor(2.0 * N_ORBITS * math.sin(polar) + 0.5)))
        for p in range(cnt):
            az = 2.0 * math.pi * (p + 0.5 * (o & 1)) / cnt
            q.append((math.sin(polar) * math.cos(az), math.sin(polar) * math.sin(az), math.cos(polar)))
    return np.array(q)


def _nerf(a, b, c, length, ang, tor):
    """Atom bonded to c at length, with the angle b-c-d and the torsion a-b-c-d (degrees)."""
    e1 = (c - b) / np.linalg.norm(c - b)
    n = np.cross(b - a, e1)
    n = n / np.linalg.norm(n)
    t, p = math.radians(ang), math.radians(tor)
    return c - e1 * (length * math.cos(t)) + (np.cross(n, e1) * math.cos(p) + n * math.sin(p)) * (length * math.sin(t))


def _template(m):
    """Zero position: phi = psi = omega = 180 degrees; slots N, H, CA, HA, CB, HB1-3, C, O."""
    at = np.zeros((m, APR, 3))
    t = math.radians(111.2)
    for i in range(m):
        if i == 0:
            N, CA = np.zeros(3), np.array([1.458, 0.0, 0.0])
            Cc = np.array([1.458 - 1.525 * math.cos(t), 1.525 * math.sin(t), 0.0])
        else:
            N = _nerf(N0, CA0, C0, 1.329, 116.2, 180.0)
            CA = _nerf(CA0, C0, N, 1.458, 121.7, 180.0)
            Cc = _nerf(C0, N, CA, 1.525, 111.2, 180.0)
        CB = _nerf(Cc, N, CA, 1.53, 109.5, -120.0)
        at[i] = [N, _nerf(Cc, CA, N, 1.01, 0.5 * (360.0 - 121.7), 0.0), CA, _nerf(Cc, N, CA, 1.09, 109.5, 120.0), CB,
                 _nerf(N, CA, CB, 1.09, 109.5, 60.0), _nerf(N, CA, CB, 1.09, 109.5, 180.0),
                 _nerf(N, CA, CB, 1.09, 109.5, -60.0), Cc, _nerf(N, CA, Cc, 1.231, 120.8, 0.0)]
        N0, CA0, C0 = N, CA, Cc
    return at.reshape(-1, 3)


def _bond_paths():
    """Bonds between the atoms of a residue window i-1, i, i+1: paths[10 (dres + 1) + slot_j][slot_i], 0 beyond 3."""
    near = [[] for _ in range(3 * APR)]
    for r in range(3):
        bonds = [(0, 1), (0, 2), (2, 3), (2, 4), (2, 8), (4, 5), (4, 6), (4, 7), (8, 9)] + ([(8, APR)] if r < 2 else [])
        for a, b in bonds:
            near[APR * r + a].append(APR * r + b)
            near[APR * r + b].append(APR * r + a)
    paths = np.zeros((3 * APR, APR), dtype=np.int64)
    for s in range(APR):
        seen, rim = {APR + s}, [APR + s]
        for d in (1, 2, 3):
            rim = sorted({y for x in rim for y in near[x]} - seen)
            seen |= set(rim)
            paths[rim, s] = d
    return paths


class _Chains:
    """Chains of about equal length, padded to the longest one, evaluated together in 64 bits."""

    def __init__(self, case, T, seqs):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.case, self.chi = case, case["side_chains"]
        self.m = np.array([len(s) for s in seqs])
        self.M, self.B = int(self.m.max()), len(seqs)
        self.n = APR * self.M
        self.r0 = _template(self.M)
        sig, eps, q, hyd = (np.zeros((self.B, self.M, APR)) for _ in range(4))
        for b, s in enumerate(seqs):
            sig[b, :len(s)], eps[b, :len(s)], q[b, :len(s)] = T.sigma[s], T.eps[s], T.q[s]
            hyd[b, :len(s)] = np.asarray(T.hydro)[s][:, None]
        flat = lambda v: torch.from_numpy(v.reshape(self.B, self.n)).to(self.dev)  # noqa: E731
        self.R, self.q, self.eps = flat(0.5 * 2.0 ** (1.0 / 6.0) * sig), flat(q), flat(eps)
        self.roff = self.R + 1.4
        self.real = torch.arange(self.n, device=self.dev)[None] < torch.from_numpy(APR * self.m).to(self.dev)[:, None]
        self.gamma = 0.025 * flat(hyd)
        self.dirs = torch.from_numpy(_directions()).to(self.dev)
        self.paths = torch.from_numpy(_bond_paths()).to(self.dev)
        self.max_step = 1e-2 if case["ala"] else 1e-3

    def pad(self, thetas):
        """[B, 2M (+ M)] angles, the padding at the zero position."""
        out = np.full((self.B, 2 * self.M), math.pi)
        chi = np.full((self.B, self.M), math.pi / 3.0)
        for b, t in enumerate(thetas):
            out[b, :2 * self.m[b]] = t[:2 * self.m[b]]
            if self.chi:
                chi[b, :self.m[b]] = t[2 * self.m[b]:]
        return np.concatenate([out, chi], axis=1) if self.chi else out

    def unpad(self, v):
        J = 2 * self.M
        return [np.concatenate([v[b, :2 * k], v[b, J:J + k]]) if self.chi else v[b, :2 * k] for b, k in enumerate(self.m)]

    def place(self, th):
        """Positions [B, n, 3], joint axes and points [B, J, 3] by the product of joint rotations."""
        B, J = self.B, 2 * self.M
        r0 = np.broadcast_to(self.r0, (B, self.n, 3)).copy()
        if self.chi:
            for i in range(self.M):
                ca, cb = self.r0[APR * i + 2], self.r0[APR * i + 4]
                u = (cb - ca) / np.linalg.norm(cb - ca)
                a = th[:, J + i, None, None] - math.pi / 3.0
                v = self.r0[APR * i + 5:APR * i + 8] - cb
                r0[:, APR * i + 5:APR * i + 8] = (cb + v * np.cos(a) + np.cross(u, v) * np.sin(a) +
                                                  u * (v @ u)[:, None] * (1.0 - np.cos(a)))
        rot, tr = np.broadcast_to(np.eye(3), (B, 3, 3)).copy(), np.zeros((B, 3))
        r = np.zeros((B, self.n, 3))
        U, P = np.zeros((B, J, 3)), np.zeros((B, J, 3))
        r[:, :2] = r0[:, :2]
        for j in range(J):
            i, psi = divmod(j, 2)
            a, b = self.r0[APR * i + (2 if psi else 0)], self.r0[APR * i + (8 if psi else 2)]
            u = (b - a) / np.linalg.norm(b - a)
            K = np.array([[0, -u[2], u[1]], [u[2], 0, -u[0]], [-u[1], u[0], 0]])
            ang = th[:, j] - math.pi
            T = np.eye(3) + np.sin(ang)[:, None, None] * K + (1.0 - np.cos(ang))[:, None, None] * (K @ K)
            tr = np.einsum("bij,bj->bi", rot, a - T @ a) + tr
            rot = rot @ T
            U[:, j], P[:, j] = rot @ u, rot @ a + tr
            at = slice(APR * i + 8, min(self.n, APR * i + 12)) if psi else slice(APR * i + 2, APR * i + 8)
            r[:, at] = np.einsum("bij,bnj->bni", rot, r0[:, at]) + tr[:, None]
        return r, U, P

    def evaluate(self, th):
        """Energies [B, 3] (elec, vdw, cav), forces and kinematics at the angles."""
        r, U, P = self.place(th)
        x = torch.from_numpy(r).to(self.dev)
        F = torch.zeros_like(x)
        E = torch.zeros(self.B, 3, dtype=torch.float64, device=self.dev)
        res = torch.arange(self.n, device=self.dev) // APR
        slot = torch.arange(self.n, device=self.dev) % APR
        rows = max(1, int(2e7 // (self.B * self.n)))
        for a0 in range(0, self.n, rows):
            i = torch.arange(a0, min(self.n, a0 + rows), device=self.dev)
            d = x[:, None, :, :] - x[:, i, None, :]                     # r_j - r_i
            d2 = (d * d).sum(-1)
            pair = self.real[:, i, None] & self.real[:, None, :] & (i[:, None] != torch.arange(self.n, device=self.dev))
            dres = res[None, :] - res[i][:, None]
            idx = ((dres + 1) * APR + slot[None, :]).clamp(0, 3 * APR - 1)
            path = torch.where(dres.abs() <= 1, self.paths[idx, slot[i][:, None]], torch.zeros_like(idx))
            near = torch.where(path == 3, 1.0, torch.where(path > 0, 0.0, 1.0).double())
            we, wv = near * torch.where(path == 3, 1.0 / 1.2, 1.0), near * torch.where(path == 3, 0.5, 1.0)
            ok = pair & (d2 <= 100.0)
            inv = torch.where(ok, 1.0 / torch.where(ok, d2, torch.ones_like(d2)), torch.zeros_like(d2))
            el = we * (COULOMB / 4.0) * self.q[:, i, None] * self.q[:, None, :] * inv
            s6 = ((self.R[:, i, None] + self.R[:, None, :]) ** 2 * inv) ** 3
            ee = wv * torch.sqrt(self.eps[:, i, None] * self.eps[:, None, :])
            F[:, i] -= ((2.0 * el + 12.0 * ee * (s6 * s6 - s6)) * inv).unsqueeze(-1).mul(d).sum(2)
            E[:, 0] += 0.5 * el.sum((1, 2))
            E[:, 1] += 0.5 * (ee * (s6 * s6 - 2.0 * s6)).sum((1, 2))
            if self.case["terms"] == "all":
                lim = self.roff[:, i, None] + self.roff[:, None, :] + 0.05
                self._solvation(x, i, pair & (d2 <= lim * lim), F, E)
        return E.cpu().numpy(), F.cpu().numpy(), r, U, P

    def _solvation(self, x, i, nbr, F, E):
        """Exposed samples of the atoms i and the events of eq F_cav_patch, neighbours nbr [B, len(i), n]."""
        N, dr = self.dirs.shape[0], 0.05
        b, k, j = nbr.nonzero(as_tuple=True)
        count = nbr.sum(2).reshape(-1)
        first = torch.cumsum(count, 0) - count
        row = b * len(i) + k
        pos = torch.arange(len(row), device=self.dev) - first[row]
        width = max(1, int(count.max()))
        lists = torch.full((self.B * len(i), width), -1, dtype=torch.int64, device=self.dev)
        lists[row, pos] = j
        own = self.real[:, i].reshape(-1).nonzero()[:, 0]
        for s in range(0, len(own), max(1, int(4e7 // (N * width)))):
            rw = own[s:s + max(1, int(4e7 // (N * width)))]
            bb, ii, jj = rw // len(i), i[rw % len(i)], lists[rw]
            have, jj = jj >= 0, jj.clamp(min=0)
            pts = x[bb, ii][:, None] + self.roff[bb, ii][:, None, None] * self.dirs
            R2 = torch.where(have, self.roff[bb[:, None], jj] ** 2, torch.full_like(jj, -1.0, dtype=torch.float64))
            c = x[bb[:, None], jj]
            diff = pts[:, None] - c[:, :, None]                          # [rows, width, N, 3]
            sq = (diff * diff).sum(-1)
            cov = sq <= R2[..., None]
            C = cov.sum(1)
            crit, free = (C == 1)[:, None] & cov, (C == 0)[:, None]
            G = 4.0 * math.pi * self.gamma[bb, ii] * self.roff[bb, ii] ** 2
            E[:, 2].index_add_(0, bb, G * (C == 0).sum(1) / N)
            for ax in range(3):
                moved = sq - 2.0 * dr * diff[..., ax] + dr * dr <= R2[..., None]
                ev = ((crit & ~moved).sum(2) - (free & moved).sum(2)).double() * (G / (N * dr))[:, None]
                F[..., ax].index_put_((bb, ii), ev.sum(1), accumulate=True)
                F[..., ax].index_put_((bb[:, None].expand_as(jj), jj), torch.where(have, -ev, torch.zeros_like(ev)),
                                      accumulate=True)

    def step(self, th):
        """One iteration: (new angles, energies, max |tau|, max |dtheta|, (positions, forces, torques, step))."""
        E, F, r, U, P = self.evaluate(th)
        J = 2 * self.M
        T = np.cross(r, F)
        sufF, sufT = (np.cumsum(v[:, ::-1], axis=1)[:, ::-1] for v in (F, T))
        a = [APR * (j >> 1) + (8 if j & 1 else 2) for j in range(J)]
        tau = np.einsum("bjk,bjk->bj", U, sufT[:, a] - np.cross(P, sufF[:, a]))
        live = np.repeat(np.arange(self.M)[None] < self.m[:, None], 2, axis=1)
        if self.chi:
            A = r.reshape(self.B, self.M, APR, 3)
            Fr = F.reshape(self.B, self.M, APR, 3)
            u = A[:, :, 4] - A[:, :, 2]
            u = u / np.linalg.norm(u, axis=-1, keepdims=True)
            t = np.cross(A[:, :, 5:8] - A[:, :, 2:3], Fr[:, :, 5:8]).sum(2)
            tau = np.concatenate([tau, (u * t).sum(-1)], axis=1)
            live = np.concatenate([live, np.arange(self.M)[None] < self.m[:, None]], axis=1)
        tau = np.where(live, tau, 0.0)
        top = np.abs(tau).max(axis=1)
        scale = np.where(1e-3 * top > self.max_step, self.max_step / np.where(top > 0, top, 1.0), 1e-3)
        move = scale[:, None] * tau
        new = th + move
        new = np.where(new > math.pi, new - 2.0 * math.pi, new)
        new = np.where(new <= -math.pi, new + 2.0 * math.pi, new)
        return np.where(live, new, th), E, top, scale * top, (r, F, tau, move)

    def descend(self, thetas, iters, tol):
        th = _wrap(self.pad(thetas))
        E, top, mx = np.zeros((self.B, 3)), np.zeros(self.B), np.zeros(self.B)
        on = np.ones(self.B, bool)
        for _ in range(iters):
            new, e, t, d, (r, F, tau, move) = self.step(th)
            th = np.where(on[:, None], new, th)
            E, top, mx = np.where(on[:, None], e, E), np.where(on, t, top), np.where(on, d, mx)
            on &= ~(mx < tol)
        out = {"theta": self.unpad(th), "energies": E, "max_tau": top, "max_dtheta": mx}
        if self.case["whole"]:
            out.update(xyz=[r[b, :APR * k] for b, k in enumerate(self.m)],
                       force=[F[b, :APR * k] for b, k in enumerate(self.m)], tau=self.unpad(tau), dtheta=self.unpad(move))
        return out

    def search(self, thetas, delta, u):
        vac = self.case["terms"] != "all"
        total = lambda e: e[:, 0] + e[:, 1] + (0.0 if vac else e[:, 2])  # noqa: E731
        acc = _wrap(self.pad(thetas))
        start = low = e_acc = total(self.evaluate(acc)[0])
        best = acc
        for k in range(u.shape[1]):
            move = self.pad([d[k] for d in delta]) * (self.pad([np.ones(d.shape[1]) for d in delta]) == 1.0)
            th = _wrap(acc + move)
            for _ in range(self.case["iters"]):
                th = self.step(th)[0]
            e = total(self.evaluate(th)[0])
            yes = (e <= e_acc) | (u[:, k] < np.exp(np.minimum(0.0, e_acc - e)))
            less = e < low
            best, low = np.where(less[:, None], th, best), np.where(less, e, low)
            acc, e_acc = np.where(yes[:, None], th, acc), np.where(yes, e, e_acc)
        return {"energies": np.stack([start, e_acc, low], axis=1), "best": self.unpad(best), "theta": self.unpad(acc)}
