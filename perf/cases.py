"""Performance cases of the coupled lattice-Boltzmann / bead-dynamics library.

Each case is work that a user's program asks of the library through its Python binding: coupled
steps of one pore box in each storage type, the paper's rigid chain, the trilinear stencil, an
ensemble of replicas with and without the solvent, lattice-only steps of plain and ragged boxes,
the 512^3 box, and the read-out of the fluid fields.  A pass is one block of steps and the small
read-outs that follow it in such a program; its outputs are the updated populations (the
library's own buffer) and the bead state.

The bead dynamics is chaotic: two roundings of one trajectory part by orders of magnitude within
a hundred steps, so blocks are at most 16 coupled steps.  Bead positions and velocities are
returned in the arithmetic type of the storage (FP32 for FP32 and 16-bit storage).

exact() is the same step in 64 bits, written against the method (plain torch): D3Q19 BGK with
half-way bounce-back and specular free-slip faces, kick-drift Langevin beads with harmonic or
rigid bonds, nearest-node or trilinear coupling, Philox4x32-10 random numbers.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_0710_1272_amd import lbmd as B
from workloads import configs as WC
from workloads import generate as G

STORAGE = {"f64": WC.STORE_F64, "f32": WC.STORE_F32, "f16": WC.STORE_F16, "bf16": WC.STORE_BF16}
DTYPE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # the smallest call: one step of a small pore box and its bead state, as an interactive
        # or step-by-step driver makes it; launches and latency decide
        dict(name="pore48_n12_one_step_f32", kind="coupled", storage="f32", nx=48, ny=24, nz=24, beads=12, steps=1),
        # the plain periodic box of the conservation and viscosity studies, FP64, 100 steps
        dict(name="shear32_f64", kind="lattice", storage="f64", nx=32, ny=32, nz=32, periodic=True, walls=0, steps=100),
        # a ragged box (rows that are no whole waves), two walls, BF16
        dict(name="lattice_203x77x91_bf16", kind="lattice", storage="bf16", nx=203, ny=77, nz=91, periodic=False,
             walls=2, steps=16),
        # one translocating chain, the paper's box: the ordinary single run
        dict(name="pore128x64x64_n100_f32", kind="coupled", storage="f32", nx=128, ny=64, nz=64, beads=100, steps=16),
        # the same with the paper's own bead model, rigid bonds and M = 5
        dict(name="pore128x64x64_n100_rigid_f32", kind="coupled", storage="f32", nx=128, ny=64, nz=64, beads=100,
             steps=16, rigid=True),
        # the same with the trilinear coupling stencil in 16-bit storage
        dict(name="pore128x64x64_n100_tri_f16", kind="coupled", storage="f16", nx=128, ny=64, nz=64, beads=100,
             steps=16, trilinear=True),
        # a long chain in a larger box, 16-bit storage
        dict(name="pore256x128x128_n400_f16", kind="coupled", storage="f16", nx=256, ny=128, nz=128, beads=400,
             steps=16),
        # replicas of different sizes and chain lengths in one batch, 16-bit storage
        dict(name="batch24_48to96_f16", kind="ensemble", storage="f16", nx=96, ny=96, nz=96, mixed=True, replicas=24,
             beads=200, steps=8),
        # a translocation-time ensemble of the paper's complete model: rigid chains in a
        # fluctuating fluid, 100x50x50 boxes
        dict(name="ensemble32_100x50x50_rigid_thermal_f32", kind="ensemble", storage="f32", nx=100, ny=50, nz=50,
             replicas=32, beads=60, steps=8, rigid=True, fluid_kT=1e-4),
        # the no-solvent comparison run of an ensemble, with its trajectories
        dict(name="nosolvent16_48_n32_f32", kind="no_solvent", storage="f32", nx=48, ny=48, nz=48, replicas=16,
             beads=32, steps=25),
        # the largest box: two walls, a long chain and crowders, tuned launch shapes as a long
        # run has them
        dict(name="large512_two_walls_f32", kind="coupled", storage="f32", nx=512, ny=512, nz=512, walls=2, beads=800,
             crowders=64, steps=4, flow=False, autotune=True),
        # the fluid fields and conserved totals of a box, copied to the host for a plot or file
        dict(name="fields128x64x64_f32", kind="fields", storage="f32", nx=128, ny=64, nz=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["coupled", "coupled", "coupled", "lattice", "ensemble", "no_solvent", "fields"])
    storage = rng.choice(["f64", "f32", "f32", "f16", "bf16"])
    if kind == "lattice":
        walls = rng.choice([0, 1, 2])
        return dict(kind=kind, storage=storage, nx=_log_int(rng, 32, 256), ny=_log_int(rng, 16, 160),
                    nz=_log_int(rng, 16, 160), periodic=walls == 0 and rng.random() < 0.5, walls=walls,
                    steps=_log_int(rng, 1, 100), fluid_kT=rng.choice([0.0, 0.0, 1e-4]))
    if kind == "coupled":
        nx, ny, nz = _log_int(rng, 48, 256), _log_int(rng, 24, 128), _log_int(rng, 24, 128)
        rigid = rng.random() < 0.3
        most = min(500 if rigid else 900, nx * ny * nz // 160)
        return dict(kind=kind, storage=storage, nx=nx, ny=ny, nz=nz, beads=_log_int(rng, 8, most),
                    steps=rng.randint(1, 16), rigid=rigid, trilinear=rng.random() < 0.25)
    if kind == "ensemble":
        side = rng.randint(40, 72)
        return dict(kind=kind, storage=storage, nx=2 * side, ny=side, nz=side + rng.randint(-5, 5),
                    replicas=rng.randint(2, 32), beads=_log_int(rng, 16, 160), steps=rng.randint(2, 8),
                    rigid=rng.random() < 0.5, fluid_kT=rng.choice([0.0, 1e-4]))
    if kind == "no_solvent":
        return dict(kind=kind, storage=rng.choice(["f64", "f32"]), nx=rng.randint(48, 64), ny=48, nz=48,
                    replicas=rng.randint(2, 24), beads=_log_int(rng, 16, 128), steps=rng.randint(4, 25),
                    rigid=rng.random() < 0.3)
    return dict(kind=kind, storage=storage, nx=_log_int(rng, 32, 160), ny=_log_int(rng, 24, 96),
                nz=_log_int(rng, 24, 96))


# ---------------------------------------------------------------------------------------------
# Inputs, from the case and the seed alone
# ---------------------------------------------------------------------------------------------
def _md(case):
    md = WC.paper_polymer() if case.get("rigid") else WC.MDParams()
    md.stencil = 1 if case.get("trilinear") else 0
    return md


def _replicas(case, seed):
    kT = float(case.get("fluid_kT", 0.0))
    reps = []
    for k in range(case.get("replicas", 1)):
        nx, ny, nz, n = case["nx"], case["ny"], case["nz"], case.get("beads", 0)
        if case.get("mixed"):
            # cubic boxes of 48, 64, 80 and 96 nodes a side and chains of 20 to `beads` beads
            side = (48, 64, 80, 96)[k % 4] * nx // 96
            nx = ny = nz = side
            n = 20 + (n - 20) * ((7 * k + 3) % 24) // 23
        if case.get("walls", 1) == 0:
            bc = (WC.PERIODIC,) * 3 if case.get("periodic") else (WC.FREESLIP,) * 3
            box = WC.Box(nx, ny, nz, bc, (), 1.0, 1.0, kT)
        else:
            box = WC.pore_box(nx, ny, nz, case.get("walls", 1))
            box.fluid_kT = kT
        chains = [n] + [25] * case.get("crowders", 0) if n else []
        reps.append(WC.Replica(box, chains, 1_000_003 * (seed + 1) + k))
    return reps


def _beads(rep, md):
    if not rep.chain_len:
        return np.zeros((0, 3))
    first = G.replica_beads(WC.Replica(rep.box, rep.chain_len[:1], rep.seed), md)
    if len(rep.chain_len) == 1:
        return first
    # crowders: one compact chain in each cell of a grid beyond the first wall, clear of the walls
    rng = np.random.default_rng(rep.seed + 1)
    box, out = rep.box, [first]
    lo, hi = box.walls[0][1] + 36, box.walls[1][0] - 36
    n = len(rep.chain_len) - 1
    side = max(1, int(math.ceil(n ** (1 / 3))))
    free = WC.Box(400, 400, 400, (WC.FREESLIP,) * 3)
    for c in range(n):
        i, j, k = c % side, (c // side) % side, c // side ** 2
        pts = G.grow_chain(free, md, rep.chain_len[1 + c], rng, start=np.array([200.0, 200.0, 200.0]), cis_only=False)
        cell = np.array([lo + (hi - lo) * (i + 0.5) / side, box.ny * (j + 0.5) / side, box.nz * (k + 0.5) / side])
        out.append(pts - pts.mean(axis=0) + cell + rng.random(3))
    return np.concatenate(out)


def _flow(case, rep):
    """A fluid in motion: density 1 +- 0.01 and velocity components within 0.01 at each node."""
    return G.random_small_flow(rep.box, rep.seed % (1 << 31), du=0.01)


def _inputs(case, seed):
    md, reps = _md(case), _replicas(case, seed)
    beads = [_beads(r, md) for r in reps]
    flows = None
    if case.get("flow", True) and case["kind"] != "no_solvent":
        flows = [_flow(case, r) for r in reps]
    return md, reps, beads, flows


def prepare(case, seed):
    md, reps, beads, flows = _inputs(case, seed)
    init = {}
    if sum(len(b) for b in beads):
        init["bead_r"] = np.concatenate(beads)
    if flows is not None:
        init["rho"] = np.concatenate([f[0] for f in flows])
        init["u"] = np.concatenate([f[1].ravel() for f in flows])
    flags = B.LB_CFG_AUTOTUNE if case.get("autotune") else 0
    sim = B.Simulation(reps, md, STORAGE[case["storage"]], init, flags=flags)
    state = {"case": case, "sim": sim, "updates": 0, "reps": reps}
    if case["kind"] != "fields":
        coupled, hydro = case["kind"] in ("coupled", "ensemble"), case["kind"] != "no_solvent"
        sim.prepare(case["steps"], coupled=coupled, hydro=hydro)
    if case["kind"] in ("coupled", "ensemble", "lattice"):
        # views of the replicas' populations in the caller-visible buffers ([19][S], S >= V)
        views = []
        for buf in sim._tensors[:2]:
            flat, at, per = buf.view(DTYPE[case["storage"]]), 0, []
            for k, r in enumerate(reps):
                S = sim.plane_stride(k)
                per.append(torch.as_strided(flat, (19, r.box.nodes), (S, 1), at))
                at += 19 * S
            views.append(per)
        state["views"] = views
    return state


def run(state):
    case, sim = state["case"], state["sim"]
    kind = case["kind"]
    if kind == "fields":
        rho, u = sim.fields()
        return {"conserved": sim.conserved(), "rho": rho, "u": u}
    if kind == "no_solvent":
        sim.step(case["steps"], hydro=False)
        return {"beads": _bead_state(case, sim, range(len(state["reps"])))}
    sim.step(case["steps"], coupled=kind != "lattice")
    state["updates"] += case["steps"]
    out = {"pops": state["views"][state["updates"] & 1]}
    if kind == "coupled":
        out["beads"] = _bead_state(case, sim, [0])
    if kind == "ensemble":
        # the poll of an ensemble driver: every replica's translocation state
        t = [sim.transloc(k) for k in range(len(state["reps"]))]
        out["n_t"] = np.array([d["n_t"] for d in t])
        out["t_done"] = np.array([d["t_done"] for d in t])
        out["com"] = np.array([d["com"] for d in t], dtype=np.float64 if case["storage"] == "f64" else np.float32)
    return out


def _bead_state(case, sim, replicas):
    real = np.float64 if case["storage"] == "f64" else np.float32
    rv = [sim.beads(k) for k in replicas]
    return [np.concatenate([r for r, _ in rv]).astype(real), np.concatenate([v for _, v in rv]).astype(real)]


def work(case):
    """Bytes: populations read and written once a step, bead state once a pass.  Operations: about
    250 a node update, 400 a bead and substep."""
    reps = _replicas(case, 0)
    nodes = sum(r.box.fluid_nodes() for r in reps)
    beads = sum(r.n_beads for r in reps)
    if case["kind"] == "fields":
        return {"bytes": nodes * (19 * BYTES[case["storage"]] + 32), "flops": nodes * 40}
    lattice = 0 if case["kind"] == "no_solvent" else nodes
    moved = lattice * 2 * 19 * BYTES[case["storage"]] * case["steps"] + beads * 96
    return {"bytes": moved, "flops": case["steps"] * (250 * lattice + beads * 400 * _md(case).M)}


# ---------------------------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------------------------
CX = [0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0]
CY = [0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1]
CZ = [0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1]
WT = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
SCALE = [2.0] + [16.0] * 6 + [32.0] * 12
VEL = list(zip(CX, CY, CZ))
M32 = 0xFFFFFFFF


def _philox(c, key):
    """Philox4x32-10 (Salmon et al., SC'11) of four int64 tensors of 32-bit words."""
    k0, k1 = key & M32, (key >> 32) & M32

    def mul(m, x):
        lo, hi = m * (x & 0xFFFF), m * (x >> 16)
        t = hi + (lo >> 16)
        return t >> 16, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)

    for _ in range(10):
        ah, al = mul(0xD2511F53, c[0])
        bh, bl = mul(0xCD9E8D57, c[2])
        c = [bh ^ c[1] ^ k0, bl, ah ^ c[3] ^ k1, al]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c


class _Exact:
    """One replica in 64 bits."""

    def __init__(self, rep, md, beads, flow, lattice):
        self.dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.rep, self.md, self.box, self.step_no = rep, md, rep.box, 0
        self.n = (rep.box.nx, rep.box.ny, rep.box.nz)
        self.r = torch.tensor(beads, dtype=torch.float64)
        self.v = torch.zeros_like(self.r)
        ids = np.repeat(np.arange(len(rep.chain_len)), rep.chain_len)
        self.bond = torch.tensor(np.append(ids[1:] == ids[:-1], False) if len(ids) else np.zeros(0, bool))
        self.t_done = -1
        self.u = torch.zeros_like(self.r)
        if lattice:
            self._lattice(flow)

    # -- lattice
    def _solid(self, x, y, z):
        s = torch.zeros_like(x, dtype=torch.bool)
        for (x0, x1, y0, y1, z0, z1) in self.box.walls:
            s |= (x >= x0) & (x <= x1) & ~((y >= y0) & (y <= y1) & (z >= z0) & (z <= z1))
        return s

    def _lattice(self, flow):
        nx, ny, nz = self.n
        V = nx * ny * nz
        i = torch.arange(V, device=self.dev)
        X = [i % nx, (i // nx) % ny, i // (nx * ny)]
        self.fluid = ~self._solid(*X)
        self.src = torch.empty((19, V), dtype=torch.int64, device=self.dev)
        for p in range(19):
            s, flips = [], []
            for a in range(3):
                t = X[a] - VEL[p][a]
                out = (t < 0) | (t >= self.n[a])
                if self.box.bc[a] == WC.FREESLIP:
                    t = torch.where(out, X[a], t)
                else:
                    t, out = t % self.n[a], torch.zeros_like(out)
                s.append(t)
                flips.append(out)
            q = torch.zeros_like(i)
            for m in range(8):
                if any((m >> a) & 1 and VEL[p][a] == 0 for a in range(3)):
                    continue
                want = tuple(-VEL[p][a] if (m >> a) & 1 else VEL[p][a] for a in range(3))
                hit = torch.ones_like(flips[0])
                for a in range(3):
                    hit &= flips[a] == bool((m >> a) & 1) if VEL[p][a] else True
                q[hit] = VEL.index(want)
            solid = self._solid(*s)
            q = torch.where(solid, VEL.index(tuple(-c for c in VEL[p])), q)
            at = torch.where(solid, i, s[0] + nx * (s[1] + ny * s[2]))
            self.src[p] = q * V + at
            del s, flips, q, solid, at
        rho = torch.full((V,), self.box.rho0, dtype=torch.float64, device=self.dev)
        u = torch.zeros((3, V), dtype=torch.float64, device=self.dev)
        if flow is not None:
            rho, u = (torch.tensor(t, dtype=torch.float64, device=self.dev) for t in flow)
        self.post = torch.empty((19, V), dtype=torch.float64, device=self.dev)
        for p in range(19):
            self.post[p] = WT[p] * self.box.rho0
        for p in range(19):
            self.post.view(-1)[self.src[p][self.fluid]] = self._feq(p, rho, u)[self.fluid]

    def _feq(self, p, rho, u):
        cu = VEL[p][0] * u[0] + VEL[p][1] * u[1] + VEL[p][2] * u[2]
        return WT[p] * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * (u[0] ** 2 + u[1] ** 2 + u[2] ** 2))

    def moments(self, f):
        rho = f.sum(0)
        j = [sum(VEL[p][a] * f[p] for p in range(19) if VEL[p][a]) for a in range(3)]
        return rho, torch.stack([c / rho for c in j])

    def stream_collide(self):
        om = 1.0 / self.box.tau
        f = torch.empty_like(self.post)
        for p in range(19):
            f[p] = self.post.view(-1)[self.src[p]]
        rho, u = self.moments(f)
        for p in range(19):
            f[p] += om * (self._feq(p, rho, u) - f[p])
        if self.box.fluid_kT > 0:
            self._thermal(f, rho, om)
        for p in range(19):
            self.post[p] = torch.where(self.fluid, f[p], WT[p] * self.box.rho0)

    def _thermal(self, f, rho, om):
        V = rho.numel()
        node = torch.arange(V, device=self.dev)
        eta = []
        for j in range(5):
            z = torch.zeros_like(node)
            w = _philox([node, z + (self.step_no & M32), z + j, z + 2], self.rep.seed)
            eta += [((t >> 8).double() + 0.5) / 2.0 ** 24 - 0.5 for t in w]
        eta = [math.sqrt(12 * WT[p]) * eta[p] for p in range(19)]
        phi = torch.sqrt(3 * self.box.fluid_kT * rho * (1 - (1 - om) ** 2))
        s = sum(eta)
        sc = [sum(VEL[p][a] * eta[p] for p in range(19) if VEL[p][a]) for a in range(3)]
        for p in range(19):
            f[p] += phi * (eta[p] - WT[p] * (s + 3 * sum(VEL[p][a] * sc[a] for a in range(3))))

    # -- coupling: nodes and weights of each bead, then the velocity there and the reaction
    def stencil(self):
        nodes = []
        base = torch.floor(self.r) if self.md.stencil else torch.floor(self.r + 0.5)
        fr = self.r - base
        for c in range(8 if self.md.stencil else 1):
            w = torch.ones(len(self.r), dtype=torch.float64)
            x = []
            for a in range(3):
                d = (c >> a) & 1
                if self.md.stencil:
                    w = w * (fr[:, a] if d else 1 - fr[:, a])
                t = base[:, a].long() + d
                x.append(t.clamp(0, self.n[a] - 1) if self.box.bc[a] == WC.FREESLIP else t % self.n[a])
            ok = ~self._solid(*x)
            nodes.append((x[0] + self.n[0] * (x[1] + self.n[1] * x[2]), w * ok))
        return nodes

    def interpolate(self, nodes):
        self.u = torch.zeros_like(self.r)
        for at, w in nodes:
            f = self.post.view(-1)[self.src[:, at.to(self.dev)]]
            _, u = self.moments(f)
            self.u += torch.where(w > 0, w, 0.0)[:, None] * u.T.cpu()

    def spread(self, nodes, fbar):
        for at, w in nodes:
            for p in range(1, 19):
                s = -3 * WT[p] * w * sum(VEL[p][a] * fbar[:, a] for a in range(3))
                self.post[p].index_add_(0, at.to(self.dev), s.to(self.dev))

    # -- beads
    def _wca(self, d, d2, eps, sigma):
        s6 = (sigma * sigma / d2) ** 3
        on = (d2 < 2 ** (1 / 3) * sigma * sigma) & (d2 > 0)
        c = torch.where(on, 24 * eps * (2 * s6 * s6 - s6) / d2, 0.0)
        return c[..., None] * d

    def forces(self):
        md, r, n = self.md, self.r, len(self.r)
        d = r[:, None, :] - r[None, :, :]
        d2 = (d * d).sum(-1)
        d2.fill_diagonal_(1e9)
        b = torch.nonzero(self.bond).flatten()
        d2[b, b + 1] = 1e9
        d2[b + 1, b] = 1e9
        F = self._wca(d, d2, md.eps, md.sigma).sum(1)
        if not md.rigid and len(b):
            e = r[b] - r[b + 1]
            f = -md.k_bond * (1 - md.r0 / e.norm(dim=1, keepdim=True)) * e
            F[b] += f
            F[b + 1] -= f
        node = torch.floor(r + 0.5)
        best = torch.full((n,), math.inf, dtype=torch.float64)
        vec = torch.zeros_like(r)
        for (x0, x1, y0, y1, z0, z1) in self.box.walls:
            dv = torch.zeros_like(r)
            dv[:, 0] = r[:, 0] - r[:, 0].clamp(x0 - 0.5, x1 + 0.5)
            sides = torch.stack([r[:, 1] - (y0 - 0.5), (y1 + 0.5) - r[:, 1], r[:, 2] - (z0 - 0.5), (z1 + 0.5) - r[:, 2]])
            m, k = sides.min(0)
            inside = m >= 0
            for s, (a, sg) in enumerate(((1, 1), (1, -1), (2, 1), (2, -1))):
                dv[:, a] += torch.where(inside & (k == s), sg * m, 0.0)
            q = (dv * dv).sum(1)
            vec = torch.where((q < best)[:, None], dv, vec)
            best = torch.minimum(q, best)
            pore = ((node[:, 0] >= x0) & (node[:, 0] <= x1) & (node[:, 1] >= y0) & (node[:, 1] <= y1)
                    & (node[:, 2] >= z0) & (node[:, 2] <= z1))
            F[:, 0] += pore.double() * (md.drive_sign * md.f_drive)
        F += self._wca(vec, best, md.eps_w, md.sigma_w)
        for a in range(3):
            if self.box.bc[a] == WC.FREESLIP:
                for d1, sg in ((r[:, a] + 0.5, 1.0), (self.n[a] - 0.5 - r[:, a], -1.0)):
                    F[:, a] += sg * self._wca(d1[:, None], d1 * d1, md.eps_w, md.sigma_w)[:, 0]
        return F

    def _rigid(self, r_old):
        """SHAKE on the positions, then RATTLE on the velocities (dense solves)."""
        md = self.md
        b = torch.nonzero(self.bond).flatten()
        m = len(b)
        C = torch.zeros((m, len(self.r)), dtype=torch.float64)
        C[torch.arange(m), b], C[torch.arange(m), b + 1] = 1.0, -1.0
        K = C @ C.T / md.mass
        d = C @ r_old
        lam = torch.zeros(m, dtype=torch.float64)
        free = self.r
        for _ in range(md.shake_iter):
            s = C @ (free + C.T @ (lam[:, None] * d) / md.mass)
            g = (s * s).sum(1) - md.r0 ** 2
            if g.abs().max() <= md.shake_tol * md.r0 ** 2:
                break
            lam = lam - torch.linalg.solve(2 * (s @ d.T) * K, g)
        self.r = free + C.T @ (lam[:, None] * d) / md.mass
        self.v = (self.r - r_old) * md.M
        s = C @ self.r
        mu = torch.linalg.solve((s @ s.T) * K, -((C @ self.v) * s).sum(1))
        self.v = self.v + C.T @ (mu[:, None] * s) / md.mass

    def substeps(self):
        md, n = self.md, len(self.r)
        h = 1.0 / md.M
        A = math.sqrt(24 * md.mass * md.gamma * md.kT / h)
        fbar = torch.zeros_like(self.r)
        i = torch.arange(n)
        for sub in range(md.M):
            w = _philox([i, 0 * i + (self.step_no & M32), 0 * i + sub, 0 * i + 1], self.rep.seed)[:3]
            w = [(t & 0xFFFFFF00) - ((t >> 31) << 32) for t in w]
            noise = A * torch.stack(w, 1).double() / 2.0 ** 32
            drag = -md.mass * md.gamma * (self.v - self.u)
            F = self.forces() + drag + noise
            fbar += (drag + noise) / md.M
            r_old = self.r
            self.v = self.v + h / md.mass * F
            self.r = self.r + h * self.v
            if md.rigid and self.bond.any():
                self._rigid(r_old)
        return fbar

    def step(self, kind):
        n = len(self.r)
        if kind == "lattice" or n == 0:
            self.stream_collide()
        elif kind == "no_solvent":
            self.substeps()
        else:
            nodes = self.stencil()
            self.interpolate(nodes)
            fbar = self.substeps()
            self.stream_collide()
            self.spread(nodes, fbar)
        self.step_no += 1
        if n and self.t_done < 0 and int((self.r[:, 0] > self.xmid()).sum()) == n:
            self.t_done = self.step_no

    def xmid(self):
        return 0.5 * (self.box.walls[0][0] + self.box.walls[0][1]) if self.box.walls else 0.5 * (self.n[0] - 1)


def exact(case, seed):
    nodes = sum(r.box.nodes for r in _replicas(case, seed))
    if not torch.cuda.is_available() and nodes * case.get("steps", 1) > 3e7:
        return None  # minutes on a CPU
    torch.set_num_threads(min(8, torch.get_num_threads()))
    md, reps, beads, flows = _inputs(case, seed)
    kind, out = case["kind"], []
    pops, r, v, n_t, t_done, com = [], [], [], [], [], []
    for k, rep in enumerate(reps):
        e = _Exact(rep, md, beads[k], flows[k] if flows is not None else None, kind != "no_solvent")
        if kind == "fields":
            rho = torch.where(e.fluid, torch.tensor(flows[k][0], device=e.dev), 0.0)
            u = torch.where(e.fluid, torch.tensor(flows[k][1], device=e.dev), 0.0)
            total = [float(rho.sum())] + [float((rho * u[a]).sum()) for a in range(3)]
            return {"conserved": np.array(total), "rho": rho, "u": u}
        for _ in range(case["steps"]):
            e.step(kind)
        if kind != "no_solvent":
            if case["storage"] in ("f16", "bf16"):
                for p in range(19):
                    e.post[p] = (e.post[p] - WT[p] * rep.box.rho0) * SCALE[p]
            pops.append(e.post)
        r.append(e.r)
        v.append(e.v)
        n_t.append(int((e.r[:, 0] > e.xmid()).sum()))
        t_done.append(e.t_done)
        com.append(e.r.mean(0).numpy() if len(e.r) else np.zeros(3))
    out = {"pops": pops} if kind != "no_solvent" else {}
    if kind in ("coupled", "no_solvent"):
        out["beads"] = [torch.cat(r), torch.cat(v)]
    if kind == "ensemble":
        out.update(n_t=np.array(n_t), t_done=np.array(t_done), com=np.array(com))
    return out
