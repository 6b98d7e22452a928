"""The engine's performance cases: what its users have it do, over the sizes of the repository's workloads.

A case names one pass through the public entry points (``System``, ``Batch``, ``RigidBodies``, ``SwapModel``):

* ``md``      n steps of Langevin or NVE dynamics of one system, continued from pass to pass
* ``batch``   the same for a set of independent replicas advanced together
* ``rigid``   steps of the planar mixture of rigid patchy disks
* ``build``   one neighbour-list build (cell sort and list)
* ``frame``   the evaluation of one configuration: forces, energy, virial, bond count, soft bond count
* ``forces``  forces, energy and virial alone, called in a loop
* ``hvp``     Hessian-vector products of many tangent vectors (normal modes, Lanczos)
* ``grad``    one differentiated evaluation: energy and forces forward, gradients of positions and parameters backward
* ``stress``  the stress autocorrelation of a logged series

Inputs are made from the seed alone.  Positions are jittered lattices of molecules in the composition the dynamics
leads to (dumbbells, bonded sites, chains), so that they are quick to make at every size and start free of overlaps.
Dynamics are reported by tag, with positions unwrapped, since the engine re-orders particles and folds them.  Single
evaluations take configurations stored along the cells' Morton curve (as a saved run's are), so that the engine's order
is theirs.
``exact`` evaluates the same definitions in FP64 with plain torch.
"""
import math

import numpy as np
import torch

from paper_1912_08569_amd import Batch, RigidBodies, System
from paper_1912_08569_amd.autograd import SwapModel, swap_energy, swap_forces

NONE, SWAP, WCA = 0, 1, 2
WCA_CUT = 2.0 ** (1.0 / 6.0)


def listed():
    return [
        # the smallest system of the dumbbell scaling study: latency and launches decide
        dict(name="md_dumbbells_512", kind="md", system="dumbbells", n=512, rcut=1.3, steps=100, log=100),
        # the middle of that study, at a size that fills no block evenly; the two-pass form of the step
        dict(name="md_dumbbells_20011", kind="md", system="dumbbells", n=20011, rcut=1.3, steps=100, log=100),
        # the headline workload: the self-assembly mixture at full size, without logging
        dict(name="md_assembly_1048576", kind="md", system="assembly", n=1048576, lam=1.0, steps=40, log=0),
        # the vitrimer-like network: dense, springs, crosslinkers
        dict(name="md_network_67200", kind="md", system="network", n=67200, steps=40, log=100),
        # a parameter sweep: replicas of uneven size, density, lambda and composition advanced together
        dict(name="batch_96", kind="batch", replicas=96, n_lo=500, n_hi=20000, steps=20, log=0),
        # the planar patchy mixture: 1000 rigid disks, 3 or 2 patches each
        dict(name="rigid_1000", kind="rigid", bodies=1000, steps=40),
        # a list build of the large mixture (every ~40 steps of a run)
        dict(name="build_assembly_1000003", kind="build", system="assembly", n=1000003, lam=1.0),
        # a saved configuration evaluated: several types with unequal coefficients, the default force kernel
        dict(name="frame_unequal_200003", kind="frame", system="unequal", n=200003),
        # forces in a caller's own loop at the validation system's size
        dict(name="forces_reactive_1000", kind="forces", system="reactive", n=1000, density=0.2, eps=1.0, path="gather"),
        # the differentiation workload: 64 tangent vectors at once
        dict(name="hvp_32768x64", kind="hvp", system="reactive", n=32768, density=0.25, eps=10.0, nvec=64),
        # one differentiated evaluation of a fit: energy and forces, gradients of positions and parameters
        dict(name="grad_reactive_32768", kind="grad", system="reactive", n=32768, density=0.25, eps=10.0),
        # the relaxation modulus of a long logged run
        dict(name="stress_20000x5000", kind="stress", rows=20000, lags=5000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["md", "md", "md", "batch", "rigid", "build", "frame", "forces", "hvp", "grad", "stress"])
    if kind == "md":
        system = rng.choice(["dumbbells", "dumbbells", "assembly", "network"])
        c = dict(kind="md", system=system, log=rng.choice([0, 50, 100]))
        if system == "dumbbells":
            c.update(n=_log(rng, 512, 131072), rcut=rng.choice([1.15, 1.3]), steps=rng.randint(20, 100))
        elif system == "assembly":
            c.update(n=_log(rng, 4096, 1048576), lam=rng.choice([0.0, 0.5, 1.0, 1.5]), steps=rng.randint(20, 40))
        else:
            c.update(n=_log(rng, 4000, 67200), steps=rng.randint(20, 40))
        return c
    if kind == "batch":
        return dict(kind="batch", replicas=_log(rng, 8, 96), n_lo=500, n_hi=_log(rng, 2000, 20000),
                    steps=rng.randint(10, 20), log=rng.choice([0, 10]))
    if kind == "rigid":
        return dict(kind="rigid", bodies=_log(rng, 100, 1000), steps=rng.randint(10, 40))
    if kind == "build":
        s = rng.choice(["assembly", "dumbbells", "reactive"])
        c = dict(kind="build", system=s, n=_log(rng, 1000, 1000003))
        c.update({"assembly": dict(lam=1.0), "dumbbells": dict(rcut=1.3), "reactive": dict(density=0.25, eps=1.0)}[s])
        return c
    if kind == "frame":
        return dict(kind="frame", system="unequal", n=_log(rng, 2000, 200003))
    if kind == "forces":
        return dict(kind="forces", system="reactive", n=_log(rng, 1000, 100000), density=rng.choice([0.2, 0.25, 0.35]),
                    eps=1.0, path=rng.choice(["triplet", "gather", "sums"]))
    if kind == "hvp":
        return dict(kind="hvp", system="reactive", n=_log(rng, 1000, 32768), density=0.25,
                    eps=rng.choice([1.0, 10.0]), nvec=_log(rng, 1, 64))
    if kind == "grad":
        return dict(kind="grad", system=rng.choice(["reactive", "unequal"]), n=_log(rng, 2000, 32768), density=0.25,
                    eps=rng.choice([1.0, 10.0]))
    rows = _log(rng, 500, 20000)
    return dict(kind="stress", rows=rows, lags=rng.randint(rows // 20, rows // 4))


# ---- coefficient tables --------------------------------------------------------------------------------------

class Table:
    """Symmetric per-type-pair coefficients, as the engine takes them."""

    def __init__(self, nt):
        self.kind = np.zeros((nt, nt), np.int32)
        self.epsilon = np.zeros((nt, nt))
        self.sigma = np.ones((nt, nt))
        self.n = np.full((nt, nt), 6, np.int32)
        self.rcut = np.zeros((nt, nt))
        self.lam = np.zeros((nt, nt))

    def copy(self):
        t = Table(self.kind.shape[0])
        for k, v in self.__dict__.items():
            setattr(t, k, v.copy())
        return t

    def swap(self, a, b, eps, sigma, n, rcut, lam):
        for p, q in ((a, b), (b, a)):
            self.kind[p, q], self.epsilon[p, q], self.sigma[p, q] = SWAP, eps, sigma
            self.n[p, q], self.rcut[p, q], self.lam[p, q] = n, rcut, lam
        return self

    def wca(self, a, b, sigma=1.0, eps=1.0):
        for p, q in ((a, b), (b, a)):
            self.kind[p, q], self.epsilon[p, q], self.sigma[p, q], self.rcut[p, q] = WCA, eps, sigma, WCA_CUT * sigma
        return self


class Sys:
    """A system as its generator leaves it (the attributes System, Batch and exact() read)."""

    def __init__(self, pos, types, L, table, rng, kT, **more):
        self.pos, self.types, self.L, self.table = pos, types, L, table
        self.mass = np.ones(table.kind.shape[0])
        self.vel = (rng.standard_normal(pos.shape) * math.sqrt(kT)).astype(np.float32)
        self.bonds = self.fene = None
        self.__dict__.update(more)


# ---- configurations ------------------------------------------------------------------------------------------

def _edge(n, density):
    return float(np.float32((n / density) ** (1.0 / 3.0)))


def _dims(m):
    a = math.ceil(round(m ** (1.0 / 3.0), 9))
    b = math.ceil(math.sqrt(m / a))
    return a, b, math.ceil(m / (a * b))


def _fold(x, L):
    """Unwrapped float64 coordinates to FP32 in [-L/2, L/2)."""
    L = np.asarray(L, np.float64)
    y = (x - L * np.floor(x / L + 0.5)).astype(np.float32)
    h = (0.5 * L).astype(np.float32)
    return np.where(y >= h, -h, np.maximum(y, -h)).astype(np.float32)


def _sites(rng, m, L, gap):
    """m of the sites of a lattice that fills the box, each jittered so that two stay `gap` apart."""
    d = _dims(m)
    h = np.array([L / k for k in d])
    at = rng.permutation(d[0] * d[1] * d[2])[:m]
    x = np.stack([at % d[0], (at // d[0]) % d[1], at // (d[0] * d[1])], axis=1) + 0.5
    jit = np.maximum(0.0, 0.5 * (h - gap))
    return x * h - 0.5 * L + rng.uniform(-1.0, 1.0, (m, 3)) * jit


def _directions(rng, m):
    v = rng.standard_normal((m, 3))
    return v / np.linalg.norm(v, axis=1)[:, None]


def _dumbbells(c, rng):
    """A:B = 3:2 at density 0.125, kT 0.03: every B holds an A, the other A are free."""
    n = c["n"]
    nb = int(round(0.4 * n))
    t = Table(2).wca(0, 0).wca(1, 1).swap(0, 1, 1.0, 1.0, 100, c["rcut"], 1.0)
    L = _edge(n, 0.125)
    x = _sites(rng, n - nb, L, 2.1)
    half = 0.5 * (2.0 ** 0.01 + 0.001 * np.clip(rng.standard_normal(nb), -2.5, 2.5))[:, None] * _directions(rng, nb)
    pos = np.concatenate([x[:nb] - half, x[nb:], x[:nb] + half])
    types = np.concatenate([np.zeros(n - nb, np.int32), np.ones(nb, np.int32)])
    p = rng.permutation(n)
    return Sys(_fold(pos, L)[p], types[p], L, t, rng, 0.03)


def _assembly(c, rng):
    """Colloids and reactive sites 1:1 at density 0.3, kT 0.05: 30 % of the sites bonded in pairs, 3 % in triplets."""
    n = c["n"]
    t = Table(2).wca(0, 0).wca(0, 1, 0.65).swap(1, 1, 15.0, 0.3, 10, 0.45, c["lam"])
    L = _edge(n, 0.3)
    ns = n // 2
    n3 = int(0.01 * ns)
    n2 = int(0.15 * ns)
    single = n - 2 * n2 - 3 * n3
    x = _sites(rng, single + n2 + n3, L, 1.1)        # a triplet's ends lie up to 0.4 from its middle site
    rm = 0.3 * 2.0 ** 0.1
    mid, far = x[single:], _directions(rng, n2 + n3)
    bond = (rm + 0.0013 * np.clip(rng.standard_normal(n2 + n3), -2.5, 2.5))[:, None]
    lean = np.where(np.arange(n2 + n3) < n2, 0.5, 0.0)[:, None]
    pos = np.concatenate([x[:single], mid - (1.0 - lean) * bond * far, mid + lean * bond * far,
                          mid[n2:] + rng.uniform(1.05 * rm, 0.4, (n3, 1)) * far[n2:]])
    types = np.ones(n, np.int32)
    types[:n - ns] = 0
    p = rng.permutation(n)
    return Sys(_fold(pos, L)[p], types[p], L, t, rng, 0.05)


def _reactive(c, rng):
    """Identical reactive particles (swap eps, sigma 1, n 10, r_cut 1.5, lambda 1), kT 0.1."""
    L = _edge(c["n"], c["density"])
    t = Table(1).swap(0, 0, c["eps"], 1.0, 10, 1.5, 1.0)
    return Sys(_fold(_sites(rng, c["n"], L, 0.95), L), np.zeros(c["n"], np.int32), L, t, rng, 0.1)


def _unequal(c, rng):
    """Three reactive types with their own lambda, eps, sigma and cutoff per pair, thirds, density 0.3."""
    n = c["n"]
    t = Table(3).swap(0, 0, 1.0, 1.0, 10, 1.5, 1.0).swap(0, 1, 1.5, 0.9, 10, 1.4, 0.4)
    t.swap(0, 2, 0.8, 1.1, 10, 1.6, 1.7).swap(1, 2, 2.0, 1.0, 10, 1.5, 0.9).wca(1, 1, 0.9)
    L = _edge(n, 0.3)
    return Sys(_fold(_sites(rng, n, L, 0.9), L), rng.integers(0, 3, n).astype(np.int32), L, t, rng, 0.1)


def _network(c, rng):
    """Chains of 16 beads and crosslinker dimers (FENE K 30, R0 1.5) at density 0.85, kT 1; 10 % of the chain
    beads are reactive sites.  The molecules follow each other along a path through a lattice."""
    n = c["n"]
    t = Table(3).wca(0, 0).wca(0, 1).wca(0, 2).wca(2, 2)
    t.swap(1, 1, 20.0, 0.3, 10, 0.45, 1.0).swap(1, 2, 20.0, 0.3, 10, 0.45, 1.0)
    L = _edge(n, 0.85)
    d = _dims(n)
    h = np.array([L / k for k in d])
    at = np.arange(n)
    ix, iy, iz = at % d[0], (at // d[0]) % d[1], at // (d[0] * d[1])
    ix = np.where((at // d[0]) % 2 == 1, d[0] - 1 - ix, ix)
    iy = np.where(iz % 2 == 1, d[1] - 1 - iy, iy)
    pos = (np.stack([ix, iy, iz], axis=1) + 0.5) * h - 0.5 * L + rng.uniform(-0.03, 0.03, (n, 3))
    nd = int(n / 42)                                 # dimers: one for every 2.5 chains
    size = np.array([2] * nd + [16] * ((n - 2 * nd) // 16))
    rng.shuffle(size)
    of = np.repeat(np.arange(len(size)), size)       # molecule of every bead; the last few stay alone
    of = np.concatenate([of, len(size) + np.arange(n - len(of))])
    joined = of[1:] == of[:-1]
    bonds = np.full((n, 2), -1, np.int32)
    bonds[:-1, 1][joined] = at[1:][joined]
    bonds[1:, 0][joined] = at[:-1][joined]
    chain = np.concatenate([size[of[of < len(size)]] == 16, np.ones(int((of >= len(size)).sum()), bool)])
    types = np.where(chain, np.where(rng.random(n) < 0.1, 1, 0), 2).astype(np.int32)
    return Sys(_fold(pos, L), types, L, t, rng, 1.0, bonds=bonds, fene=(30.0, 1.5))


def _replicas(c, rng):
    """Replicas of log-uniform size, density 0.2-0.4, lambda 0-1.5 and 0-50 % inert particles.  The sweep (sizes and
    parameters) is the case's, the configurations and the noise are the seed's."""
    sweep = np.random.default_rng([c["replicas"], c["n_lo"], c["n_hi"]])
    out = []
    for _ in range(c["replicas"]):
        n = int(round(math.exp(sweep.uniform(math.log(c["n_lo"]), math.log(c["n_hi"])))))
        L = _edge(n, sweep.uniform(0.2, 0.4))
        t = Table(2).swap(0, 0, 1.0, 1.0, 10, 1.5, float(sweep.uniform(0.0, 1.5))).wca(0, 1).wca(1, 1)
        types = (rng.random(n) < sweep.uniform(0.0, 0.5)).astype(np.int32)
        out.append(Sys(_fold(_sites(rng, n, L, 0.95), L), types, L, t, rng, 0.1))
    return out


def _patchy(c, rng):
    """2 : 3 trifunctional and difunctional disks of diameter 1 with rim patches, in the plane, kT 1."""
    B = c["bodies"]
    n3 = int(round(0.4 * B))
    L = float(np.float32(39.63 * math.sqrt(B / 1000.0)))
    t = Table(3).wca(0, 0).wca(0, 1).wca(1, 1).swap(2, 2, 10.0, 0.1, 6, 0.2, 1.0)
    mx = math.ceil(round(math.sqrt(B), 9))
    my = math.ceil(B / mx)
    h = np.array([L / mx, L / my])
    at = np.sort(rng.permutation(mx * my)[:B])
    cen = np.zeros((B, 3))
    cen[:, :2] = (np.stack([at % mx, at // mx], axis=1) + 0.5) * h - 0.5 * L
    cen[:, :2] += rng.uniform(-1.0, 1.0, (B, 2)) * np.maximum(0.0, 0.5 * (h - 0.98))
    ctype = np.array([0] * n3 + [1] * (B - n3), np.int32)
    rng.shuffle(ctype)
    arms = np.where(ctype == 0, 3, 2)
    first = np.concatenate([[0], np.cumsum(arms)]).astype(np.int32)
    own = np.repeat(np.arange(B), arms)
    ang = (np.arange(len(own)) - first[own]) * (2.0 * math.pi / arms[own])
    offset = (0.5 * np.stack([np.cos(ang), np.sin(ang)], axis=1)).astype(np.float32)
    theta = rng.uniform(-math.pi, math.pi, B).astype(np.float32)

    def rim():
        th = theta.astype(np.float64)[own] + ang
        return cen[own] + 0.5 * np.stack([np.cos(th), np.sin(th), 0.0 * th], axis=1)

    for _ in range(200):     # patches of different bodies start outside the core of their stiff term
        p = torch.from_numpy(rim()[:, :2])
        i, j, _ = _pairs(torch.cat([p, 0 * p[:, :1]], dim=1), (L, L, 8.0), 0.15)
        i, j = i.numpy(), j.numpy()
        bad = np.unique(own[i][own[i] != own[j]])
        if not len(bad):
            break
        theta[bad] = rng.uniform(-math.pi, math.pi, len(bad))
    inertia = np.full(B, 0.125, np.float32)
    omega = (rng.standard_normal(B) / np.sqrt(inertia)).astype(np.float32)
    pos = np.concatenate([cen, rim()])
    s = Sys(_fold(pos, (L, L, 8.0)), np.concatenate([ctype, np.full(len(own), 2, np.int32)]), (L, L, 8.0), t, rng, 1.0)
    s.vel[:, 2] = 0.0
    d = rim() - cen[own]
    s.vel[B:, 0] = s.vel[own, 0] - omega[own] * d[:, 1]
    s.vel[B:, 1] = s.vel[own, 1] + omega[own] * d[:, 0]
    s.bodies = dict(centre=np.arange(B, dtype=np.int32), first=first,
                    member=np.arange(B, B + len(own), dtype=np.int32), offset=offset, inertia=inertia)
    s.theta, s.omega = theta, omega
    return s


_MAKE = dict(dumbbells=_dumbbells, assembly=_assembly, reactive=_reactive, unequal=_unequal, network=_network)
#: dt and kT of the workloads
_DYN = dict(dumbbells=(0.001, 0.03), assembly=(0.001, 0.05), network=(0.001, 1.0), batch=(0.002, 0.1), rigid=(0.001, 1.0))


def _inputs(case, seed):
    rng = np.random.default_rng([seed, 1912])
    if case["kind"] == "batch":
        return _replicas(case, rng), rng
    if case["kind"] == "rigid":
        return _patchy(case, rng), rng
    if case["kind"] == "stress":
        return None, rng
    s = _MAKE[case["system"]](case, rng)
    return (_curved(s) if case["kind"] in ("frame", "forces", "hvp") else s), rng


def _curved(s, skin=0.3):
    """The particles sorted along the Morton curve of cells one list radius wide (in FP32, as positions are)."""
    L = np.float64(s.L)
    nc = min(256, max(3, int(L / ((float(s.table.rcut.max()) + skin) * (1.0 + 1e-5)))))
    c = np.clip(np.floor((s.pos + np.float32(0.5 * L)) * np.float32(nc / L)).astype(np.int64), 0, nc - 1)
    key = sum(((c[:, d] >> b) & 1) << (3 * b + d) for b in range(8) for d in range(3))
    p = np.argsort(key, kind="stable")
    s.pos, s.vel, s.types = s.pos[p], s.vel[p], s.types[p]
    return s


def _rows(case, rng):
    """A logged series (E, W(6), K(6)): correlated noise over a few to a few hundred rows around its means."""
    T = case["rows"]
    x = rng.standard_normal((T, 13))
    decay = np.array([0.9] + [0.7, 0.7, 0.7, 0.99, 0.98, 0.985] + [0.6] * 6)
    k = np.arange(512)
    f = np.fft.rfft(decay[None, :] ** k[:, None], n=T + 512, axis=0)
    y = np.fft.irfft(f * np.fft.rfft(x, n=T + 512, axis=0), n=T + 512, axis=0)[:T]
    return np.ascontiguousarray(40.0 * y + np.array([2e4] + [900.0] * 3 + [0.0] * 3 + [1000.0] * 3 + [0.0] * 3))


def _theta_of(t):
    return torch.tensor(np.stack([t.epsilon, t.sigma, t.lam], axis=-1), dtype=torch.float64)


# ---- what a program has in hand ------------------------------------------------------------------------------

def prepare(case, seed):
    s, rng = _inputs(case, seed)
    kind = case["kind"]
    st = dict(case=case, step=0)
    if kind == "stress":
        small, _ = _inputs(dict(kind="forces", system="reactive", n=1000, density=0.2, eps=1.0), seed)
        st.update(S=System.from_workload(small), rows=_rows(case, rng))
        return st
    if kind == "batch":
        B = Batch(s, seeds=[seed + r for r in range(len(s))])
        B.set_step_form("sums")
        edge = np.zeros((B.n_slots, 4), np.float32)
        for r, x in enumerate(s):
            edge[B.slots(r), :3] = x.L
        tags = np.concatenate([np.arange(B.offsets[r], B.offsets[r] + len(x.pos)) for r, x in enumerate(s)])
        dt, kT = _DYN["batch"]
        st.update(S=B, L=torch.from_numpy(edge).cuda(), tags=torch.from_numpy(tags.astype(np.int64)).cuda(),
                  cfg=B.integrator(dt=dt, kT=kT, gamma=1.0))
        return st
    S = System.from_workload(s)
    st["S"] = S
    st["L"] = torch.tensor(list(S.edges) + [0.0], dtype=torch.float32, device="cuda")
    if kind == "md":
        dt, kT = _DYN[case["system"]]
        st["cfg"] = S.integrator(dt=dt, kT=kT, gamma=1.0, seed=seed)
        return st
    if kind == "rigid":
        dt, kT = _DYN["rigid"]
        st["R"] = RigidBodies(S, s.bodies, s.theta, s.omega)
        st["cfg"] = S.integrator(dt=dt, kT=kT, gamma=1.0, seed=seed, dim=2)
        return st
    if kind == "build":
        return st
    if kind == "grad":
        st["M"] = SwapModel(S)
        x, a, th = _grad_inputs(s, rng)
        st.update(x=x.cuda().requires_grad_(), a=a.cuda(), theta=th.requires_grad_())
        return st
    S.build()
    assert bool((S.rtag == torch.arange(S.N, device="cuda")).all())
    if kind == "hvp":
        V = torch.zeros((case["nvec"], case["n"], 4), dtype=torch.float32)
        V[:, :, :3] = _tangents(case, rng)
        st["V"] = V.cuda()
        S.reserve_hvp_vectors(case["nvec"])
    return st


def _tangents(case, rng):
    return torch.from_numpy(rng.standard_normal((case["nvec"], case["n"], 3)).astype(np.float32))


def _grad_inputs(s, rng):
    """Positions moved a little from those the list was built at, a cotangent of the forces, the parameters."""
    x = torch.from_numpy(_fold(s.pos.astype(np.float64) + rng.uniform(-0.01, 0.01, s.pos.shape), s.L))
    a = torch.from_numpy(rng.standard_normal(s.pos.shape).astype(np.float32))
    return x, a, _theta_of(s.table)


# ---- one pass ------------------------------------------------------------------------------------------------

def _state(S, L, rtag):
    """Unwrapped positions and velocities by tag."""
    x = torch.addcmul(S.pos, S.image.to(torch.float32), L)
    at = rtag.long()
    return x[:, :3][at], S.vel[:, :3][at]


def run(st):
    c, S = st["case"], st["S"]
    kind = c["kind"]
    if kind in ("md", "batch"):
        r = S.run(c["steps"], st["cfg"], step0=st["step"], log_period=c["log"])
        st["step"] += c["steps"]
        rtag = S.rtag if kind == "md" else S.rtag[st["tags"]]
        x, v = _state(S, st["L"], rtag)
        return dict(x=x, v=v, ev=r.ev, bonds=r.bonds)
    if kind == "rigid":
        st["R"].run(c["steps"], st["cfg"], step0=st["step"])
        st["step"] += c["steps"]
        x, v = _state(S, st["L"], S.rtag)
        return dict(x=x, v=v, theta=st["R"].theta, omega=st["R"].omega)
    if kind == "build":
        S.build()
        return dict(tags=S.pos.view(torch.int32)[:, 3], rtag=S.rtag, nn=S.nn, nlist=S.nlist)
    if kind == "frame":
        F, ev = S.compute_forces()
        value, grad = S.soft_bonds(grad=True)
        n = S.bond_count()
        return dict(F=F, ev=ev, soft=value, grad=grad[:, :3], bonds=n)
    if kind == "forces":
        F, ev = S.compute_forces(gather={"triplet": False, "gather": True, "sums": "sums"}[c["path"]])
        return dict(F=F, ev=ev)
    if kind == "hvp":
        return S.hvp_batch(st["V"])[:, :, :3]
    if kind == "grad":
        E = swap_energy(st["M"], st["x"], st["theta"])
        F = swap_forces(st["M"], st["x"], st["theta"])
        gx, gt = torch.autograd.grad(E + (F * st["a"]).sum(), [st["x"], st["theta"]])
        return dict(E=E, F=F, gx=gx, gt=gt)
    return S.stress_autocorrelation(st["rows"], 1.0, c["lags"])


# ---- what a pass cannot do without ---------------------------------------------------------------------------

#: mean list length (with the skin) and mean pairs inside the cutoff per particle
_K = dict(dumbbells=(1.6, 0.9), assembly=(1.4, 0.3), reactive=(5.0, 2.5), unequal=(5.6, 2.8), network=(7.5, 4.5),
          batch=(5.0, 2.5), rigid=(2.0, 0.8))


def work(case):
    kind = case["kind"]
    if kind == "stress":
        return dict(bytes=8.0 * (6 * case["rows"] + case["lags"]), flops=6.0 * case["rows"] * case["lags"])
    if kind == "batch":   # the mean of a log-uniform size
        lo, hi = case["n_lo"], case["n_hi"]
        n = case["replicas"] * (hi - lo) / math.log(hi / lo)
    elif kind == "rigid":
        n = 3.4 * case["bodies"]
    else:
        n = case["n"]
    k, a = _K[case.get("system", kind)]
    pair = 20.0 * k + 60.0 * a
    if kind in ("md", "batch", "rigid"):   # positions, velocities in and out, the list
        return dict(bytes=case["steps"] * n * (68.0 + 4.0 * k), flops=case["steps"] * n * (150.0 + pair))
    if kind == "build":                    # the state in and out, the list out
        return dict(bytes=n * (96.0 + 4.0 + 4.0 + 4.0 * k), flops=n * 27.0 * 10.0)
    if kind == "hvp":
        return dict(bytes=n * (20.0 + 4.0 * k + case["nvec"] * 32.0), flops=n * (30.0 * k + case["nvec"] * a * 60.0))
    if kind == "grad":                     # positions and list in; forces, the HVP and two gradients out
        return dict(bytes=n * (12.0 + 4.0 + 4.0 * k + 12.0 + 12.0 + 12.0), flops=n * 5.0 * pair)
    if kind == "frame":
        return dict(bytes=n * (16.0 + 4.0 + 4.0 * k + 32.0), flops=n * 2.0 * pair)
    return dict(bytes=n * (16.0 + 4.0 + 4.0 * k + 16.0), flops=n * pair)


# ---- the same in 64 bits -------------------------------------------------------------------------------------

def _pairs(x, L, reach):
    """(i, j, x_j - x_i) of every pair i < j nearer than `reach` in the periodic box (float64 positions)."""
    dev, n = x.device, x.shape[0]
    edge = torch.as_tensor(L, dtype=torch.float64, device=dev).expand(3)
    cap = max(8, 2 * round(n ** (1.0 / 3.0)))
    nc = [max(3, min(cap, int(e // reach))) for e in edge.tolist()]
    w = x / edge + 0.5
    w = w - torch.floor(w)
    c = torch.stack([torch.clamp((w[:, d] * nc[d]).long(), max=nc[d] - 1) for d in range(3)], dim=1)
    key = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
    order = torch.argsort(key, stable=True)
    cells = nc[0] * nc[1] * nc[2]
    start = torch.searchsorted(key[order].contiguous(), torch.arange(cells + 1, device=dev))
    most = int((start[1:] - start[:-1]).max())
    off = [(a, b, d) for d in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)]
    got = []
    at = torch.arange(most, device=dev)
    for s in range(0, n, 1 << 17):
        me = torch.arange(s, min(n, s + (1 << 17)), device=dev)
        for a, b, d in off:
            q = torch.remainder(c[me] + torch.tensor([a, b, d], device=dev), torch.tensor(nc, device=dev))
            q = (q[:, 2] * nc[1] + q[:, 1]) * nc[0] + q[:, 0]
            slot = start[q][:, None] + at[None, :]
            ok = slot < start[q + 1][:, None]
            j = order[torch.clamp(slot, max=n - 1)]
            ok &= j > me[:, None]
            i, j = me[:, None].expand_as(j)[ok], j[ok]
            r = x[j] - x[i]
            r = r - edge * torch.round(r / edge)
            near = (r * r).sum(1) < reach * reach
            got.append((i[near], j[near], r[near]))
    return tuple(torch.cat(v) for v in zip(*got))


class _Fp64:
    """Energy, forces and virial of one system in FP64 (pair terms, switching factors, springs)."""

    def __init__(self, s, dev, theta=None):
        self.s, self.dev = s, dev
        t = s.table
        f = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev).reshape(-1)  # noqa: E731
        self.nt = t.kind.shape[0]
        self.kind = torch.as_tensor(t.kind, device=dev).reshape(-1)
        self.n, self.rcut = f(np.where(t.kind == WCA, 6, t.n)), f(t.rcut)
        th = _theta_of(t) if theta is None else theta
        self.eps, self.sigma, self.lam = (th[..., q].to(dev).reshape(-1) for q in range(3))
        rmin2 = (t.sigma * t.sigma) * 2.0 ** (2.0 / np.where(t.kind == WCA, 6, t.n))
        self.rmin2 = f(rmin2)
        self.type = torch.as_tensor(s.types, device=dev).long()
        self.L = torch.as_tensor(s.L, dtype=torch.float64, device=dev).expand(3)
        self.reach = 0.6
        self.ref = None
        if s.bonds is not None:
            b = torch.as_tensor(s.bonds, device=dev).long()[:, 1]
            self.bi = torch.nonzero(b >= 0)[:, 0]
            self.bj = b[self.bi]

    def list(self, x):
        if self.ref is None or float(((x - self.ref).detach() ** 2).sum(1).max()) > (0.5 * self.reach) ** 2:
            self.ref = x.detach().clone()
            self.i, self.j, _ = _pairs(self.ref, self.L, float(self.rcut.max()) + self.reach)

    def terms(self, x):
        """Per active pair: i, j, d, r2, entry, swap and inside masks."""
        self.list(x)
        d = x[self.j] - x[self.i]
        d = d - self.L * torch.round(d / self.L).detach()
        r2 = (d * d).sum(1)
        e = self.type[self.i] * self.nt + self.type[self.j]
        on = (r2 < self.rcut[e] ** 2) & (self.kind[e] != NONE)
        i, j, d, r2, e = self.i[on], self.j[on], d[on], r2[on], e[on]
        return i, j, d, r2, e, self.kind[e] == SWAP, r2 <= self.rmin2[e]

    def energy(self, x):
        """The energy as a differentiable function (for autograd references)."""
        i, j, d, r2, e, sw, inside = self.terms(x)
        q = (self.sigma[e] ** 2 / r2) ** (0.5 * self.n[e])
        phi = 4.0 * self.eps[e] * (q * q - q) + torch.where(sw, 0.0, self.eps[e])
        u = torch.where(inside, torch.ones_like(q), 4.0 * (q - q * q))
        one = torch.ones_like(q)
        w = torch.where(sw, torch.sqrt(torch.where(sw, self.lam[e] * self.eps[e], one)) * u, 0.0 * one)
        S = torch.zeros_like(x[:, 0]).index_add(0, i, w).index_add(0, j, w)
        return phi.sum() + 0.5 * (S * S).sum() - (w * w).sum()

    def forces(self, x):
        """(F, [E, W(6)], per-particle energies, active terms)."""
        i, j, d, r2, e, sw, inside = self.terms(x)
        n, eps = self.n[e], self.eps[e]
        q = (self.sigma[e] ** 2 / r2) ** (0.5 * n)
        phi = 4.0 * eps * (q * q - q) + torch.where(sw, 0.0, eps)
        f = 4.0 * eps * n * (q - 2.0 * q * q) / r2
        root = torch.where(sw, torch.sqrt(self.lam[e] * eps), 0.0)
        w = root * torch.where(inside, torch.ones_like(q), 4.0 * (q - q * q))
        k1 = torch.where(inside, 0.0, root * 4.0 * n * (2.0 * q * q - q) / r2)
        S = torch.zeros_like(x[:, 0]).index_add_(0, i, w).index_add_(0, j, w)
        f = f + k1 * (S[i] + S[j] - 2.0 * w)
        F = torch.zeros_like(x).index_add_(0, i, f[:, None] * d).index_add_(0, j, -f[:, None] * d)
        half = 0.5 * (phi - w * w)
        pe = 0.5 * S * S
        pe = pe.index_add(0, i, half).index_add(0, j, half)
        if self.s.bonds is not None:
            K, R0 = self.s.fene
            b = x[self.bj] - x[self.bi]
            b = b - self.L * torch.round(b / self.L)
            z = 1.0 - (b * b).sum(1) / R0 ** 2
            g = K / z
            F.index_add_(0, self.bi, g[:, None] * b).index_add_(0, self.bj, -g[:, None] * b)
            h = -0.25 * K * R0 ** 2 * torch.log(z)
            pe = pe.index_add(0, self.bi, h).index_add(0, self.bj, h)
            d, f = torch.cat([d, b]), torch.cat([f, g])
        ab = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
        ev = [pe.sum()] + [-(f * d[:, p] * d[:, q_]).sum() for p, q_ in ab]
        return F, torch.stack(ev), pe, (i, j, d, r2, e, sw, inside)


def _normals(seed, tags, step):
    """Three normals per tag and step: Philox4x32-10 words mapped by Box-Muller."""
    m32 = 0xFFFFFFFF
    c = [tags.clone(), torch.full_like(tags, step & m32), torch.full_like(tags, step >> 32), torch.zeros_like(tags)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57     # wraps modulo 2^64: the bits are the product's
        h0, l0, h1, l1 = (p0 >> 32) & m32, p0 & m32, (p1 >> 32) & m32, p1 & m32
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
    u = [(v.to(torch.float64) + 0.5) * 2.0 ** -32 for v in c]
    r0, r1 = torch.sqrt(-2.0 * torch.log(u[0])), torch.sqrt(-2.0 * torch.log(u[2]))
    a0, a1 = 2.0 * math.pi * u[1], 2.0 * math.pi * u[3]
    return torch.stack([r0 * torch.cos(a0), r0 * torch.sin(a0), r1 * torch.cos(a1)], dim=1)


def _md64(s, dt, kT, seed, steps, log, dev):
    """(x unwrapped, v, log rows) after BAOAB steps from the start, gamma 1, unit masses."""
    E = _Fp64(s, dev)
    x = torch.as_tensor(s.pos, dtype=torch.float64, device=dev)
    v = torch.as_tensor(s.vel, dtype=torch.float64, device=dev)
    tags = torch.arange(len(s.pos), device=dev)
    c1 = math.exp(-dt)
    c2 = math.sqrt((1.0 - c1 * c1) * kT)
    ab = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
    rows = []

    def row(ev, v):
        rows.append(torch.cat([ev, torch.stack([(v[:, p] * v[:, q]).sum() for p, q in ab])]))

    F, ev, _, _ = E.forces(x)
    for k in range(steps):
        if log and k % log == 0:
            row(ev, v)
        v = v + 0.5 * dt * F
        x = x + 0.5 * dt * v
        v = c1 * v + c2 * _normals(seed, tags, k)
        x = x + 0.5 * dt * v
        F, ev, _, _ = E.forces(x)
        v = v + 0.5 * dt * F
    row(ev, v)
    return x, v, torch.stack(rows)


def _rigid64(s, dt, kT, seed, steps, dev):
    E = _Fp64(s, dev)
    f = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)  # noqa: E731
    B = len(s.theta)
    x, v, th, w, I = f(s.pos), f(s.vel), f(s.theta), f(s.omega), f(s.bodies["inertia"])
    own = torch.as_tensor(np.repeat(np.arange(B), np.diff(s.bodies["first"])), device=dev)
    o = f(s.bodies["offset"])
    x0, L = x.clone(), E.L
    c1 = math.exp(-dt)
    c2 = math.sqrt((1.0 - c1 * c1) * kT)
    tags = torch.arange(B, device=dev)
    cen, vc = x[:B, :2].clone(), v[:B, :2].clone()

    def arm(th):
        c, n = torch.cos(th)[own], torch.sin(th)[own]
        return torch.stack([c * o[:, 0] - n * o[:, 1], n * o[:, 0] + c * o[:, 1]], dim=1)

    def load(x, d):
        F = E.forces(x)[0][:, :2]
        t = d[:, 0] * F[B:, 1] - d[:, 1] * F[B:, 0]
        return F[:B].clone().index_add_(0, own, F[B:]), torch.zeros_like(th).index_add_(0, own, t)

    d = x[B:, :2] - cen[own]
    F, T = load(x, d - L[:2] * torch.round(d / L[:2]))
    for k in range(steps):
        vc, w = vc + 0.5 * dt * F, w + 0.5 * dt * T / I
        z = _normals(seed, tags, k)
        cen, th = cen + 0.5 * dt * vc, th + 0.5 * dt * w
        vc, w = c1 * vc + c2 * z[:, :2], c1 * w + c2 * z[:, 2] / torch.sqrt(I)
        cen, th = cen + 0.5 * dt * vc, th + 0.5 * dt * w
        d = arm(th)
        x = torch.cat([torch.cat([cen, cen[own] + d]), x0[:, 2:]], dim=1)
        F, T = load(x, d)
        vc, w = vc + 0.5 * dt * F, w + 0.5 * dt * T / I
    d = arm(th)
    turn = torch.stack([-w[own] * d[:, 1], w[own] * d[:, 0]], dim=1)
    v = torch.cat([torch.cat([vc, vc[own] + turn]), 0.0 * v[:, 2:]], dim=1)
    move = x - x0
    th = th - 2.0 * math.pi * torch.floor(th / (2.0 * math.pi) + 0.5)
    return dict(x=x0 + move - L * torch.round(move / L), v=v, theta=th, omega=w)


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    s, rng = _inputs(case, seed)
    kind = case["kind"]
    if kind == "build":
        return None                       # whole numbers only
    if kind == "stress":
        rows = _rows(case, rng)
        y = rows[:, 4:7] + rows[:, 10:13]
        T, m = len(y), 1 << (2 * len(y)).bit_length()
        f = np.fft.rfft(y, n=m, axis=0)
        c = np.fft.irfft(f * np.conj(f), n=m, axis=0)[:case["lags"] + 1].sum(axis=1)
        V = float(np.float32((1000 / 0.2) ** (1.0 / 3.0))) ** 3
        return c / (3.0 * (T - np.arange(case["lags"] + 1.0))) / V
    if kind == "md":
        dt, kT = _DYN[case["system"]]
        x, v, rows = _md64(s, dt, kT, seed, case["steps"], case["log"], dev)
        return dict(x=x, v=v, ev=rows, bonds=None)
    if kind == "batch":
        dt, kT = _DYN["batch"]
        got = [_md64(q, dt, kT, seed + r, case["steps"], case["log"], dev) for r, q in enumerate(s)]
        return dict(x=torch.cat([g[0] for g in got]), v=torch.cat([g[1] for g in got]),
                    ev=torch.stack([g[2] for g in got], dim=1), bonds=None)
    if kind == "rigid":
        dt, kT = _DYN["rigid"]
        return _rigid64(s, dt, kT, seed, case["steps"], dev)
    if kind == "grad":
        x, a, th = _grad_inputs(s, rng)
        x = x.to(dev).to(torch.float64).requires_grad_()
        th.requires_grad_()
        upper = torch.triu(torch.ones(th.shape[:2], dtype=torch.bool))[..., None]
        E = _Fp64(s, dev, torch.where(upper, th, th.transpose(0, 1))).energy(x)
        (g,) = torch.autograd.grad(E, x, create_graph=True)
        gx, gt = torch.autograd.grad(E - (g * a.to(dev)).sum(), [x, th])
        return dict(E=E.detach(), F=-g.detach(), gx=gx, gt=gt)
    E = _Fp64(s, dev)
    x = torch.as_tensor(s.pos, dtype=torch.float64, device=dev)
    if kind == "hvp":
        V = _tangents(case, rng).to(dev).to(torch.float64)
        x.requires_grad_()
        (g,) = torch.autograd.grad(E.energy(x), x, create_graph=True)
        return torch.stack([torch.autograd.grad(g, x, t, retain_graph=True)[0] for t in V])
    F, ev, pe, (i, j, d, r2, e, sw, inside) = E.forces(x)
    F = torch.cat([F, pe[:, None]], dim=1)
    if kind == "forces":
        return dict(F=F, ev=ev)
    i, j, d, r2, e, inside = i[sw], j[sw], d[sw], r2[sw], e[sw], inside[sw]
    n = E.n[e]
    q = (E.sigma[e] ** 2 / r2) ** (0.5 * n)
    u = torch.where(inside, torch.ones_like(q), 4.0 * (q - q * q))
    k1 = torch.where(inside, 0.0, 4.0 * n * (2.0 * q * q - q) / r2)[:, None] * d
    G = torch.zeros_like(x).index_add_(0, i, -k1).index_add_(0, j, k1)
    return dict(F=F, ev=ev, soft=u.sum().reshape(1), grad=G, bonds=None)
