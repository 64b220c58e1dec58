"""The work whose speed is tracked: hPF-MD calls as a simulation program makes them.

Every case is one of seven kinds of call:
  density  counts of cell-sorted beads that have moved since their sort, through the entry
           point that allocates nothing (a serving loop that watches a composition)
  field    density, potential and gradient of a frame whose beads are in no order (analysis
           of a stored trajectory)
  start    sort, forces and energies of a freshly loaded system (HpfState.start)
  run      one sort interval of fused steps, launched one by one, from a loaded checkpoint
           (x_n, v_n-1/2); optionally with a field-update interval and the thermostat
  graph    two sort intervals of fused steps replayed from a HIP graph
  steps    whole steps from the separate calls (angles, the staggered stencil)
  sweep    a batch of replicas stepped together over one sort interval

Systems are the repository's: random-walk chains of bond step 0.97 at bead density 3,
diblocks, blends, an amphiphile in solvent, lipids in water, and three-armed stars (a bond
table of three rows with a bond length).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1310_2041_amd import engine, hpf

DT, K_BOND, STEP = 0.03, 100.0, 0.97


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest call: the 20,000-bead diblock's density on 20^3 points, latency only
        dict(name="density_20k", kind="density", arch="diblock", beads=20000, mx=20, my=20, mz=20, halo=1),
        # analysis of a stored 1M-bead frame on a 64^3 mesh, beads in chain order
        dict(name="field_1m", kind="field", arch="diblock", beads=1000000, mx=64, my=64, mz=64),
        # a freshly loaded 3M-bead three-species system on a ragged mesh
        dict(name="start_3m", kind="start", arch="amphiphile", beads=3000000, mx=101, my=84, mz=91, halo=1),
        # the smallest simulation: 20,000 beads, replayed, where launches are everything
        dict(name="graph_20k", kind="graph", arch="diblock", beads=20000, mx=20, my=20, mz=20, halo=1, steps=20),
        # the 1M-bead diblock melt of the benchmark, replayed
        dict(name="graph_1m", kind="graph", arch="diblock", beads=1000000, mx=64, my=64, mz=64, halo=2, steps=30),
        # the 10M-bead blend of the benchmark, energies every step, a sort every 30
        dict(name="run_10m", kind="run", arch="blend", beads=10000000, mx=128, my=128, mz=128, halo=2, steps=30,
             field_every=1, rate=0.0),
        # MD-SCF use: the field rebuilt every 10 steps under the thermostat, on a ragged mesh
        dict(name="run_nvt_3m", kind="run", arch="blend", beads=3300000, mx=97, my=90, mz=101, halo=1, steps=20,
             field_every=10, rate=5.0),
        # the large amphiphile in solvent: three species, thousands of bricks, incremental re-sort
        dict(name="run_42m", kind="run", arch="amphiphile", beads=42000000, mx=192, my=192, mz=192, halo=2, steps=10,
             field_every=1, rate=0.0),
        # branched molecules: three bond rows and a bond length
        dict(name="run_star_600k", kind="run", arch="star", beads=600000, mx=58, my=61, mz=55, halo=1, steps=30,
             field_every=1, rate=0.0),
        # lipids in water: five species, branched bonds, angles
        dict(name="steps_lipid_1m", kind="steps", arch="lipid", beads=1200000, mx=74, my=74, mz=74, steps=20,
             stencil="centred"),
        # the paper-literal force stencil on the 20-bead diblock
        dict(name="steps_stag_300k", kind="steps", arch="diblock", beads=300000, mx=47, my=47, mz=47, steps=20,
             stencil="staggered"),
        # the phase-diagram sweep: 64 uneven replicas
        dict(name="sweep_64", kind="sweep", arch="diblock", replicas=64, beads=8000, most=400000, halo=1, steps=10),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def _mesh(rng, beads, fine):
    """A ragged mesh of about beads / fine cells, every edge at least 14."""
    e = (beads / fine) ** (1.0 / 3.0)
    m = [max(14, int(round(e * rng.uniform(0.85, 1.18)))) for _ in range(3)]
    return dict(mx=m[0], my=m[1], mz=m[2])


def draw(rng):
    kind = rng.choice(["density", "field", "start", "graph", "run", "run", "steps", "sweep"])
    fine = rng.uniform(2.5, 6.0)              # beads per cell
    halo = rng.choice([1, 2])
    if kind == "density":
        n = _log(rng, 6000, 700000)
        return dict(kind=kind, arch=rng.choice(["diblock", "lipid"]), beads=n, halo=1, **_mesh(rng, n, 5.0))
    if kind == "field":
        n = _log(rng, 20000, 4000000)
        return dict(kind=kind, arch=rng.choice(["diblock", "amphiphile"]), beads=n, **_mesh(rng, n, fine))
    if kind == "start":
        n = _log(rng, 50000, 12000000)
        return dict(kind=kind, arch=rng.choice(["amphiphile", "star", "blend"]), beads=n, halo=halo,
                    **_mesh(rng, n, fine))
    if kind == "graph":
        n = _log(rng, 9000, 2000000)
        return dict(kind=kind, arch=rng.choice(["diblock", "blend", "star"]), beads=n, halo=halo,
                    steps=rng.choice([20, 30]), **_mesh(rng, n, fine))
    if kind == "run":
        n = _log(rng, 200000, 30000000)
        nvt = rng.random() < 0.4
        return dict(kind=kind, arch=rng.choice(["diblock", "blend", "amphiphile", "star"]), beads=n, halo=halo,
                    steps=10 if n > 12000000 else rng.choice([20, 30]), field_every=rng.choice([5, 10]) if nvt else 1,
                    rate=5.0 if nvt else 0.0, **_mesh(rng, n, fine))
    if kind == "steps":
        n = _log(rng, 60000, 1500000)
        stag = rng.random() < 0.35
        return dict(kind=kind, arch="diblock" if stag else "lipid", beads=n, steps=rng.choice([10, 20]),
                    stencil="staggered" if stag else "centred", **_mesh(rng, n, 3.0))
    r = rng.randint(6, 72)
    return dict(kind=kind, arch="diblock", replicas=r, beads=rng.choice([8000, 12000]), most=_log(rng, 30000, 400000),
                halo=halo, steps=10)


# ---------------------------------------------------------------- systems
# A molecule: parent of each bead (a random walk along it), bead types, bonded pairs, angle
# triplets (end, middle, end, type).

def _chain(n):
    return [-1] + list(range(n - 1)), [(i, i + 1) for i in range(n - 1)]


_LIPID_PAIRS = [(0, 1), (1, 2), (2, 3), (2, 4), (4, 5), (5, 6), (6, 7), (3, 8), (8, 9), (9, 10), (10, 11)]
_LIPID_ANGLES = [(1, 2, 3, 0), (1, 2, 4, 0), (2, 4, 5, 1), (4, 5, 6, 1), (5, 6, 7, 1), (2, 3, 8, 1), (3, 8, 9, 1),
                 (8, 9, 10, 1), (9, 10, 11, 1)]


def _molecule(arch):
    """(parents, types, pairs, angles, K, chi, r0, share of the beads in molecules)"""
    if arch == "diblock":
        p, b = _chain(20)
        return p, [0] * 10 + [1] * 10, b, [], 2, {(0, 1): 1.0}, 0.0, 1.0
    if arch == "blend":                       # half of the 50-bead chains are of each type
        p, b = _chain(50)
        return p, None, b, [], 2, {(0, 1): 0.5}, 0.0, 1.0
    if arch == "amphiphile":
        p, b = _chain(12)
        return p, [0] * 4 + [1] * 8, b, [], 3, {(0, 1): 1.0, (0, 2): 1.5, (1, 2): -0.5}, 0.0, 0.2
    if arch == "star":                        # a centre and three arms of four
        p = [-1, 0, 1, 2, 3, 0, 5, 6, 7, 0, 9, 10, 11]
        return p, [0] + [0, 0, 1, 1] * 3, [(p[i], i) for i in range(1, 13)], [], 2, {(0, 1): 1.0}, 0.5, 1.0
    p = [-1, 0, 1, 2, 2, 4, 5, 6, 3, 8, 9, 10]
    chi = {(0, 1): 0.5, (0, 2): 1.5, (1, 2): 1.5, (0, 3): 5.0, (1, 3): 5.0, (2, 3): 3.0, (3, 4): 7.0, (2, 4): 3.0}
    return p, [0, 1, 2, 2] + [3] * 8, _LIPID_PAIRS, _LIPID_ANGLES, 5, chi, 0.5, 0.4


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _system(arch, beads, M, seed):
    """A system of about `beads` beads (whole molecules, then single solvent beads)."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    parents, types, pairs, angles, K, chi, r0, share = _molecule(arch)
    per = len(parents)
    nmol = max(1, int(beads * share) // per)
    N = nmol * per if share == 1.0 else max(beads, nmol * per)
    # the box: bead density 3, its edges in the mesh's proportions
    h = (N / 3.0 / (M[0] * M[1] * M[2])) ** (1.0 / 3.0)
    L = [float(np.float32(h * m)) for m in M]
    Lt = torch.tensor(L, dtype=torch.float64, device=dev)
    pos = torch.empty((nmol, per, 3), dtype=torch.float64, device=dev)
    walk = torch.randn((nmol, per, 3), generator=gen, dtype=torch.float64, device=dev)
    walk *= STEP / walk.norm(dim=2, keepdim=True)
    pos[:, 0] = torch.rand((nmol, 3), generator=gen, dtype=torch.float64, device=dev) * Lt
    for b in range(1, per):
        pos[:, b] = pos[:, parents[b]] + walk[:, b]
    T = torch.full((N,), K - 1, dtype=torch.uint8, device=dev)
    if types is None:
        T[:nmol * per] = (torch.arange(nmol, device=dev) * 2 >= nmol).to(torch.uint8).repeat_interleave(per)
    else:
        T[:nmol * per] = torch.tensor(types, dtype=torch.uint8, device=dev).repeat(nmol)
    free = torch.rand((N - nmol * per, 3), generator=gen, dtype=torch.float64, device=dev) * Lt
    R = torch.remainder(torch.cat([pos.reshape(-1, 3), free]), Lt).float()
    R = torch.where(R >= Lt.float(), torch.zeros_like(R), R)
    V = torch.randn((N, 3), generator=gen, dtype=torch.float32, device=dev)
    V -= V.mean(dim=0, keepdim=True)
    # bond table [D, N] and angle table [3A, N] from the molecule's
    nbr = [[] for _ in range(per)]
    for i, j in pairs:
        nbr[i].append(j)
        nbr[j].append(i)
    base = (torch.arange(nmol, device=dev) * per).view(-1, 1)

    def table(rows, fill):
        out = torch.full((len(rows), N), fill, dtype=torch.int32, device=dev)
        for r, row in enumerate(rows):
            t = torch.tensor(row, device=dev)
            out[r, :nmol * per] = torch.where(t >= 0, t + base, t).reshape(-1).to(torch.int32)
        return out

    D = max(len(v) for v in nbr)
    bonds = table([[v[d] if d < len(v) else -1 for v in nbr] for d in range(D)], -1)
    ang = None
    if angles:
        slots = [[] for _ in range(per)]
        for i, j, k, t in angles:
            slots[j].append((i, k, 1 + 2 * t))
            slots[i].append((j, k, 2 * t))
            slots[k].append((j, i, 2 * t))
        A = max(len(v) for v in slots)
        ang = torch.empty((3 * A, N), dtype=torch.int32, device=dev)
        ang[0::3] = table([[v[a][0] if a < len(v) else -1 for v in slots] for a in range(A)], -1)
        ang[1::3] = table([[v[a][1] if a < len(v) else -1 for v in slots] for a in range(A)], -1)
        ang[2::3] = 0
        for a in range(A):
            code = torch.tensor([v[a][2] if a < len(v) else 0 for v in slots], dtype=torch.int32, device=dev)
            ang[3 * a + 2, :nmol * per] = code.repeat(nmol)
    x = np.zeros((K, K))
    for (a, b), v in chi.items():
        x[a, b] = x[b, a] = v
    return SimpleNamespace(R=R, V=V, T=T, tag=torch.arange(N, dtype=torch.int32, device=dev), bonds=bonds, L=tuple(L),
                           M=tuple(M), K=K, kT=1.0, inv_kappa=10.0, chi=x, k_bond=K_BOND, r0=r0, dt=DT, N=N,
                           angles=ang, angle_k=(12.0, 12.0) if angles else (),
                           angle_theta0=(2.0 * math.pi / 3.0, math.pi) if angles else (),
                           angle_form=(0, 1) if angles else ())


def _one(case, seed):
    return _system(case["arch"], case["beads"], (case["mx"], case["my"], case["mz"]), seed)


def _replicas(case, seed):
    """Replicas of beads..most beads, spread over the logarithm, in no order; chi from 0 to 2;
    cells of about one length unit."""
    n = case["replicas"]
    out = []
    for r in range(n):
        at = ((r * 7) % n) / max(1, n - 1) if n % 7 else r / max(1, n - 1)
        beads = int(case["beads"] * (case["most"] / case["beads"]) ** at)
        m = max(14, math.ceil((beads / 3.0) ** (1.0 / 3.0)))
        s = _system(case["arch"], beads, (m,) * 3, seed * 1000 + r)
        s.chi = np.array([[0.0, 2.0 * r / max(1, n - 1)], [2.0 * r / max(1, n - 1), 0.0]])
        out.append(s)
    return out


def _host(s):
    """The system as a program loads it: arrays in host memory."""
    d = dict(vars(s))
    for k in ("R", "V", "T", "tag", "bonds", "angles"):
        if d[k] is not None:
            d[k] = d[k].cpu().numpy()
    return SimpleNamespace(**d)


def _brick(s, halo):
    """Sort brick edge: 16 cells where the mesh has 512 of them and the box fits, else 8."""
    P = 17 + 2 * halo
    nb = math.prod(-(-m // 16) for m in s.M)
    return 16 if nb >= 512 and s.K * P ** 3 * 8 <= 160 * 1024 and min(s.M) >= P else 8


# ---------------------------------------------------------- prepare and run

def prepare(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        b = engine.BatchState([_host(s) for s in _replicas(case, seed)], sort_every=case["steps"], halo=case["halo"])
        b.start()
        return SimpleNamespace(kind=kind, case=case, batch=b)
    s = _one(case, seed)
    if kind == "field":
        mesh = hpf.hpf_mesh_make(s.L, s.M, s.N)
        nm = math.prod(s.M)
        z = dict(device=s.R.device)
        return SimpleNamespace(kind=kind, case=case, R=s.R, T=s.T, K=s.K, mesh=mesh,
                               field=hpf.make_field(s.K, s.kT, s.inv_kappa, s.chi),
                               counts=torch.zeros((s.K, nm), dtype=torch.int64, **z),
                               V=torch.empty((s.K, nm), dtype=torch.float32, **z),
                               G=torch.empty((s.K, nm, 3), dtype=torch.float32, **z),
                               part=torch.zeros((1, hpf.HPF_NPART), dtype=torch.float64, **z),
                               W=torch.zeros(1, dtype=torch.float64, **z))
    more = dict(halo=case["halo"]) if "halo" in case else {}
    if kind in ("run", "start"):
        more["sort_brick"] = _brick(s, case["halo"])
    if kind == "run":
        more["field_every"] = case["field_every"]
    if kind == "steps":
        more["stencil"] = case["stencil"]
    st = engine.HpfState.from_system(_host(s), **more)
    state = SimpleNamespace(kind=kind, case=case, st=st)
    if kind == "density":
        # the beads have moved a third of a cell since their sort
        st.sort()
        st.R.copy_(_moved(st.R, st.tag, s, seed))
    elif kind == "run" and case["field_every"] > 1:
        # the first steps gather from the start's field
        st.set_thermostat(case["rate"], seed=int(seed))
        st.start(sort=True)
        st.prime()
    elif kind == "steps":
        st.start(sort=True)
    elif kind == "graph":
        st.start(sort=True)
        st.prime()
        state.graph = engine.Graph(lambda: [st.step_fused(report=True, sort=k % case["steps"] == 0)
                                            for k in range(2 * case["steps"])])
    return state


def _moved(R, tag, s, seed):
    gen = torch.Generator(device=R.device)
    gen.manual_seed(int(seed) + 1)
    L = torch.tensor(s.L, dtype=torch.float64, device=R.device)
    h = L / torch.tensor(s.M, dtype=torch.float64, device=R.device)
    d = torch.randn((s.N, 3), generator=gen, dtype=torch.float64, device=R.device)
    x = torch.remainder(R.double() + 0.33 * h * d[tag.long()], L).float()
    return torch.where(x >= L.float(), torch.zeros_like(x), x)


def _frame(a, tag):
    """Rows in the beads' original order, as a trajectory writer stores them."""
    out = torch.empty_like(a)
    out[tag.long()] = a
    return out


def run(state):
    case = state.case
    if state.kind == "density":
        st = state.st
        hpf.hpf_density_scatter_cells_static(st.R, st.T, st.mesh, st.K, st.cell_start, st.B, st.halo, st.counts)
        return st.counts
    if state.kind == "field":
        s = state
        hpf.hpf_density_scatter(s.R, s.T, s.mesh, s.K, s.counts)
        hpf.hpf_field_potential(s.counts, s.mesh, s.field, s.V, s.part)
        hpf.hpf_field_gradient(s.V, s.mesh, s.K, s.G)
        hpf.hpf_reduce_partials(s.part, 1, s.W)
        return dict(V=s.V, G=s.G, W=s.W)
    if state.kind == "sweep":
        b = state.batch
        b.step(case["steps"], report_last=True)
        at = hpf.hpf_batch_current(b.handle)
        R, V, tag = (next(t for t in getattr(b, n) if t.data_ptr() == at[n]) for n in ("R", "Vel", "tag"))
        return dict(energies=b.energies(), R=_frame(R, tag), Vel=_frame(V, tag))
    st = state.st
    if state.kind == "start":
        st.start(sort=True)
        return dict(F=st.F, tag=st.tag, energy=st.energy)
    if state.kind == "graph":
        state.graph.launch(torch.cuda.current_stream())
        return dict(R=_frame(st.R, st.tag), Vel=_frame(st.Vel, st.tag), energy=st.energy)
    if state.kind == "run":
        for k in range(case["steps"]):
            st.step_fused(report=True, sort=k == 0)
        if case["field_every"] > 1:
            return dict(R=_frame(st.R, st.tag), Vel=_frame(st.Vel, st.tag), energy=st.energy)
        return dict(R=st.R, Vel=st.Vel, tag=st.tag, energy=st.energy)
    n = case["steps"]
    for k in range(n):
        st.step(report=k == n - 1, sort=k == 0)
    return dict(R=_frame(st.R, st.tag), Vel=_frame(st.Vel, st.tag), F=_frame(st.F, st.tag), energy=st.energy)


# ------------------------------------------------------------------- work

def work(case):
    """Per step the bead rows (x, v read and written, types, bond and angle slots) and the mesh
    (counts and V written and read once); a call of one part only its own."""
    if case["kind"] == "sweep":
        n = case["replicas"]
        beads = [int(case["beads"] * (case["most"] / case["beads"]) ** (r / max(1, n - 1))) for r in range(n)]
        nm = sum(max(14, math.ceil((b / 3.0) ** (1.0 / 3.0))) ** 3 for b in beads)
        N, K, D, A = sum(beads), 2, 2, 0
    else:
        N, nm = case["beads"], case["mx"] * case["my"] * case["mz"]
        K = {"amphiphile": 3, "lipid": 5}.get(case["arch"], 2)
        D = {"star": 3, "lipid": 3}.get(case["arch"], 2)
        A = 5 if case["arch"] == "lipid" and case["kind"] == "steps" else 0
    if case["kind"] == "density":
        return {"bytes": 13 * N + 8 * K * nm, "flops": 40 * N}
    if case["kind"] == "field":
        return {"bytes": 13 * N + 16 * K * nm, "flops": 40 * N + 20 * K * nm}
    if case["kind"] == "start":
        # bead rows, tags and bond rows read and written by the sort, forces written
        return {"bytes": (2 * (29 + 4 * D) + 12) * N + 24 * K * nm, "flops": 200 * N + 20 * K * nm}
    n = case["steps"] * (2 if case["kind"] == "graph" else 1)
    rebuilt = n // case.get("field_every", 1)
    return {"bytes": n * (49 + 4 * D + 12 * A) * N + rebuilt * 24 * K * nm,
            "flops": n * (200 + 60 * A) * N + rebuilt * 20 * K * nm}


# ------------------------------------------------------------------ exact
# The method in 64 bits, from its definitions; cells and the 16-bit weights are decided in
# single precision as the method defines them. Rows are kept in the original bead order.

class _Exact:
    def __init__(self, s, stencil="centred"):
        self.s, self.stencil = s, stencil
        dev = s.R.device
        f64 = dict(dtype=torch.float64, device=dev)
        self.x, self.v = s.R.double(), s.V.double()
        self.T = s.T.long()
        self.L = torch.tensor(s.L, **f64)
        self.scale32 = torch.tensor([float(np.float32(m / l)) for m, l in zip(s.M, s.L)], dtype=torch.float32,
                                    device=dev)
        self.scale = self.scale32.double()
        self.M = torch.tensor(s.M, device=dev)
        self.nm = math.prod(s.M)
        self.A = torch.tensor(s.kT * s.chi, **f64)
        self.dt = float(np.float32(s.dt))
        self.e = dict(W=0.0, EB=0.0, EA=0.0)

    def cells(self):
        u = self.x.float() * self.scale32
        fl = torch.floor(u)
        q = torch.floor((u - fl) * 65536.0).long()
        return torch.remainder(fl.long(), self.M), q

    def corners(self, c, q):
        c1 = torch.remainder(c + 1, self.M)
        for a in range(8):
            d = [(a >> k) & 1 for k in range(3)]
            i = [(c1 if d[k] else c)[:, k] for k in range(3)]
            w = [(q if d[k] else 65536 - q)[:, k] for k in range(3)]
            yield self.T * self.nm + (i[2] * self.s.M[1] + i[1]) * self.s.M[0] + i[0], w[0] * w[1] * w[2]

    def counts(self):
        n = torch.zeros(self.s.K * self.nm, dtype=torch.int64, device=self.x.device)
        for i, w in self.corners(*self.cells()):
            n.index_add_(0, i, w)
        return n

    def field(self):
        s = self.s
        rho = s.N / self.nm
        phi = self.counts().double().view(s.K, self.nm) / (2.0 ** 48 * rho)
        off = phi.sum(0) - 1.0
        mix = self.A @ phi
        self.e["W"] = float(rho * (0.5 * (phi * mix).sum() + 0.5 * s.inv_kappa * off.square().sum()))
        self.V = mix + s.inv_kappa * off
        V = self.V.view(s.K, s.M[2], s.M[1], s.M[0])
        self.G = torch.stack([0.5 * self.scale[d] * (torch.roll(V, -1, 3 - d) - torch.roll(V, 1, 3 - d))
                              for d in range(3)], dim=-1).view(s.K * self.nm, 3)

    def field_force(self):
        c, q = self.cells()
        if self.stencil == "centred":
            F = torch.zeros_like(self.x)
            for i, w in self.corners(c, q):
                F -= (w.double() / 2.0 ** 48).view(-1, 1) * self.G[i]
            return F
        up = q >= 32768
        n = torch.remainder(c + up.long(), self.M)
        delta = (q - 65536 * up.long()).double() / 65536.0
        V = self.V.view(-1)

        def at(i):
            return V[self.T * self.nm + (i[:, 2] * self.s.M[1] + i[:, 1]) * self.s.M[0] + i[:, 0]]

        F = torch.empty_like(self.x)
        for d in range(3):
            e = torch.zeros(3, dtype=torch.int64, device=n.device)
            e[d] = 1
            back = at(n) - at(torch.remainder(n - e, self.M))
            fore = at(torch.remainder(n + e, self.M)) - at(n)
            F[:, d] = -self.scale[d] * ((0.5 - delta[:, d]) * back + (0.5 + delta[:, d]) * fore)
        return F

    def image(self, d):
        return d - self.L * torch.round(d / self.L)

    def bonded(self):
        s = self.s
        F = torch.zeros_like(self.x)
        k, r0 = float(np.float32(s.k_bond)), float(np.float32(s.r0))
        eb = 0.0
        for row in s.bonds:
            has = row >= 0
            d = self.image(self.x[row.long().clamp(min=0)] - self.x)
            r = d.norm(dim=1)
            eb += float((0.5 * k * (r - r0).square())[has].sum())
            coef = 2.0 * k * (1.0 - r0 / r) if r0 else torch.full_like(r, 2.0 * k)
            F += torch.where(has & (r > 0 if r0 else has), coef, torch.zeros_like(r)).nan_to_num().view(-1, 1) * d
        self.e["EB"] = eb
        if s.angles is None:
            return F
        ak, th0 = (torch.tensor([float(np.float32(v)) for v in t], dtype=torch.float64, device=F.device)
                   for t in (s.angle_k, s.angle_theta0))
        ea = 0.0
        for a in range(s.angles.shape[0] // 3):
            p, o, code = (s.angles[3 * a + j].long() for j in range(3))
            i = torch.nonzero(p >= 0).view(-1)
            p, o, code = p[i], o[i], code[i]
            mid = (code & 1) == 1
            t = code >> 1
            xm = torch.where(mid.view(-1, 1), self.x[i], self.x[p])
            u = self.image(torch.where(mid.view(-1, 1), self.x[p], self.x[i]) - xm)
            w = self.image(self.x[o] - xm)
            nu, nw = u.norm(dim=1, keepdim=True), w.norm(dim=1, keepdim=True)
            dot, cr = (u * w).sum(1), torch.linalg.cross(u, w).norm(dim=1)
            c = dot / (nu * nw).view(-1)
            th = torch.atan2(cr, dot) - th0[t]
            dc = c - torch.cos(th0[t])
            harm = t == 0                                          # type 0 harmonic in theta, 1 in its cosine
            U = ak[t] * torch.where(harm, th, dc).square()
            dU = torch.where(harm, -2.0 * ak[t] * th / (cr / (nu * nw).view(-1)).clamp(min=1e-3), 2.0 * ak[t] * dc)
            g1 = (w / nw - c.view(-1, 1) * u / nu) / nu
            g2 = (u / nu - c.view(-1, 1) * w / nw) / nw
            F.index_add_(0, i, -dU.view(-1, 1) * torch.where(mid.view(-1, 1), -(g1 + g2), g1))
            ea += float(U.sum()) / 3.0
        self.e["EA"] = ea
        return F

    def force(self, rebuild=True):
        if rebuild:
            self.field()
        return self.field_force() + self.bonded()

    def drift(self):
        self.x = torch.remainder(self.x + self.dt * self.v, self.L)

    def collide(self, rate, seed, level):
        """Andersen collisions of one time level: Philox4x32-10 on (tag, level)."""
        m32 = 0xffffffff

        def philox(last):
            N = self.s.N
            c = [torch.arange(N, device=self.x.device), torch.full((N,), level, device=self.x.device),
                 torch.zeros(N, dtype=torch.int64, device=self.x.device),
                 torch.full((N,), last, device=self.x.device)]
            k0, k1 = seed & m32, seed >> 32
            for _ in range(10):
                a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57        # wraps to the same 64 bits
                c = [((b >> 32) & m32) ^ c[1] ^ k0, b & m32, ((a >> 32) & m32) ^ c[3] ^ k1, a & m32]
                k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
            return c

        r = philox(0)
        r4 = philox(1)[0]
        p = float(np.float32(rate * self.s.dt))
        hit = (r[0] >> 8) < int(p * 16777216.0)
        rad1 = torch.sqrt(-2.0 * torch.log(((r[1] >> 8) + 1).double() * 2.0 ** -24))
        rad2 = torch.sqrt(-2.0 * torch.log(((r[3] >> 8) + 1).double() * 2.0 ** -24))
        a1, a2 = (2.0 * math.pi * (t >> 8).double() * 2.0 ** -24 for t in (r[2], r4))
        g = torch.stack([rad1 * torch.cos(a1), rad1 * torch.sin(a1), rad2 * torch.cos(a2)], dim=1)
        self.v = torch.where(hit.view(-1, 1), math.sqrt(self.s.kT) * g, self.v)

    def energy(self):
        v = self.v
        ke = 0.5 * float(v.square().sum())
        return torch.tensor([self.e["W"], self.e["EB"], ke, *v.sum(0).tolist(), self.e["EA"], 0.0],
                            dtype=torch.float64)

    def fused(self, n, case=None, seed=0):
        """n steps (x, v half a step behind) -> the same one step on; the energies of the last."""
        every, rate = (case["field_every"], case["rate"]) if case else (1, 0.0)
        for k in range(n):
            # force evaluation k + 1 (evaluation 0 was the start's)
            F = self.force(rebuild=(k + 1) % every == 0)
            self.v = self.v + 0.5 * self.dt * F
            if rate > 0.0:
                self.collide(rate, seed, k + 1)
            e = self.energy()
            self.v = self.v + 0.5 * self.dt * F
            self.drift()
        return e


def exact(case, seed):
    kind = case["kind"]
    n = case.get("steps", 1) * (2 if kind == "graph" else 1)
    if kind != "sweep" and case["beads"] * n > 500000000:
        return None                                    # over 20 seconds
    if kind == "sweep":
        es, xs, vs = [], [], []
        for s in _replicas(case, seed):
            E = _Exact(s)
            E.v = E.v + 0.5 * E.dt * E.force()
            E.drift()
            e = E.fused(n)
            es.append(torch.stack([e[2], e[1], e[0], e[0] + e[1] + e[2], e[3], e[4], e[5], torch.zeros_like(e[0])]))
            xs.append(E.x)
            vs.append(E.v)
        return dict(energies=torch.stack(es).numpy(), R=torch.cat(xs), Vel=torch.cat(vs))
    s = _one(case, seed)
    E = _Exact(s, case.get("stencil", "centred"))
    if kind == "field":
        E.field()
        return dict(V=E.V, G=E.G.view(s.K, E.nm, 3), W=torch.tensor([E.e["W"]], dtype=torch.float64))
    if kind in ("density", "start") or kind == "run" and case["field_every"] == 1:
        # storage order: (brick, tag) of the loaded positions
        B = 8 if kind == "density" else _brick(s, case["halo"])
        c, _ = E.cells()
        nb = [-(-m // B) for m in s.M]
        key = ((c[:, 2] // B) * nb[1] + c[:, 1] // B) * nb[0] + c[:, 0] // B
        order = torch.argsort(key, stable=True)
    if kind == "density":
        tag = s.tag[order]
        moved = _moved(s.R[order], tag, s, seed)
        E.x = _frame(moved, tag).double()
        return E.counts().view(s.K, E.nm)
    if kind == "start":
        F = E.force()
        return dict(F=F[order], tag=order.to(torch.int32), energy=E.energy())
    if kind == "run" and case["field_every"] == 1:
        e = E.fused(n)
        return dict(R=E.x[order], Vel=E.v[order], tag=order.to(torch.int32), energy=e)
    F = E.force()
    if kind in ("graph", "run"):
        E.v = E.v + 0.5 * E.dt * F
        E.drift()
        e = E.fused(n, case if kind == "run" else None, seed)
        return dict(R=E.x, Vel=E.v, energy=e)
    for _ in range(n):
        E.v = E.v + 0.5 * E.dt * F
        E.drift()
        F = E.force()
        E.v = E.v + 0.5 * E.dt * F
    return dict(R=E.x, Vel=E.v, F=F, energy=E.energy())
