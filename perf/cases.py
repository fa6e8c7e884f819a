"""Timed cases of the energy / force / virial path, their inputs and a plain
float64 reference.

A case is one system and one way of calling the library:

  point  a structure not seen before: neighbour list, then energies, forces,
         virials and the totals read back (screening, relaxation, a server)
  eval   one evaluation on a list that is already there, as in every MD step
         between rebuilds
  md     one list lifetime of a velocity-Verlet run restarted from a saved
         state: a rebuild, then `steps` steps with the displacement check

Systems are FCC and BCC crystals with Gaussian displacements, some sites
vacant, 1 to 6 species, cutoffs of 6 and 6.5 A, the radial widths and angular
orders of the hyper-parameter grid, in both precisions of the network.
Weights are drawn N(0, 1/fan_in) with the head's output layer scaled so that
forces are about 1 eV/A.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2608_16329_amd import Potential

SITES = {"fcc": [(0, 0, 0), (0, .5, .5), (.5, 0, .5), (.5, .5, 0)], "bcc": [(0, 0, 0), (.5, .5, .5)]}
MASSES = [180.948, 92.906, 183.84, 95.95, 50.942, 26.982]   # Ta Nb W Mo V Al
HEAD_SCALE = 0.01                                           # on the head's output layer
KB = 8.617333262e-5                                         # eV/K
ACC = 9.648533212e-3                                        # (eV/A)/amu -> A/fs^2
ENC, HEAD, ENC_LAYERS, HEAD_LAYERS, SKIN, DT = 128, 64, 3, 4, 0.5, 1.0


def _case(name, **over):
    c = dict(name=name, mode="eval", lattice="fcc", nx=8, ny=8, nz=8, a=3.6, vacancy=0.0, species=6, dilute=False,
             sigma=0.1, cutoff=6.0, k=32, lmax=3, precision=64, recompute=False, steps=10)
    c.update(over)
    return c


def _cube(n):
    return dict(nx=n, ny=n, nz=n)


BCC = dict(lattice="bcc", a=3.2)
TERNARY = dict(species=3, dilute=True, a=4.05, cutoff=6.5)


def listed():
    return [
        # a single point of a small binary cell: launches and latency
        _case("point-binary-256-f64", mode="point", species=2, sigma=0.05, **_cube(4)),
        # the same use with the float32 network, one element
        _case("point-unary-432-f32", mode="point", species=1, sigma=0.08, precision=32, **BCC, **_cube(6)),
        # short MD of a small binary alloy: rebuild, 10 steps, displacement checks
        _case("md-binary-2k-f64", mode="md", species=2, sigma=0.05, **_cube(8)),
        # odd counts: a slab-like six-component cell with vacancies
        _case("eval-ragged-5k-f64", nx=13, ny=11, nz=9, vacancy=0.03),
        # a mid-sized six-component BCC cell, float32 network
        _case("eval-hea6-14k-f32", precision=32, **BCC, **_cube(19)),
        # one element, 65,536 atoms
        _case("eval-unary-65k-f64", species=1, sigma=0.08, **BCC, **_cube(32)),
        # dilute ternary alloy with the longer cutoff
        _case("eval-ternary-131k-f64", **TERNARY, **_cube(32)),
        # wide radial basis
        _case("eval-k64-55k-f64", k=64, **_cube(24)),
        # high angular order, float32 network
        _case("eval-lmax5-65k-f32", lmax=5, precision=32, **BCC, **_cube(32)),
        # evaluation that keeps nothing per pair between its passes
        _case("eval-recompute-55k-f64", recompute=True, **_cube(24)),
        # the production size per evaluation: six components, 1,048,576 atoms
        _case("eval-hea6-1m-f64", **_cube(64)),
        # the same with the float32 network, list and evaluation (rebuild steps)
        _case("point-hea6-1m-f32", mode="point", precision=32, **_cube(64)),
    ]


def draw(rng):
    """Another case of the same ranges; at most 2^20 sites, fewer where an
    option makes an atom dearer."""
    lattice = rng.choice(["fcc", "bcc"])
    mode = rng.choice(["point", "eval", "eval", "md"])
    c = _case("", mode=mode, lattice=lattice, a=3.6 if lattice == "fcc" else 3.2,
              species=rng.choice([1, 2, 3, 4, 6]), dilute=rng.random() < 0.25, sigma=rng.uniform(0.04, 0.1),
              precision=rng.choice([64, 32]), vacancy=rng.choice([0.0, 0.0, rng.uniform(0.0, 0.1)]),
              k=rng.choice([32, 32, 16, 64]), lmax=rng.choice([3, 3, 1, 2, 5]))
    if rng.random() < 0.25:
        c["cutoff"], c["a"] = 6.5, 4.05 if lattice == "fcc" else 3.4
    c["recompute"] = mode == "eval" and c["k"] == 32 and c["lmax"] <= 3 and rng.random() < 0.25
    low = math.ceil(2.0 * (c["cutoff"] + SKIN) / c["a"])
    sites = (1 << 20) / (3.0 if c["lmax"] > 3 else 1.0) / (2.0 if c["k"] == 64 else 1.0) \
        / (2.0 if c["recompute"] else 1.0) / (16.0 if mode == "md" else 1.0)
    edge = math.exp(rng.uniform(math.log(low), math.log((sites / len(SITES[lattice])) ** (1 / 3))))
    for d in ("nx", "ny", "nz"):
        c[d] = max(low, min(round(edge * rng.uniform(0.8, 1.25)), 2 * round(edge)))
    while c["nx"] * c["ny"] * c["nz"] * len(SITES[lattice]) > sites:
        d = max(("nx", "ny", "nz"), key=lambda e: c[e])
        if c[d] <= low:
            break
        c[d] -= 1
    del c["name"]
    return c


# ---- inputs ------------------------------------------------------------------

def _hparams(case):
    return SimpleNamespace(n_species=case["species"], cutoff=case["cutoff"], skin=SKIN, k=case["k"], lmax=case["lmax"],
                           angular=0, enc_cond=2, reg_cond=1, enc_width=ENC, enc_hidden=ENC_LAYERS, reg_width=HEAD,
                           reg_hidden=HEAD_LAYERS, precision=case["precision"])


def _layers(case):
    """(rows, columns, fan-in) of every weight segment of one encoder table and
    of one head table, in the order of the blob (columns 0: a vector)."""
    k, nin = case["k"], (case["lmax"] + 1) * case["k"]
    enc = [(ENC, 0, 1), (ENC, 0, 1)] + [(ENC, ENC, ENC), (ENC, 0, ENC)] * (ENC_LAYERS - 1) + [(k, ENC, ENC), (k, 0, ENC)]
    head = [(HEAD, nin, nin), (HEAD, 0, nin)] + [(HEAD, HEAD, HEAD), (HEAD, 0, HEAD)] * (HEAD_LAYERS - 1) \
        + [(HEAD, 0, HEAD), (1, 0, HEAD)]
    return enc, head


def _weights(case, seed):
    """Weight tensors per table and the flat blob the library takes."""
    rng = np.random.default_rng([seed, 1])
    enc, head = _layers(case)
    tables, blob = [], []
    for segments, count in ((enc, case["species"] ** 2), (head, case["species"])):
        for _ in range(count):
            t = []
            for i, (rows, cols, fan) in enumerate(segments):
                w = rng.standard_normal(rows * max(cols, 1)) / math.sqrt(fan)
                if segments is head and i >= len(segments) - 2:
                    w *= HEAD_SCALE
                t.append(w.reshape(rows, cols) if cols else w)
                blob.append(w)
            tables.append(t)
    return tables, np.concatenate(blob)


def _system(case, seed):
    """Positions, species, velocities, forces-to-be, box and masses on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dev = torch.device("cuda")
    n = [case["nx"], case["ny"], case["nz"]]
    cells = torch.cartesian_prod(*[torch.arange(m, device=dev, dtype=torch.float64) for m in n])
    pos = (cells[:, None, :] + torch.tensor(SITES[case["lattice"]], device=dev, dtype=torch.float64)[None]).reshape(-1, 3)
    pos = pos * case["a"]
    if case["vacancy"] > 0:
        kept = torch.randperm(len(pos), device=dev, generator=g)[:round(len(pos) * (1.0 - case["vacancy"]))]
        pos = pos[torch.sort(kept)[0]]
    pos = pos + case["sigma"] * torch.randn(pos.shape, device=dev, dtype=torch.float64, generator=g)
    C = case["species"]
    types = torch.randint(0, C, (len(pos),), device=dev, dtype=torch.int32, generator=g)
    if case["dilute"]:
        types = torch.where(torch.rand(len(pos), device=dev, generator=g) < 0.9, torch.zeros_like(types), types)
    masses = np.array(MASSES[:C])
    m = torch.tensor(masses, device=dev)[types.long()]
    vel = torch.randn(pos.shape, device=dev, dtype=torch.float64, generator=g) * torch.sqrt(KB * 300.0 * ACC / m)[:, None]
    vel -= (m[:, None] * vel).sum(0) / m.sum()
    return pos.contiguous(), types, vel.contiguous(), np.array(n, float) * case["a"], masses


def prepare(case, seed):
    """A context with the model's weights and the caller's arrays; for eval and
    md also the list (md: and the forces of the saved state)."""
    pos, types, vel, box, masses = _system(case, seed)
    s = SimpleNamespace(case=case, pos=pos, types=types, box=box, pot=Potential(_hparams(case), _weights(case, seed)[1]))
    if case["recompute"]:
        s.pot.set_fusion(1)
    s.F = torch.zeros_like(pos)
    s.E = torch.zeros(len(pos), dtype=torch.float64, device=pos.device)
    s.V = torch.zeros((len(pos), 9), dtype=torch.float64, device=pos.device)
    if case["mode"] != "point":
        s.pot.build_neighbors(pos, types, box)
    if case["mode"] == "md":
        s.pot.set_masses(masses)
        s.pot.compute(pos, s.F, s.E, s.V)
        s.start = (pos.clone(), vel.clone(), s.F.clone())
        s.vel = vel
    return s


def run(s):
    mode = s.case["mode"]
    if mode == "point":
        s.pot.build_neighbors(s.pos, s.types, s.box)
        totals = s.pot.compute(s.pos, s.F, s.E, s.V, totals=True)
        return {"E": s.E, "F": s.F, "V": s.V, "totals": totals}
    if mode == "eval":
        s.pot.compute(s.pos, s.F, s.E, s.V)
        return {"E": s.E, "F": s.F, "V": s.V}
    for dst, src in zip((s.pos, s.vel, s.F), s.start):
        dst.copy_(src)
    s.pot.build_neighbors(s.pos, s.types, s.box)
    for _ in range(s.case["steps"]):
        moved = s.pot.md_first_half(s.pos, s.vel, s.F, DT, track=True)
        if moved > (0.5 * SKIN) ** 2:
            s.pot.build_neighbors(s.pos, s.types, s.box)
        s.pot.compute(s.pos, s.F, s.E, s.V)
        s.pot.md_second_half(s.vel, s.F, DT)
    return {"pos": s.pos, "vel": s.vel, "E": s.E, "F": s.F, "V": s.V}


# ---- size of the work -------------------------------------------------------

def work(case):
    """Arithmetic of the model as it is defined (encoder value and slope in r,
    moment and the two adjoint contractions per pair inside the cutoff; head
    forward and backward per atom) and each array once."""
    sites = len(SITES[case["lattice"]])
    n = case["nx"] * case["ny"] * case["nz"] * sites * (1.0 - case["vacancy"])
    density = sites / case["a"] ** 3 * (1.0 - case["vacancy"])
    near = 4.0 / 3.0 * math.pi * case["cutoff"] ** 3 * density
    listed_pairs = 4.0 / 3.0 * math.pi * (case["cutoff"] + SKIN) ** 3 * density
    k, d = case["k"], (case["lmax"] + 1) ** 2
    enc = ENC + (ENC_LAYERS - 1) * ENC * ENC + ENC * k
    head = (case["lmax"] + 1) * k * HEAD + (HEAD_LAYERS - 1) * HEAD * HEAD + HEAD
    flops = n * (near * (4.0 * enc + 6.0 * d * k) + 4.0 * head)
    size = case["precision"] // 8
    tables = sum(r * max(c, 1) for r, c, _ in _layers(case)[0]) * case["species"] ** 2 \
        + sum(r * max(c, 1) for r, c, _ in _layers(case)[1]) * case["species"]
    out = n * (24 + 8 + 72)
    evaluation = n * (24 + 4) + out + tables * size
    entries = 2.0 * n * listed_pairs
    if case["mode"] == "point":
        return {"bytes": evaluation, "flops": flops}
    if case["mode"] == "eval":
        return {"bytes": evaluation + entries, "flops": flops}
    # positions, velocities and forces of the saved state in, all arrays out
    return {"bytes": evaluation + n * (72 + 48), "flops": case["steps"] * flops}


def tolerance(case):
    # four times the largest difference from `exact` seen over the listed cases,
    # 50 drawn ones and 360 small systems: one-element models, whose energies
    # and forces cancel the most, reach 2.9e-14 and 1.1e-5
    return {"rel": 1.2e-13, "max": 2.5e-12} if case["precision"] == 64 else {"rel": 5e-5, "max": 4e-4}


# ---- float64 reference ------------------------------------------------------

def _pairs(pos, box, rc):
    """Directed pairs (i, j) within rc in a periodic box, i ascending, and
    r_j - r_i: the half-width cell grid for large systems, all pairs otherwise."""
    dev, n = pos.device, len(pos)
    L = torch.tensor(box, device=dev)
    w = torch.remainder(pos, L)
    found = []
    if n <= 6000:
        for i in range(0, n, 512):
            d = w[None, :, :] - w[i:i + 512, None, :]
            d = d - L * torch.round(d / L)
            hit = (d * d).sum(-1) < rc * rc
            hit[torch.arange(hit.shape[0], device=dev), torch.arange(i, i + hit.shape[0], device=dev)] = False
            a, j = torch.nonzero(hit, as_tuple=True)
            found.append((a + i, j, d[a, j]))
    else:
        nc = [max(1, int(b // rc)) for b in box]
        cell = [torch.clamp((w[:, d] * (nc[d] / box[d])).long(), max=nc[d] - 1) for d in range(3)]
        flat = (cell[0] * nc[1] + cell[1]) * nc[2] + cell[2]
        order = torch.argsort(flat)
        ncell = nc[0] * nc[1] * nc[2]
        count = torch.bincount(flat, minlength=ncell)
        start = torch.cumsum(count, 0) - count
        widest = int(count.max())
        around = sorted({tuple((o % m) for o, m in zip((x, y, z), nc)) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)})
        for o in around:
            other = [(cell[d] + o[d]) % nc[d] for d in range(3)]
            f2 = (other[0] * nc[1] + other[1]) * nc[2] + other[2]
            step = max(1, (1 << 24) // widest)
            for i in range(0, n, step):
                f = f2[i:i + step]
                t = torch.arange(widest, device=dev)[None, :]
                ok = t < count[f][:, None]
                j = order[torch.where(ok, start[f][:, None] + t, torch.zeros_like(t))]
                a = torch.arange(i, i + len(f), device=dev)
                d = w[j] - w[a][:, None, :]
                d = d - L * torch.round(d / L)
                a, c = torch.nonzero(ok & ((d * d).sum(-1) < rc * rc) & (j != a[:, None]), as_tuple=True)
                found.append((a + i, j[a, c], d[a, c]))
    i, j, d = (torch.cat(x) for x in zip(*found))
    order = torch.argsort(i, stable=True)
    return i[order], j[order], d[order]


def _angular(u, lmax):
    """Real harmonics of unit vectors, order by order, scaled so that the sum
    over one order at two directions is l!/(2l-1)!! P_l of their cosine."""
    x, y, z = u.unbind(1)
    re, im = [torch.ones_like(x)], [torch.zeros_like(x)]
    for _ in range(lmax):
        re, im = re + [re[-1] * x - im[-1] * y], im + [re[-1] * y + im[-1] * x]
    q = {}
    for m in range(lmax + 1):
        q[m, m] = torch.full_like(x, float(math.prod(range(1, 2 * m, 2))))
        if m < lmax:
            q[m + 1, m] = (2 * m + 1) * z * q[m, m]
        for l in range(m + 2, lmax + 1):
            q[l, m] = ((2 * l - 1) * z * q[l - 1, m] - (l + m - 1) * q[l - 2, m]) / (l - m)
    rows = []
    for l in range(lmax + 1):
        s = math.sqrt(math.factorial(l) / math.prod(range(1, 2 * l, 2)))
        for m in range(l + 1):
            f = s * math.sqrt((2.0 if m else 1.0) * math.factorial(l - m) / math.factorial(l + m)) * q[l, m]
            rows += [f * re[m]] + ([f * im[m]] if m else [])
    return torch.stack(rows, 1)


def _network(x, t):
    """Residual SiLU network; t: first weights and bias, hidden layers, output."""
    y = torch.nn.functional.silu(x @ t[0].T + t[1])
    for h in range(2, len(t) - 2, 2):
        y = y + torch.nn.functional.silu(y @ t[h].T + t[h + 1])
    return y @ t[-2].T + t[-1]


def _reference(case, tables, pos, types, box):
    """E_i, F and per-atom virial by automatic differentiation, a block of
    centre atoms at a time."""
    dev, n, C, k, lmax = pos.device, len(pos), case["species"], case["k"], case["lmax"]
    tab = [[torch.tensor(w, device=dev) for w in t] for t in tables]
    enc = [[t[0][:, None]] + t[1:] for t in tab[:C * C]]
    head = [t[:-2] + [t[-2][None, :], t[-1]] for t in tab[C * C:]]
    types = types.long()
    pi, pj, d = _pairs(pos, box, case["cutoff"])
    first = torch.searchsorted(pi, torch.arange(n + 1, device=dev))
    E = torch.zeros(n, dtype=torch.float64, device=dev)
    F, V = torch.zeros_like(pos), torch.zeros((n, 9), dtype=torch.float64, device=dev)
    for a in range(0, n, 8192):
        b = min(n, a + 8192)
        lo, hi = int(first[a]), int(first[b])
        i, j = pi[lo:hi], pj[lo:hi]
        r = d[lo:hi].clone().requires_grad_(True)
        dist = r.norm(dim=1)
        tau = types[i] * C + types[j]
        order = torch.argsort(tau)
        m = torch.cat([_network(dist[s][:, None], enc[t]) for t, s in
                       enumerate(torch.split(order, torch.bincount(tau, minlength=C * C).tolist())) if len(s)])
        m = torch.zeros_like(m).index_copy(0, order, m) if len(m) else m
        g = m * (0.5 + 0.5 * torch.cos(math.pi / case["cutoff"] * dist))[:, None]
        f = _angular(r / dist[:, None], lmax)
        P = torch.zeros((b - a, f.shape[1], k), dtype=torch.float64, device=dev)
        P = P.index_add(0, i - a, f[:, :, None] * g[:, None, :])
        G = [P[:, 0, :]] + [(P[:, l * l:(l + 1) ** 2, :] ** 2).sum(1) for l in range(1, lmax + 1)]
        G = torch.cat(G, 1)
        e = torch.zeros(b - a, dtype=torch.float64, device=dev)
        for s in range(C):
            own = torch.nonzero(types[a:b] == s)[:, 0]
            if len(own):
                e = e.index_copy(0, own, _network(G[own], head[s])[:, 0])
        f = torch.autograd.grad(e.sum(), r)[0]
        E[a:b] = e.detach()
        F.index_add_(0, i, f)
        F.index_add_(0, j, -f)
        V.index_add_(0, i, -(r.detach()[:, :, None] * f[:, None, :]).reshape(-1, 9))
    return E, F, V


def exact(case, seed):
    pos, types, vel, box, masses = _system(case, seed)
    tables = _weights(case, seed)[0]
    E, F, V = _reference(case, tables, pos, types, box)
    if case["mode"] == "md":
        acc = (ACC / torch.tensor(masses, device=pos.device))[types.long()][:, None]
        for _ in range(case["steps"]):
            vel = vel + 0.5 * DT * acc * F
            pos = pos + DT * vel
            E, F, V = _reference(case, tables, pos, types, box)
            vel = vel + 0.5 * DT * acc * F
        return {"pos": pos, "vel": vel, "E": E, "F": F, "V": V}
    out = {"E": E, "F": F, "V": V}
    if case["mode"] == "point":
        out["totals"] = torch.cat([E.sum()[None], V.sum(0)]).cpu().numpy()
    return out
