"""The work that programs have this library do, as measurable cases.

A case names a structure, a model and one kind of call:

  verlet     ``verlet_step``: a stretch of NVE dynamics, as an MD driver calls it between outputs
  nvt        ``nvt_step``: a stretch of Nose-Hoover-chain dynamics with the virial of every step
  energy     ``build_neighbors`` and ``compute_energy_forces``: one point of a relaxation or a
             Monte-Carlo walk, whose atoms have moved anywhere since the last one
  virial     the same with ``compute_energy_forces_virial``: cell relaxation, elastic constants
  reuse      ``compute_energy_forces`` on a skin list in hand: finite differences, small moves
  noalloc    ``compute_energy_forces_noalloc`` on a list in hand, into buffers in hand: a server
  neighbors  ``build_neighbors`` alone: the list of another code

``exact`` is the potential from its defining equations in plain torch, 64 bits, with autograd.
"""
import math

import numpy as np
import torch

import paper_2608_19041_amd as dp
import synth

R_C, SKIN = 6.0, 1.0
F64 = torch.float64

#: neighbours within 6 A and within 7 A of an atom, on average
NEIGHBOURS = {"fcc": (78, 134), "bcc": (76, 122), "diamond": (158, 253), "water": (91, 144),
              "cluster": (50, 75), "rhomb": (78, 134)}
ATOMS_PER_CELL = {"fcc": 4, "bcc": 2, "diamond": 8, "water": 3, "cluster": 4, "rhomb": 1}


def case(name, call, structure, nx, ny, nz, model, species=1, steps=0, every=0, dt=1.0,
         kelvin=300.0):
    return {"name": name, "call": call, "structure": structure, "nx": nx, "ny": ny, "nz": nz,
            "model": model, "species": species, "steps": steps, "every": every, "dt": dt,
            "kelvin": kelvin}


def listed():
    return [
        # a small cell on the small model: the latency of a step, launches and all
        case("md_small_108", "verlet", "fcc", 3, 3, 3, "small", steps=20),
        # the everyday crystal: about one tile of atoms for each compute unit
        case("md_copper_4000", "verlet", "fcc", 10, 10, 10, "full", steps=20, kelvin=600.0),
        # a 5-species alloy, 25 folded pair tables, a rebuild every ten steps
        case("md_alloy_31250", "verlet", "bcc", 25, 25, 25, "full", species=5, steps=10, every=10,
             kelvin=1000.0),
        # a molecular liquid with uneven neighbourhoods, two species, half a femtosecond
        case("md_water_24000", "verlet", "water", 20, 20, 20, "full", species=2, steps=10, dt=0.5),
        # the headline: a million copper atoms, one rebuild in twenty steps
        case("md_copper_1m", "verlet", "fcc", 63, 63, 63, "full", steps=20, every=20),
        # the whole-step benchmark: a million carbon atoms, NVT, the virial of every step
        case("nvt_diamond_1m", "nvt", "diamond", 50, 50, 50, "full_carbon", steps=10),
        # NVT on a middling, ragged box
        case("nvt_diamond_7056", "nvt", "diamond", 7, 9, 14, "full_carbon", steps=20),
        # an open cluster on the Air variant, a new list with every point
        case("relax_cluster_665", "energy", "cluster", 5, 7, 5, "air"),
        # cell relaxation of a sheared crystal on the Neo variant
        case("cell_rhomb_5814", "virial", "rhomb", 17, 18, 19, "neo"),
        # eight species: beyond the folded tables, on the separable ones
        case("alloy8_13718", "reuse", "bcc", 19, 19, 19, "full", species=8),
        # a server of small cells: the Plus widths with degree four, no allocation
        case("serve_l4_540", "noalloc", "fcc", 5, 3, 9, "plus_l4", species=2),
        # the neighbour list alone, for another code
        case("neighbors_1m", "neighbors", "fcc", 63, 63, 63, "full"),
    ]


def draw(rng):
    call = rng.choice(["verlet", "verlet", "verlet", "nvt", "energy", "virial", "reuse", "noalloc",
                       "neighbors"])
    structure = rng.choice({"nvt": ["diamond", "fcc"], "energy": ["cluster", "fcc", "bcc", "water"],
                            "virial": ["rhomb", "fcc"],
                            "neighbors": ["fcc", "diamond"]}.get(call, ["fcc", "bcc", "diamond",
                                                                   "water"]))
    if structure == "diamond":
        model = "full_carbon"
    else:
        model = rng.choice(["nano", "mini", "neo", "air", "full", "full", "full", "plus_l4",
                            "small" if structure == "fcc" else "mini"])   # calibrated on copper
    species = {"bcc": rng.choice([1, 3, 5, 8]), "water": 2}.get(structure, 1)
    most = {"noalloc": 4000, "cluster": 2000}.get(call, {"cluster": 2000}.get(structure, 400000))
    atoms = math.exp(rng.uniform(math.log(60), math.log(most)))
    edge = (atoms / ATOMS_PER_CELL[structure]) ** (1.0 / 3.0)
    n = [max(2, round(edge * rng.uniform(0.75, 1.3))) for _ in range(3)]
    if structure == "rhomb":
        n = [max(4, v) for v in n]
    steps = rng.randint(4, 24) if call in ("verlet", "nvt") else 0
    return case("", call, structure, *n, model, species=species, steps=steps,
                every=rng.choice([0, 0, 10]) if call == "verlet" else 0,
                dt=0.5 if structure == "water" else 1.0, kelvin=float(rng.randint(100, 1000)))


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def species_types(case):
    """The element indices that a case's atoms take."""
    if case["structure"] == "water":
        return [7, 0]
    if case["structure"] == "diamond":
        return [5]
    return [28, 12, 26, 21, 77, 45, 7, 63][: case["species"]]


def water(nx, ny, nz, rng):
    """A water-like liquid: molecules at about 1 g/cm^3, well spread, turned at random."""
    a = 3.104
    n = nx * ny * nz
    grid = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1)
    o = (grid.reshape(-1, 3) + 0.5) * a + rng.uniform(-0.3, 0.3, size=(n, 3))
    q = rng.normal(size=(n, 4))
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    ax = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y + z * w), 2 * (x * z - y * w)], -1)
    az = np.stack([2 * (x * z + y * w), 2 * (y * z - x * w), 1 - 2 * (x * x + y * y)], -1)
    half = math.radians(104.5) / 2
    pos = np.empty((n, 3, 3))
    pos[:, 0] = o
    pos[:, 1] = o + 0.96 * (math.sin(half) * ax + math.cos(half) * az)
    pos[:, 2] = o + 0.96 * (-math.sin(half) * ax + math.cos(half) * az)
    species = np.tile(np.array([7, 0, 0], dtype=np.int32), n)
    return pos.reshape(-1, 3), species, np.diag([nx * a, ny * a, nz * a])


def host_inputs(case, seed):
    """Positions, species, cell, periodicity, masses and velocities of a case, on the host."""
    rng = np.random.Generator(np.random.PCG64(seed))
    kind, reps = case["structure"], (case["nx"], case["ny"], case["nz"])
    pbc = np.ones(3, np.int32)
    mass = np.ones(synth.N_TYPES + 1)
    mass[: synth.N_TYPES] = synth.ATOMIC_MASS
    if kind == "water":
        pos, species, cell = water(*reps, rng)
    else:
        if kind == "rhomb":   # the primitive cell of the FCC crystal, sheared a little
            prim = 0.5 * 3.615 * np.array([[0, 1, 1], [1, 0, 1], [1, 1, 0]], dtype=np.float64)
            prim = prim @ (np.eye(3) + np.array([[0, 0.02, 0], [0, 0, -0.01], [0.015, 0, 0]]))
            grid = np.stack(np.meshgrid(*(np.arange(r) for r in reps), indexing="ij"), -1)
            pos, cell = grid.reshape(-1, 3) @ prim, np.array(reps)[:, None] * prim
        else:
            lattice, a = {"fcc": ("fcc", 3.615), "cluster": ("fcc", 3.615), "bcc": ("bcc", 2.87),
                          "diamond": ("diamond", 3.567)}[kind]
            pos, cell = synth.lattice(lattice, a, reps)
        jitter = 0.03 if kind == "diamond" else 0.07
        if case["call"] == "neighbors":
            # a list alone is of a nearly relaxed crystal, whose shells of neighbours are all
            # whole, with its atoms numbered from any one of them on
            jitter, pos = 0.01, np.roll(pos, int(rng.integers(len(pos))), axis=0)
        pos = pos + rng.normal(0.0, jitter, size=pos.shape)
        types = np.array(species_types(case), dtype=np.int32)
        species = types[rng.integers(0, len(types), size=len(pos))].astype(np.int32)
        if kind == "cluster":   # a few atoms are off the corner, so that the count is odd
            pos, species, pbc = pos[35:], species[35:], np.zeros(3, np.int32)
    v = rng.normal(size=pos.shape)
    m = mass[species][:, None]
    v *= np.sqrt(synth.KB_EV * case["kelvin"] / (m * synth.MVV2E))
    v -= (m * v).sum(0) / m.sum()
    return pos, species, cell, pbc, mass, v


def prepare(case, seed):
    pos, species, cell, pbc, mass, vel = host_inputs(case, seed)
    dev = torch.device("cuda", 0)
    s = {"case": case, "cell": cell, "pbc": pbc, "mass": mass,
         "pos": torch.tensor(pos, dtype=F64, device=dev)}
    if case["call"] == "neighbors":
        s["cap"] = int(NEIGHBOURS[case["structure"]][1] * len(pos) * 1.25) + 4096
        return s
    spec, weights = synth.model_weights(case["model"])
    s["model"] = dp.Model(synth.pack_blob(spec, weights))
    s["species"] = torch.tensor(species, dtype=torch.int32, device=dev)
    if case["call"] in ("energy", "virial"):
        return s
    rows = dp.build_neighbors(s["pos"], cell, pbc, R_C + SKIN)
    if case["call"] in ("reuse", "noalloc"):
        s["rows"] = rows
        n = len(pos)
        s["out"] = (torch.empty(n, dtype=F64, device=dev), torch.empty(n, 3, dtype=F64, device=dev),
                    torch.empty(1, dtype=F64, device=dev))
        return s
    # dynamics start from the forces at the first positions
    s["vel"] = torch.tensor(vel, dtype=F64, device=dev)
    s["forces"] = s["model"].compute_energy_forces(s["pos"], s["species"], cell, pbc, R_C, *rows)[1]
    s["chain"] = torch.zeros(6, dtype=F64, device=dev)
    return s


def run(s):
    c = s["case"]
    call, cell, pbc = c["call"], s["cell"], s["pbc"]
    if call == "neighbors":
        row_ptr, nbr_j, nbr_shift, n_pairs = dp.build_neighbors(s["pos"], cell, pbc, R_C + SKIN,
                                                                cap=s["cap"])
        return row_ptr, nbr_j, nbr_shift, n_pairs
    m = s["model"]
    if call == "verlet":
        e_pot, e_kin, _ = m.verlet_step(s["pos"], s["vel"], s["species"], s["mass"], cell, pbc, R_C,
                                        SKIN, c["dt"], c["steps"], c["every"], s["forces"])
        return s["pos"], s["vel"], s["forces"], e_pot, e_kin
    if call == "nvt":
        e_pot, e_kin, e_bath, virial, _ = m.nvt_step(
            s["pos"], s["vel"], s["species"], s["mass"], cell, pbc, R_C, SKIN, c["dt"], c["steps"],
            c["every"], s["forces"], c["kelvin"], 100.0, s["chain"], virial=True)
        return s["pos"], s["vel"], s["forces"], e_pot, e_kin, e_bath, virial
    if call == "energy":
        rows = dp.build_neighbors(s["pos"], cell, pbc, R_C)
        return m.compute_energy_forces(s["pos"], s["species"], cell, pbc, R_C, *rows)
    if call == "virial":
        rows = dp.build_neighbors(s["pos"], cell, pbc, R_C)
        return m.compute_energy_forces_virial(s["pos"], s["species"], cell, pbc, R_C, *rows)[:4]
    f = m.compute_energy_forces_noalloc if call == "noalloc" else m.compute_energy_forces
    return f(s["pos"], s["species"], cell, pbc, R_C, *s["rows"], *s["out"])


def atoms_of(case):
    n = case["nx"] * case["ny"] * case["nz"] * ATOMS_PER_CELL[case["structure"]]
    return n - 35 if case["structure"] == "cluster" else n


def work(case):
    """What an evaluation cannot do without: the list once and the atoms' state in and out; for
    each edge a cubic for each channel and one accumulation for each feature, and their adjoints;
    for each atom the products of the network and their adjoints."""
    n = atoms_of(case)
    near, listed_ = NEIGHBOURS[case["structure"]]
    if case["call"] == "neighbors":
        return {"bytes": n * (24 + 8 + 8 * listed_), "flops": 10.0 * n * listed_}
    spec = synth.MODELS[case["model"]]
    C1 = max(4, 2 ** math.ceil(0.5 * math.log2(spec.C0)))
    S = spec.C0 + 3 * C1 + 5 * max(4, C1 // 2) + {2: 0, 3: 7, 4: 16}[spec.L]
    D = synth.descriptor_width(spec.C0, spec.L)
    fresh = case["call"] in ("energy", "virial")   # the list of these is at the cutoff itself
    per_eval = {"bytes": n * (8 * (near if fresh else listed_) + 24 + 24 + 8 + 4),
                "flops": n * (4.0 * (D * spec.F + 2 * spec.F * spec.F)
                              + near * 2.0 * (2 * 4 * spec.C0 + 4 * S))}
    evals = case["steps"] if case["steps"] else 1
    moved = 72 * n if case["steps"] else 0   # velocities in and out, positions out
    return {"bytes": evals * (per_eval["bytes"] + moved), "flops": evals * per_eval["flops"]}


def tolerance(case):
    """32-bit sums of a few hundred terms through a network of three layers: forces differ by
    about 2e-6 of their norm from 64 bits, a single one by some 1e-5 of the rms.  In dynamics the
    stiffest (a liquid of bonded hydrogen atoms) let such a difference grow over the steps."""
    if case["call"] == "neighbors":
        return "exact"
    return {"rel": 2e-5, "max": 5e-4}


# ---------------------------------------------------------------------------------------------
# the potential in 64 bits
# ---------------------------------------------------------------------------------------------
def harmonics(u, l):
    x, y, z = u.unbind(-1)
    s = x * x + y * y + z * z
    r = math.sqrt
    if l == 0:
        return torch.ones_like(x)[:, None]
    if l == 1:
        return u
    if l == 2:
        b = [r(3) * x * y, r(3) * y * z, 1.5 * z * z - 0.5 * s, r(3) * x * z,
             0.5 * r(3) * (x * x - y * y)]
    elif l == 3:
        b = [r(5 / 8) * y * (3 * x * x - y * y), r(15) * x * y * z, r(3 / 8) * y * (5 * z * z - s),
             0.5 * z * (5 * z * z - 3 * s), r(3 / 8) * x * (5 * z * z - s),
             0.5 * r(15) * z * (x * x - y * y), r(5 / 8) * x * (x * x - 3 * y * y)]
    else:
        b = [0.5 * r(35) * x * y * (x * x - y * y), 0.25 * r(70) * y * z * (3 * x * x - y * y),
             0.5 * r(5) * x * y * (7 * z * z - s), 0.25 * r(10) * y * z * (7 * z * z - 3 * s),
             0.125 * (35 * z ** 4 - 30 * z * z * s + 3 * s * s),
             0.25 * r(10) * x * z * (7 * z * z - 3 * s),
             0.25 * r(5) * (x * x - y * y) * (7 * z * z - s),
             0.25 * r(70) * x * z * (x * x - 3 * y * y),
             0.125 * r(35) * (x ** 4 - 6 * x * x * y * y + y ** 4)]
    return torch.stack(b, -1)


class Reference:
    """The potential by its equations."""

    def __init__(self, model, dev):
        self.spec, w = synth.model_weights(model)
        self.w = {k: torch.tensor(v, dtype=F64, device=dev) for k, v in w.items()}
        C0, L = self.spec.C0, self.spec.L
        C1 = max(4, 2 ** math.ceil(0.5 * math.log2(C0)))
        C2 = max(4, C1 // 2)
        self.C, self.K = [C0, C1, C2, 1, 1][: L + 1], [0, C2, 2, 1, 1][: L + 1]
        # couplings: integrals of three harmonics over the sphere, normalised, negative sign
        zg, wg = np.polynomial.legendre.leggauss(12)
        ph = 2 * math.pi * np.arange(30) / 30
        z, p = (a.reshape(-1) for a in np.meshgrid(zg, ph, indexing="ij"))
        u = np.stack([np.sqrt(1 - z * z) * np.cos(p), np.sqrt(1 - z * z) * np.sin(p), z], -1)
        B = [harmonics(torch.tensor(u, dtype=F64, device=dev), l) for l in range(L + 1)]
        wq = torch.tensor(np.repeat(wg, 30), dtype=F64, device=dev)
        self.couplings = []
        for a in range(1, L + 1):
            for b in range(a, L + 1):
                for c in range(b, min(L, a + b) + 1):
                    if (a + b + c) % 2 == 0:
                        t = torch.einsum("p,pi,pj,pk->ijk", wq, B[a], B[b], B[c])
                        self.couplings.append(((a, b, c), -t / t.norm(), self.kept((a, b, c))))

    def kept(self, degrees):
        """The entries of a block that stand for all their permutations, and their weights."""
        ranks = [self.K[l] for l in degrees]
        found = {}
        for idx in np.ndindex(*ranks):
            key = []
            for l in sorted(set(degrees)):
                key.append(tuple(sorted(idx[k] for k in range(3) if degrees[k] == l)))
            found.setdefault(tuple(key), []).append(idx)
        first = sorted((min(v), len(v)) for v in found.values())
        return [f[0] for f in first], [math.sqrt(f[1]) for f in first]

    def gated(self, x, W):
        g, v = (x @ W).chunk(2, -1)
        return g * torch.sigmoid(g) * v

    def centres(self, r, i, n, a, b, types):
        """E_i of n centres from the edges (vector r, centre i, types a -> b)."""
        w, C = self.w, self.C
        rho = torch.sqrt((r * r).sum(-1) + 1e-14)
        u = r / rho[:, None]
        t = (1 - rho / self.spec.r_c).clamp(0, 1)
        x = 1 - t
        chi = t ** 4 * (1 + 4 * x + 10 * x ** 2 + 20 * x ** 3 + 35 * x ** 4)
        h = self.gated(torch.sin(rho[:, None] * w["omega"]) / rho[:, None], w["W_in"])
        pairs, back = torch.unique(a * 1000 + b, return_inverse=True)
        X0 = w["type_embed"]
        xa, xb = X0[pairs // 1000], X0[pairs % 1000]
        p = 0.1 * (self.gated(torch.cat([xa, xb], -1), w["Wp_in"]) @ w["Wp_out"])
        gamma, beta = 1 + torch.tanh(p[:, : C[0]]), xa + xb + torch.tanh(p[:, C[0]: 2 * C[0]])
        psi = gamma[back] * (h @ w["W_out"]) + beta[back]
        if self.spec.R:
            U = torch.tanh(p[:, 2 * C[0]:]).reshape(-1, C[0], self.spec.R)
            q = h @ w["W_mode"]
            for k in range(self.spec.R):
                psi = psi + U[back][:, :, k] * q[:, k: k + 1]
        add = lambda v: torch.zeros(n, *v.shape[1:], dtype=F64, device=v.device).index_add(0, i, v)  # noqa: E731
        M0, M1 = torch.sqrt(0.25 + add(chi ** 2)), torch.sqrt(0.25 + add(chi ** 4))
        X = [add(chi[:, None] * psi) / M0[:, None]]
        for l in range(1, len(C)):
            y = add((chi * chi)[:, None, None] * harmonics(u, l)[:, :, None] * psi[:, None, : C[l]])
            y = y / M1[:, None, None]
            X.append(y + y @ w["W_align%d" % l] if l <= 2 else y)
        d = [X0[types], X[0], M0[:, None], M1[:, None]]
        for l in range(1, len(C)):
            G = X[l].transpose(1, 2) @ X[l]
            iu, ju = (torch.tensor(v, device=G.device) for v in np.triu_indices(C[l]))
            d.append(G[:, iu, ju] * torch.where(iu == ju, 1.0, math.sqrt(2.0)).to(F64))
        Z = [None] + [X[l] if self.K[l] == C[l] else X[l] @ w["A%d" % l] for l in range(1, len(C))]
        for (l1, l2, l3), T, (at, weight) in self.couplings:
            J = torch.einsum("abc,nai,nbj,nck->nijk", T, Z[l1], Z[l2], Z[l3])
            i1, i2, i3 = (torch.tensor(v, device=J.device) for v in zip(*at))
            d.append(J[:, i1, i2, i3] * torch.tensor(weight, dtype=F64, device=J.device))
        z = Z[2].transpose(1, 2)   # [n, K2, 5]: xy, yz, zz, xz, xx - yy
        s2, s6 = 1 / math.sqrt(2), 1 / math.sqrt(6)
        xy, yz, zz, xz, dd = z.unbind(-1)
        Q = torch.stack([-s6 * zz + s2 * dd, s2 * xy, s2 * xz, s2 * xy, -s6 * zz - s2 * dd, s2 * yz,
                         s2 * xz, s2 * yz, 2 * s6 * zz], -1).reshape(n, -1, 3, 3)
        d.append(torch.einsum("nhab,nbk->nhka", Q, Z[1]).square().sum(-1).reshape(n, -1))
        v = (torch.cat(d, 1) - w["mu"]) / w["sigma"]
        for k in range(1, self.spec.n_layers + 1):
            o = v @ w["Theta%d" % k] + w["b%d" % k]
            o = o * torch.sigmoid(o)
            v = o + v if o.shape == v.shape else o
        return v @ w["w_head"] + w["b_head"][0] + w["E_ref"][types]

    def edges(self, pos, cell, pbc, r):
        """(i, j, n) of all pairs within r, ordered by i."""
        n = len(pos)
        height = 1 / torch.linalg.inv(cell).norm(dim=0)
        frac = pos @ torch.linalg.inv(cell)
        extent = frac.max(0).values - frac.min(0).values
        reach = [int(math.ceil(float(r / height[k] + extent[k]))) if pbc[k] else 0 for k in range(3)]
        shifts = torch.cartesian_prod(*(torch.arange(-k, k + 1) for k in reach)).to(pos.device)
        # images of the atoms that can be near any atom, then all distances in slabs of centres
        lo, hi = pos.min(0).values - r, pos.max(0).values + r
        img = pos[None] + (shifts.to(F64) @ cell)[:, None]
        near = ((img > lo) & (img < hi)).all(-1)
        sh, j = torch.nonzero(near, as_tuple=True)
        q = img[sh, j]
        found = []
        step = max(1, int(4e8 // (len(q) * 3)))
        for c in range(0, n, step):
            d2 = (q[None] - pos[c: c + step, None]).square().sum(-1)
            a, b = torch.nonzero(d2 < r * r, as_tuple=True)
            a = a + c
            keep = (j[b] != a) | (shifts[sh[b]] != 0).any(-1)
            found.append((a[keep], j[b][keep], shifts[sh[b]][keep]))
        return tuple(torch.cat(v) for v in zip(*found))

    def evaluate(self, pos, species, cell, edges):
        """E_i, forces and virial."""
        i, j, shift = edges
        n = len(pos)
        rows = torch.searchsorted(i, torch.arange(n + 1, device=pos.device)).tolist()
        e, F = torch.empty(n, dtype=F64, device=pos.device), torch.zeros_like(pos)
        xi = torch.zeros(3, 3, dtype=F64, device=pos.device)
        per = 2000
        for c in range(0, n, per):
            m = min(per, n - c)
            k = slice(rows[c], rows[c + m])
            r = (pos[j[k]] + shift[k].to(F64) @ cell - pos[i[k]]).requires_grad_()
            near = r.detach().square().sum(-1) < self.spec.r_c ** 2
            E = self.centres(r[near], i[k][near] - c, m, species[i[k]][near], species[j[k]][near],
                             species[c: c + m])
            (g,) = torch.autograd.grad(E.sum(), r)
            e[c: c + m] = E.detach()
            F.index_add_(0, i[k], g).index_add_(0, j[k], -g)
            xi -= g.T @ r.detach()
        return e, F, xi


def chain_half(vxi, xi, Q, kT, nf, kin, dt):
    """Half a step of a Nose-Hoover chain; the factor for the velocities."""
    M = len(Q)

    def force(k, kin):
        return ((2 * kin - nf * kT) if k == 0 else (Q[k - 1] * vxi[k - 1] ** 2 - kT)) / Q[k]

    def turn(k, kin):
        f = math.exp(-dt / 8 * vxi[k + 1]) if k + 1 < M else 1.0
        vxi[k] = (vxi[k] * f + dt / 4 * force(k, kin)) * f

    for k in reversed(range(M)):
        turn(k, kin)
    s = math.exp(-dt / 2 * vxi[0])
    for k in range(M):
        xi[k] += dt / 2 * vxi[k]
    for k in range(M):
        turn(k, kin * s * s)
    return s


def exact(case, seed):
    n, call = atoms_of(case), case["call"]
    if call == "neighbors" or n * max(1, case["steps"]) > 500000 or n > 60000:
        return None
    dev = torch.device("cuda", 0)
    pos, species, cell, pbc, mass, vel = host_inputs(case, seed)
    pos, cell, vel = (torch.tensor(v, dtype=F64, device=dev) for v in (pos, cell, vel))
    species = torch.tensor(species, dtype=torch.int64, device=dev)
    ref = Reference(case["model"], dev)
    edges = ref.edges(pos, cell, pbc, R_C + (3.0 if case["steps"] else 0.0))
    e, F, xi = ref.evaluate(pos, species, cell, edges)
    if call == "virial":
        return e, F, e.sum().reshape(1), xi
    if not case["steps"]:
        return e, F, e.sum().reshape(1)
    m = torch.tensor(mass, dtype=F64, device=dev)[species][:, None] * synth.MVV2E
    dt = case["dt"]
    kinetic = lambda: float(0.5 * (m * vel * vel).sum())  # noqa: E731
    nvt = call == "nvt"
    kT, nf = 8.617333262e-5 * case["kelvin"], 3 * n - 3
    Q = [nf * kT * 1e4, kT * 1e4, kT * 1e4]
    bath, vbath = [0.0] * 3, [0.0] * 3
    e_pot, e_kin, e_bath, virials = [], [], [], []
    for _ in range(case["steps"]):
        if nvt:
            vel = vel * chain_half(vbath, bath, Q, kT, nf, kinetic(), dt)
        vel = vel + 0.5 * dt * F / m
        pos = pos + dt * vel
        e, F, xi = ref.evaluate(pos, species, cell, edges)
        vel = vel + 0.5 * dt * F / m
        if nvt:
            vel = vel * chain_half(vbath, bath, Q, kT, nf, kinetic(), dt)
        e_pot.append(float(e.sum()))
        e_kin.append(kinetic())
        e_bath.append(sum(0.5 * q * v * v for q, v in zip(Q, vbath)) + nf * kT * bath[0]
                      + kT * (bath[1] + bath[2]))
        virials.append(xi)
    out = [pos, vel, F] + [torch.tensor(v, dtype=F64) for v in (e_pot, e_kin)]
    return out + [torch.tensor(e_bath, dtype=F64), torch.stack(virials)] if nvt else out
