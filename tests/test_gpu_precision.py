"""What the stages of an evaluation lose against 64 bits, each from its own
float32 inputs, so that no stage hides behind another: the readout from the node
state, the MLP from the descriptor; and whole energies and forces of isolated
pairs, where nothing averages the radial tables' errors.  Errors are 2-norms over all atoms of eight
jittered systems; the bounds are what plain float32 kernels (a sum over lanes in
order for the readout, v_mfma_f32_16x16x4_f32 for the MLP) reach on the same
systems, with a few percent for another order of sums: the eight seeds' own
spread is 2 to 4 percent.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import model as om

pytestmark = pytest.mark.gpu
F64 = torch.float64


def system(kind, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    lattice, a, reps = {"cluster": ("fcc", 3.615, (5, 7, 5)), "fcc": ("fcc", 3.615, (6, 6, 6)),
                        "bcc": ("bcc", 2.87, (6, 7, 7))}[kind]
    pos, cell = synth.lattice(lattice, a, reps)
    pos = pos + rng.normal(0.0, 0.07, pos.shape)
    types = np.array([28, 12, 26] if kind == "bcc" else [28], np.int32)
    species = types[rng.integers(0, len(types), len(pos))].astype(np.int32)
    pbc = np.zeros(3, np.int32) if kind == "cluster" else np.ones(3, np.int32)
    return pos, species, cell, pbc


def stage_errors(dp, name, kind, seeds=range(1, 9)):
    """(relative error of D from the node state, rms error of E_i from D in eV)"""
    spec, w = synth.model_weights(name)
    oracle = om.Oracle(spec, w)
    model = dp.Model(synth.pack_blob(spec, w))
    d2 = ref2 = e2 = n = 0.0
    for seed in seeds:
        pos, species, cell, pbc = system(kind, seed)
        p = torch.tensor(pos, dtype=F64, device="cuda")
        s = torch.tensor(species, dtype=torch.int32, device="cuda")
        rows = dp.build_neighbors(p, cell, pbc, 6.0)   # the stages read them again
        e, _, _ = model.compute_energy_forces(p, s, cell, pbc, 6.0, *rows)
        node, desc, _ = model.debug_stages(len(pos))
        torch.cuda.synchronize()
        node, desc = node.cpu().double(), desc.cpu().double()
        M0, M1 = torch.sqrt(0.25 + node[:, 0]), torch.sqrt(0.25 + node[:, 1])
        X, at = [], 2
        for l, c in enumerate(oracle.C[: spec.L + 1]):
            k = (2 * l + 1) * c
            X.append(node[:, at: at + k].reshape(len(pos), 2 * l + 1, c)
                     / (M0 if l == 0 else M1)[:, None, None])
            at += k
        D = oracle.descriptor({"X": X, "M0": M0, "M1": M1}, species)[1]
        E = oracle.mlp_energy(desc, species)
        d2 += float(((desc - D) ** 2).sum())
        ref2 += float((D ** 2).sum())
        e2 += float(((e.cpu() - E) ** 2).sum())
        n += len(pos)
    return (d2 / ref2) ** 0.5, (e2 / n) ** 0.5


@pytest.fixture(scope="module")
def dp():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_19041_amd as m
    m.library()
    return m


@pytest.mark.parametrize("name,kind,bound", [
    ("small", "cluster", 1.985e-7), ("nano", "cluster", 1.039e-7), ("mini", "bcc", 0.785e-7),
    ("neo", "cluster", 1.283e-7), ("air", "cluster", 1.748e-7), ("full", "bcc", 1.469e-7),
    ("plus_l4", "cluster", 2.236e-7)])
def test_readout_from_the_node_state(dp, name, kind, bound):
    error = stage_errors(dp, name, kind)[0]
    print(f"{name} {kind}: {error:.3e} of |D|", flush=True)
    assert error <= 1.05 * bound


@pytest.mark.parametrize("name,kind,bound", [
    ("small", "cluster", 9.42e-8), ("nano", "bcc", 6.80e-9), ("mini", "cluster", 4.08e-8),
    ("neo", "bcc", 1.911e-8), ("air", "fcc", 7.02e-9), ("air", "cluster", 8.11e-8),
    ("full", "fcc", 8.21e-9), ("full", "bcc", 2.284e-8), ("full", "cluster", 1.115e-7),
    ("plus_l4", "fcc", 8.84e-9), ("plus_l4", "cluster", 1.066e-7)])
def test_mlp_from_the_descriptor(dp, name, kind, bound):
    error = stage_errors(dp, name, kind)[1]
    print(f"{name} {kind}: {error:.3e} eV", flush=True)
    assert error <= 1.03 * bound


def gradient_errors(dp, name, kind, seeds=(1, 2, 3)):
    """Relative errors of dE/dD from the descriptor: this library's, plain float32's."""
    spec, w = synth.model_weights(name)
    oracle = om.Oracle(spec, w)
    model = dp.Model(synth.pack_blob(spec, w))

    def plain(D, dtype):   # the MLP and its adjoint with torch's products
        th = {k: torch.tensor(v, dtype=dtype, device="cuda") for k, v in w.items()
              if k.startswith(("Theta", "b1", "b2", "b3", "w_head"))}
        h, pre = D.to(dtype), []
        for t in (1, 2, 3):
            pre.append(h @ th[f"Theta{t}"] + th[f"b{t}"])
            out = torch.nn.functional.silu(pre[-1])
            h = out + h if t > 1 else out
        g = th["w_head"].reshape(1, -1).expand(len(D), -1)
        for t in (3, 2, 1):
            s = torch.sigmoid(pre[t - 1])
            p = (g * s * (1 + pre[t - 1] * (1 - s))) @ th[f"Theta{t}"].T
            g = g + p if t > 1 else p
        return g

    ours = theirs = ref2 = 0.0
    for seed in seeds:
        pos, species, cell, pbc = system(kind, seed)
        p = torch.tensor(pos, dtype=F64, device="cuda")
        s = torch.tensor(species, dtype=torch.int32, device="cuda")
        rows = dp.build_neighbors(p, cell, pbc, 6.0)
        model.compute_energy_forces(p, s, cell, pbc, 6.0, *rows)
        desc = model.debug_stages(len(pos))[1]
        ref = plain(desc, F64)
        if seed == seeds[0]:   # the reference itself against the oracle
            d = desc[:5].cpu().double().requires_grad_()
            oracle.mlp_energy(d, species[:5]).sum().backward()
            assert torch.allclose(d.grad, ref[:5].cpu(), rtol=1e-10, atol=1e-12)
        ours += float(((model.debug_gradient(len(pos)) - ref) ** 2).sum())
        theirs += float(((plain(desc, torch.float32) - ref) ** 2).sum())
        ref2 += float((ref ** 2).sum())
    return (ours / ref2) ** 0.5, (theirs / ref2) ** 0.5


@pytest.mark.parametrize("name", ["small", "nano", "mini", "neo", "air", "full", "plus_l4"])
@pytest.mark.parametrize("kind", ["fcc", "cluster"])
def test_mlp_gradient_from_the_descriptor(dp, name, kind):
    """The split float16 products of the input gradient against torch's float32 ones."""
    ours, theirs = gradient_errors(dp, name, kind)
    print(f"{name} {kind}: {ours:.3e} of |dE/dD|, plain float32 {theirs:.3e}", flush=True)
    assert ours <= theirs


def pair_errors(dp, name, lo, hi, n=400):
    """(rms error of E_i in eV, relative error of F) of pairs lo to hi apart."""
    spec, w = synth.model_weights(name)
    model = dp.Model(synth.pack_blob(spec, w))
    rng = np.random.default_rng(5)
    u = rng.normal(size=(n, 3))
    u *= (rng.uniform(lo, hi, n) / np.linalg.norm(u, axis=1))[:, None]
    centre = np.stack(np.meshgrid(*[np.arange(8) * 20.0 + 10.0] * 3), -1).reshape(-1, 3)[:n]
    pos = np.stack([centre, centre + u], 1).reshape(-1, 3)
    species = np.tile(np.array([7, 0], np.int32), n)
    cell, pbc = np.eye(3) * 200.0, np.zeros(3, np.int32)
    p, s = torch.tensor(pos, device="cuda"), torch.tensor(species, device="cuda")
    rows = dp.build_neighbors(p, cell, pbc, 6.0)
    e, f, _ = model.compute_energy_forces(p, s, cell, pbc, 6.0, *rows)
    ref_e, ref_f = om.Oracle(spec, w).energy_forces(pos, species, cell, pbc)
    return (float(np.sqrt(((e.cpu().numpy() - ref_e) ** 2).mean())),
            float(np.linalg.norm(f.cpu().numpy() - ref_f) / np.linalg.norm(ref_f)))


@pytest.mark.parametrize("name,lo,hi,bound", [
    ("mini", 0.85, 1.1, 3.54e-6), ("mini", 1.3, 2.0, 2.92e-6), ("mini", 2.3, 3.0, 2.95e-6),
    ("air", 0.85, 1.1, 3.17e-6), ("air", 1.3, 2.0, 3.17e-6), ("air", 2.3, 3.0, 2.23e-6),
    ("full", 0.85, 1.1, 6.70e-6), ("full", 1.3, 2.0, 3.87e-6), ("full", 2.3, 3.0, 1.318e-6)])
def test_forces_of_pairs(dp, name, lo, hi, bound):
    """On the folded tables.  The bounds are errors with c2, c3 rounded to float16
    on rows that run from knot to knot, where the slope feels them twice as much as
    on rows around a knot; next to them stand the float32 roundings of the edge."""
    error = pair_errors(dp, name, lo, hi)[1]
    print(f"{name} {lo}-{hi} A: {error:.3e} of |F|", flush=True)
    assert error <= 0.8 * bound


def envelope_errors(dp, name, kind, seed=1):
    """Relative rms errors of sum chi^2 and sum chi^4 from the positions."""
    model = dp.Model(synth.pack_blob(*synth.model_weights(name)))
    pos, species, cell, pbc = system(kind, seed)
    n = len(pos)
    p, s = torch.tensor(pos, device="cuda"), torch.tensor(species, device="cuda")
    rows = dp.build_neighbors(p, cell, pbc, 6.0)
    model.compute_energy_forces(p, s, cell, pbc, 6.0, *rows)
    node = model.debug_stages(n)[0].cpu().numpy()
    i = np.repeat(np.arange(n), np.diff(rows[0].cpu().numpy()))
    j, shift = rows[1].cpu().numpy()[:len(i)], dp.unpack_shift(rows[2].cpu().numpy()[:len(i)])
    x = np.linalg.norm(pos[j] + shift @ cell - pos[i], axis=1) / 6.0
    chi = (1 - x) ** 4 * (1 + 4 * x + 10 * x ** 2 + 20 * x ** 3 + 35 * x ** 4)
    ref = np.stack([np.bincount(i, chi ** k, n) for k in (2, 4)], 1)
    return np.sqrt(((node[:, :2] / ref - 1) ** 2).mean(0))


@pytest.mark.parametrize("kind", ["fcc", "cluster", "bcc"])
@pytest.mark.parametrize("name", ["small", "full"])
def test_envelope_sums(dp, name, kind):
    """chi = t^4 p(1 - t) with t to half a unit of 2^-24: four times that, the
    polynomial's roundings and those of rho make about 2^-23.5 of chi at worst, twice
    that of chi^2; over the edges of an atom they average.  With t = 1 - rho / r_c
    from a rounded product it was 2.0e-7 and 3.7e-7."""
    s0, s1 = envelope_errors(dp, name, kind)
    print(f"{name} {kind}: {s0:.3e} of sum chi^2, {s1:.3e} of sum chi^4", flush=True)
    assert s0 <= 2.0**-23 and s1 <= 1.5 * 2.0**-23
