"""The no-allocation entry point above a few thousand atoms: its own rows between
readout and MLP hold 15,000 atoms at full width (one stretch of the per-atom
stage), and a sparse system of more goes through in two.  Atoms do not depend
on the stretch or the tile they fall into, so the results are those of the
allocating call, bit for bit.  A fresh model has room for two species' folded
tables; with more it reads the separable ones until another call needed the room.
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reps,a", [((11, 11, 11), 3.615), ((13, 13, 17), 3.615),
                                    ((14, 16, 18), 6.5)])
def test_noalloc_equals_the_allocating_call(reps, a):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_19041_amd as dp
    model = dp.Model(synth.pack_blob(*synth.model_weights("full")))
    pos, cell = synth.lattice("fcc", a, reps)
    pos = pos + np.random.Generator(np.random.PCG64(3)).normal(0.0, 0.05, pos.shape)
    n = len(pos)
    p = torch.tensor(pos, dtype=torch.float64, device="cuda")
    species = torch.tensor(np.tile([28, 12], n)[:n], dtype=torch.int32, device="cuda")
    args = (p, species, cell, np.ones(3, np.int32), 6.0,
            *dp.build_neighbors(p, cell, np.ones(3, np.int32), 6.5))
    e, f, total = model.compute_energy_forces(*args)
    out = [torch.full_like(x, float("nan")) for x in (e, f, total)]
    model.compute_energy_forces_noalloc(*args, *out)
    for got, want in zip(out, (e, f, total)):
        assert torch.equal(got, want), n


@pytest.mark.parametrize("name", ["mini", "full"])
def test_a_fresh_model_reads_separable_tables_where_it_has_no_room(name):
    """Between the two tables a value may move by its float32 rounding and a slope by
    2^-14 (the condition for folding); the largest energy and force are the scales."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_19041_amd as dp
    blob = synth.pack_blob(*synth.model_weights(name))
    model, other = dp.Model(blob), dp.Model(blob)
    pos, cell = synth.lattice("bcc", 2.87, (5, 6, 7))
    rng = np.random.Generator(np.random.PCG64(4))
    p = torch.tensor(pos + rng.normal(0.0, 0.06, pos.shape), dtype=torch.float64, device="cuda")

    def call(model, kinds, alloc):
        types = np.array([28, 12, 26, 21, 77], np.int32)[:kinds]
        s = torch.tensor(np.resize(types, len(pos)), dtype=torch.int32, device="cuda")
        args = (p, s, cell, np.ones(3, np.int32), 6.0,
                *dp.build_neighbors(p, cell, np.ones(3, np.int32), 6.5))
        if alloc:
            return model.compute_energy_forces(*args)
        out = (torch.full((len(pos),), float("nan"), dtype=torch.float64, device="cuda"),
               torch.full((len(pos), 3), float("nan"), dtype=torch.float64, device="cuda"),
               torch.full((1,), float("nan"), dtype=torch.float64, device="cuda"))
        model.compute_energy_forces_noalloc(*args, *out)
        return out

    for kinds in (1, 2):                      # room from creation: the same bits
        for a, b in zip(call(model, kinds, False), call(other, kinds, True)):
            assert torch.equal(a, b), kinds
    for kinds in (3, 5):
        e, f, _ = call(model, kinds, False)   # no room: separable
        ref_e, ref_f, _ = call(other, kinds, True)
        se, sf = max(1.0, float(ref_e.abs().max())), max(1.0, float(ref_f.abs().max()))
        assert not torch.equal(f, ref_f)
        assert float((e - ref_e).abs().max()) <= 8 * 2.0**-23 * se
        assert float((f - ref_f).abs().max()) <= 2.0**-14 * sf
    call(model, 5, True)
    for kinds in (1, 3, 5):                   # now there is room
        for a, b in zip(call(model, kinds, False), call(other, kinds, True)):
            assert torch.equal(a, b), kinds
