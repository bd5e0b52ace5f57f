"""The no-allocation entry point above a few thousand atoms: its own rows between
readout and MLP hold 15,000 atoms at full width (one stretch of the per-atom
stage), and a sparse system of more goes through in two.  Atoms do not depend
on the stretch or the tile they fall into, so the results are those of the
allocating call, bit for bit.
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
