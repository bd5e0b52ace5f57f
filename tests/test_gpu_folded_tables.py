"""The folded radial tables over their whole range, at every profile's row
layout.

Isolated dimers of two species, at distances from 1 A to just inside the
cutoff, on knots of the table (multiples of 0.002 A) and between them.  The
same dimers beside single atoms of four more species run on the separable
float32 tables, since six species are not folded.  The folded coefficients
are the separable ones combined in float64 and rounded once, with c2, c3 in
float16.  A model is folded only while that moves the value of a channel by
less than its float32 rounding and its slope by less than 2^-14, so between
the two paths E_i may differ by the float32 rounding of the few terms that
dominate it, held to eight units of 2^-23 of the energies' scale, and a force
by 2^-14 of the forces' scale.  Both lie within 1e-5 and 1e-4 of these scales
of the float64 model.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import model as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["nano", "mini", "neo", "air", "plus", "plus_l4"])
def test_dimers_over_the_table_range(name):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2608_19041_amd as dp
    spec, w = synth.model_weights(name)
    rng = np.random.Generator(np.random.PCG64(23))
    dist = np.concatenate([[1.0, 1.001, 2.5, 4.0, 5.9, 5.998, 5.9985, 5.9999999],
                           rng.uniform(1.0, 6.0, 40)])
    u = rng.normal(size=(len(dist), 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    centre = np.stack(np.meshgrid(*[np.arange(4) * 20.0 + 10.0] * 3), -1).reshape(-1, 3)
    pos = np.empty((2 * len(dist), 3))
    pos[0::2] = centre[:len(dist)]
    pos[1::2] = pos[0::2] + dist[:, None] * u
    species = np.tile(np.array([29, 8, 8, 8, 29, 29], np.int32), len(pos))[:len(pos)]
    extra = centre[len(dist):len(dist) + 4]
    cell, pbc = np.eye(3) * 100.0, np.zeros(3, np.int32)

    def run(p, sp):
        model = dp.Model(synth.pack_blob(spec, w))
        assert model.info["fold_words"] == 3
        p = torch.tensor(p, dtype=torch.float64, device="cuda")
        sp = torch.tensor(sp, dtype=torch.int32, device="cuda")
        e, f, _ = model.compute_energy_forces(p, sp, cell, pbc, 6.0,
                                              *dp.build_neighbors(p, cell, pbc, 6.0))
        return e.cpu().numpy()[:len(pos)], f.cpu().numpy()[:len(pos)]

    e_f, f_f = run(pos, species)
    e_s, f_s = run(np.concatenate([pos, extra]),
                   np.concatenate([species, np.array([6, 13, 26, 28], np.int32)]))
    ref_e, ref_f = om.Oracle(spec, w).energy_forces(pos, species, cell, pbc)
    se, sf = max(1.0, np.abs(ref_e).max()), max(1.0, np.abs(ref_f).max())
    assert np.abs(e_f - e_s).max() <= 8 * 2.0**-23 * se
    assert np.abs(f_f - f_s).max() <= 2.0**-14 * sf
    for e, f in ((e_f, f_f), (e_s, f_s)):
        assert np.abs(e - ref_e).max() < 1e-5 * se and np.abs(f - ref_f).max() < 1e-4 * sf
