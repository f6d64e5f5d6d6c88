"""The grouping of atoms by species at the edges of its waves' stretches (16
waves of 64 atoms) and on both sides of the 16384 atoms where one block gives
way to three launches, species in random order with one of them absent.  The
atoms are isolated, where each gets the energy its species' network gives the
zero descriptor; the reference is the FP64 oracle on one atom per species, at
4e-6 of the larger of its largest energy and 1 (the two hidden layers of 64
and 32 units round to 64 x 6e-8 of sums of order 1 at most)."""
import numpy as np
import pytest

import oracle
from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1025, 8191, 8193, 16383, 16384, 16385])
def test_isolated_atoms(n):
    S = 4
    rng = np.random.Generator(np.random.PCG64(800 + n))
    g = np.arange(n)
    x = np.stack([g % 32, g // 32 % 32, g // 1024], axis=1) * 10.0 + 5.0
    species = rng.choice([0, 1, 3], n)
    p = synth.mbp_params(S, 4.0, 16, 8, 4)
    model = synth.random_model(S, p.dim, [64, 32], 93, in_scale=3.0)
    pot = nnpot.Potential(synth.single(x, species, cell=np.eye(3) * 400.0), p, model)
    pot.build_neighbors()
    E_atom = pot.energy_forces()[1].cpu().numpy()
    nnpot.nn_check(pot.nl)
    alone = synth.concat([synth.single(x[:1], [k], cell=np.eye(3) * 40.0) for k in range(S)])
    ref = oracle.energy_forces(p, model, alone, oracle.neighbors_cells(alone, p.rc))[0]
    assert np.abs(E_atom - ref[species]).max() <= 4e-6 * max(np.abs(ref).max(), 1.0)
