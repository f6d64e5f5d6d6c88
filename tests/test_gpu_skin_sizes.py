"""The skin test on both sides of the atom counts where its launch changes
(one block of 256, of 1024 threads, a launch of its own), for one structure and
for a batch: nothing moved, the last or the first atom moved by just less and just
more than half the skin, or one atom at a position that is not a number."""
import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [256], [257], [4096], [4097], [30] * 136, [30] * 137])
def test_rebuild_rule(sizes):
    skin = 0.5
    parts = []
    for n in sizes:
        x = np.stack([np.arange(n) + 5.0, np.full(n, 5.0), np.full(n, 5.0)], axis=1)
        parts.append(synth.single(x, np.zeros(n, np.int32), cell=np.diag([n + 10.0, 10.0, 10.0])))
    s = synth.concat(parts)
    pot = nnpot.Potential(s, synth.mbp_params(1, 2.5, 4, 4, 4), skin=skin, capacity_margin=2.0)
    pot.build_neighbors()
    assert int(pot.meta[3].item()) == 1
    at = s.pos.copy()
    for atom in (s.n_atoms - 1, 0):
        for d, rebuilt in ((0.0, 0), (0.2499, 0), (0.2501, 1)):
            x = at.copy()
            x[atom, 1] += d
            pot.set_positions(x)
            pot.build_neighbors()
            assert int(pot.meta[3].item()) == rebuilt, (atom, d)
            if rebuilt:
                at = x
    x = at.copy()
    x[s.n_atoms // 2, 2] = np.nan
    pot.set_positions(x)
    with pytest.raises(Exception):
        pot.build_neighbors()
