"""Charge equilibration at the edges of the solver's waves: structures of 1 to
64 atoms on both sides of the 32 atoms where another launch takes over, and of
the 4 x 64 and 6 x 64 pairs a wave deals to its lanes in one go, in an order
that mixes both launches' structures.  Energies, charges and forces against
the FP64 oracle at the bars of the charge equilibration's other tests."""
import numpy as np
import pytest

from oracle import qeq as oqeq
from paper_2305_11805_amd import nnpot, synth

from helpers import E_TOL, F_TOL

pytestmark = pytest.mark.gpu

Q_TOL = 1e-5


@pytest.mark.parametrize("sizes", [[1, 2, 33, 3, 64], [23, 24, 28, 29], [31, 32, 33, 63, 64], [32], [64]])
def test_structure_sizes(sizes):
    w, _ = synth.qeq_clusters(1)
    rng = np.random.Generator(np.random.PCG64(700 + sum(sizes)))
    box = 16.0
    s = synth.concat([synth.single(synth.rsa_cluster(rng, n, box, 2.2), rng.integers(0, 2, n), cell=np.eye(3) * box)
                      for n in sizes])
    Qc = rng.integers(-1, 2, len(sizes)).astype(float)
    Es_r, q_r, F_r, _ = oqeq.energy_forces_qeq(w.params, w.model, s, Qc, w.extra["sigma"])
    pot = nnpot.Potential(s, w.params, w.model)
    pot.build_neighbors()
    E, q, F = [t.cpu().numpy() for t in pot.energy_forces_qeq(Qc, w.extra["sigma"])]
    nnpot.nn_check(pot.nl)
    e = np.max(np.abs(E - Es_r) / np.diff(s.atom_ptr))
    dq, f = np.abs(q - q_r).max(), np.abs(F - F_r).max()
    print(f"[qeq sizes] {sizes}: E/atom {e:.2e}  q {dq:.2e}  F {f:.2e}", flush=True)
    assert e <= E_TOL and dq <= Q_TOL and f <= F_TOL
