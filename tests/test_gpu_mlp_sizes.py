"""The FP32 row-block MLP (plan value 1) on both sides of the atom count where
its blocks go from 16 to 64 atoms (12288): the same network on the same
descriptors must give the same energies and forces as the other launch of
it (plan value 4) within FP32 summation noise, 1e-5 of the largest value, and
meet the bars against the FP64 oracle on sampled atoms."""
import os

import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

from helpers import E_TOL, F_TOL, oracle_sampled_forces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,S", [([64, 32], 2), ([128, 128], 1), ([128, 128], 4)])
@pytest.mark.parametrize("n", [12287, 12288, 12353])
def test_block_sizes(n, hidden, S):
    rng = np.random.Generator(np.random.PCG64(9000 + n))
    counts = [n // S] * S
    counts[0] += n - sum(counts)
    s = synth.bulk_system(rng, n, 0.09, 1.2, counts)
    p = synth.mbp_params(S, 4.5, 16, 8, 4)
    model = synth.random_model(S, p.dim, hidden, 92, in_scale=3.0)
    w = synth.Workload("", s, p, model, 92)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    got = {}
    try:
        for m in (1, 4):
            os.environ["NNPOT_PLAN"] = f"1,1,{m}"
            got[m] = [t.cpu().numpy() for t in pot.energy_forces()]
    finally:
        os.environ.pop("NNPOT_PLAN", None)
    nnpot.nn_check(pot.nl)
    for a, b in zip(got[1][1:], got[4][1:]):
        assert np.abs(a - b).max() <= 1e-5 * np.abs(b).max()
    targets = rng.integers(0, n, 6)
    rows, E_rows, F = oracle_sampled_forces(w, targets)
    e = float(np.abs(got[1][1][rows] - E_rows).max())
    f = float(np.abs(got[1][2][targets] - F).max())
    print(f"[mlp sizes] {n} {hidden} S {S}: E/atom {e:.2e} F {f:.2e}", flush=True)
    assert e <= E_TOL and f <= F_TOL
