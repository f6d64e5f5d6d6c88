"""The waves per atom of the descriptor tangent: its own default, whatever the
forward pass takes (by default or tuned), and the forward's under NNPOT_PLAN.
Waves change the order of sums, so equal waves give equal bits and others do
not."""
import os

import numpy as np
import pytest
import torch

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


def tangent(pot, v, waves=None):
    if waves is not None:
        os.environ["NNPOT_PLAN"] = f"{waves},{waves},1"
    try:
        return pot.descriptor_tangent(v).clone()
    finally:
        os.environ.pop("NNPOT_PLAN", None)


@pytest.mark.parametrize("S,n,waves", [(1, 432, 4), (1, 1024, 4), (1, 1100, 2), (1, 12000, 2), (1, 17000, 2),
                                       (2, 1000, 4), (2, 12000, 2), (2, 17000, 1), (4, 1000, 2), (4, 2048, 2), (4, 2100, 1)])
def test_default_waves(S, n, waves):
    rng = np.random.Generator(np.random.PCG64(630 + n))
    counts = [n // S] * S
    counts[0] += n - sum(counts)
    s = synth.bulk_system(rng, n, 0.09, 1.2, counts)
    p = synth.mbp_params(S, 4.5, 16, 8, 8)
    pot = nnpot.Potential(s, p, synth.random_model(S, p.dim, [64, 32], 99))
    pot.build_neighbors()
    nnpot.nn_autotune_reset()
    v = torch.tensor(rng.normal(size=(n, 3)).astype(np.float32), device="cuda")
    got = tangent(pot, v)
    for w in (1, 2, 4):
        assert torch.equal(got, tangent(pot, v, w)) == (w == waves), w
    try:
        pot.autotune()
        assert torch.equal(got, tangent(pot, v))
    finally:
        nnpot.nn_autotune_reset()
    nnpot.nn_check(pot.nl)
