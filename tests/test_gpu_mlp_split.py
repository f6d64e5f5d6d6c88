"""The row-block MLP where it runs (12288 atoms and more): its products of
three-part operands against the tile kernel's FP32 instructions (plan values 4
and 8) on the same descriptors.  All fused shapes, descriptor lengths on both
sides of a chunk of 32 (with a remainder of 4 too, and an odd number of
chunks), a species of one atom and one of none, ragged last blocks.  Energies,
forces and the weight gradient, which reads the stored activations, agree to
FP32 summation noise, 1e-5 of the largest value (1e-4 for the gradients, sums
over all atoms).  ReLU's derivative jumps, so its energies only."""
import os

import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


def run(pot, plan, grad):
    os.environ["NNPOT_PLAN"] = plan
    try:
        out = [t.cpu().numpy().copy() for t in pot.energy_forces()]
        alone = pot.energy_forces(forces=False)[1].cpu().numpy()
        assert np.array_equal(out[1], alone, equal_nan=True)
        g = []
        if grad:
            _, layers = pot.grad(np.ones(pot.B), positions=False)
            g = [t.cpu().numpy().copy() for net in layers for pair in net for t in pair]
    finally:
        os.environ.pop("NNPOT_PLAN", None)
    return out, g


@pytest.mark.parametrize("hidden,act,n_rad,S,n", [
    ([64, 32], "gaussian", 4, 1, 12289),     # D 20
    ([64, 32], "tanh", 7, 4, 12288),         # D 188: six chunks, the last of 28
    ([128, 128], "gaussian", 16, 4, 12351),  # D 224: seven chunks
    ([128, 128], "tanh", 4, 1, 12416),       # D 20
    ([256, 128], "gaussian", 12, 3, 12353),  # D 132: five chunks, the last of 4
    ([256, 128], "relu", 16, 1, 12289),      # D 32
])
def test_against_fp32_instructions(hidden, act, n_rad, S, n):
    rng = np.random.Generator(np.random.PCG64(9500 + n))
    counts = [n, 0, 0, 0][:S] if S < 3 else [n // 2, 1, n - n // 2 - 1, 0][:S]
    s = synth.bulk_system(rng, n, 0.09, 1.2, counts)
    p = synth.mbp_params(S, 4.0, n_rad, 4, 4)
    model = synth.random_model(S, p.dim, hidden, 95, act=act, in_scale=3.0)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    got, g = run(pot, "1,1,1", True)
    ref, r = run(pot, "1,1,8" if hidden[0] == 256 else "1,1,4", True)
    nnpot.nn_check(pot.nl)
    assert np.abs(got[1] - ref[1]).max() <= 1e-5 * np.abs(ref[1]).max()
    if act == "relu":
        return
    assert np.abs(got[2] - ref[2]).max() <= 1e-5 * np.abs(ref[2]).max()
    for a, b in zip(g, r):
        assert np.abs(a - b).max() <= 1e-4 * max(np.abs(b).max(), 1e-30)


def test_infinite_weight():
    """An infinite weight gives what FP32 products give: its unit is off
    (Gaussian), or not a number where the descriptor is zero, not everywhere."""
    n = 12300
    rng = np.random.Generator(np.random.PCG64(77))
    s = synth.bulk_system(rng, n, 0.09, 1.2, [n])
    p = synth.mbp_params(1, 4.0, 16, 4, 4)
    model = synth.random_model(1, p.dim, [64, 32], 96, in_scale=3.0)
    model[0][2][0][5, 3] = np.inf
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    got, _ = run(pot, "1,1,1", False)
    ref, _ = run(pot, "1,1,4", False)
    assert np.isfinite(ref[1]).any()
    assert np.array_equal(np.isfinite(got[1]), np.isfinite(ref[1]))
    on = np.isfinite(ref[1])
    assert np.abs(got[1] - ref[1])[on].max() <= 1e-5 * np.abs(ref[1][on]).max()
