"""Forces that are not finite from the distance-sorted tile passes, which leave
out the radius terms that no neighbor feels: they are where the packed passes,
which evaluate every term, put them."""
import os

import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


def run(pot, plan):
    os.environ["NNPOT_PLAN"] = plan
    try:
        return [t.cpu().numpy().copy() for t in pot.energy_forces()[1:]]
    finally:
        os.environ.pop("NNPOT_PLAN", None)


@pytest.mark.parametrize("wpa", [1, 2, 4])
@pytest.mark.parametrize("S", [1, 2])
@pytest.mark.parametrize("bin_", ["radial", "angular"])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_weight(value, bin_, S, wpa):
    """A first-layer weight that is not finite makes dE/dG of its bin so for
    every atom, and the forces of all its neighbors, near the bin or not."""
    rng = np.random.Generator(np.random.PCG64(610))
    s = synth.clusters_system(rng, [12] * 40, lambda n: (n / 0.05) ** (1 / 3), 0.9, S)
    p = synth.mbp_params(S, 4.6, 16, 8, 4, eta_rad=16.0, eta_ang=12.0)
    model = synth.random_model(S, p.dim, [64, 32], 98, act="linear", in_scale=3.0)
    # the bin of the smallest radius: far from most neighbors
    model[0][2][0][3, 0 if bin_ == "radial" else S * p.n_rad] = value
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    ref = run(pot, "0,0,4")[1]
    got = run(pot, f"0,{wpa},4")[1]
    nnpot.nn_check(pot.nl)
    bad = ~np.isfinite(ref)
    print(f"[tiles nonfinite] {bin_} S {S} {wpa} waves: {int(bad.sum())} of {bad.size} not finite", flush=True)
    assert bad.any()
    assert np.array_equal(~np.isfinite(got), bad)
    if not bad.all():
        assert np.abs(got[~bad] - ref[~bad]).max() <= 1e-4 * max(np.abs(ref[~bad]).max(), 1e-30)


@pytest.mark.parametrize("wpa", [1, 2, 4])
def test_lines_without_smoothing(wpa):
    """With eps = 0 the angular term has no derivative where two neighbors and
    the atom lie on a line: chains of 3 to 12 atoms, and the same atoms off it."""
    rng = np.random.Generator(np.random.PCG64(611))
    systems = []
    for n in (3, 9, 12):
        x = np.zeros((n, 3))
        x[:, 0] = 1.25 * np.arange(n)
        systems += [synth.single(x, np.zeros(n, int)), synth.single(x + rng.uniform(-0.2, 0.2, x.shape), np.zeros(n, int))]
    s = synth.concat(systems)
    p = synth.mbp_params(1, 4.6, 16, 8, 4, eps=0.0)
    model = synth.random_model(1, p.dim, [64, 32], 98, in_scale=3.0)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    ref, got = run(pot, "0,0,4"), run(pot, f"{wpa},{wpa},4")
    nnpot.nn_check(pot.nl)
    bad = ~np.isfinite(ref[1]).all(1)
    print(f"[tiles nonfinite] lines, {wpa} waves: {int(bad.sum())} of {bad.size} atoms without a force", flush=True)
    assert np.abs(got[0] - ref[0]).max() <= 1e-5 * np.abs(ref[0]).max()
    assert bad.any() and not bad.all()
    assert np.array_equal(~np.isfinite(got[1]).all(1), bad)
    assert np.abs(got[1] - ref[1])[~bad].max() <= 1e-4 * np.abs(ref[1][~bad]).max()


@pytest.mark.parametrize("wpa", [1, 2, 4])
def test_two_atoms_in_one_place(wpa):
    """A pair at distance zero has radial terms and no direction: energies of a
    dimer are finite, forces and every triplet are not."""
    a = np.array([[1.0, 2.0, 3.0]])
    line = np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 0.0], [1.5, 0.2, 0.1]])
    s = synth.concat([synth.single(np.concatenate([a, a]), np.zeros(2, int)),
                      synth.single(line, np.zeros(3, int)),
                      synth.single(line * 2.0 + np.array([[0.0, 0.0, 0.0], [1.3, 0.0, 0.0], [0.0, 0.0, 0.0]]), np.zeros(3, int))])
    p = synth.mbp_params(1, 4.6, 16, 8, 4)
    model = synth.random_model(1, p.dim, [64, 32], 98, in_scale=3.0)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    ref, got = run(pot, "0,0,4"), run(pot, f"{wpa},{wpa},4")
    nnpot.nn_check(pot.nl)
    assert np.isfinite(ref[0]).any() and not np.isfinite(ref[0]).all() and np.isfinite(ref[1][-3:]).all()
    for a, b in zip(got, ref):
        assert np.array_equal(np.isfinite(a), np.isfinite(b))
        on = np.isfinite(b)
        assert np.abs(a[on] - b[on]).max() <= 1e-4 * np.abs(b[on]).max()
