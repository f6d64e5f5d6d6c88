"""Neighbors at exactly equal distances in the distance-sorted tile passes, where
only the place in the row orders them: atoms on the sites of periodic lattices, in
rows of up to 128 entries and in longer ones (with a skin), one and several
species, each number of waves.  Against the FP64 oracle at the bars of these
passes."""
import os

import numpy as np
import pytest

import oracle
from paper_2305_11805_amd import nnpot, synth

from helpers import E_TOL, F_TOL, descriptor_errors

pytestmark = pytest.mark.gpu


def lattice(cells, a, S, seed, basis=((0, 0, 0),)):
    grid = np.stack(np.meshgrid(*[np.arange(cells)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(float)
    pos = np.concatenate([(grid + np.array(b)) * a for b in basis])
    rng = np.random.Generator(np.random.PCG64(seed))
    order = rng.permutation(len(pos))
    return synth.single(pos[order], rng.integers(0, S, len(pos)), cell=np.eye(3) * cells * a, pbc=(1, 1, 1))


@pytest.mark.parametrize("wpa", [1, 2, 4])
@pytest.mark.parametrize("S", [1, 2, 3])
@pytest.mark.parametrize("skin", [0.0, 1.0])
def test_lattices(skin, S, wpa):
    # 1.75 A: 92 neighbors within 5 A, 170 entries within 6 A; and a body-centred one
    for s in (lattice(6, 1.75, S, 640), lattice(5, 2.4, S, 641, basis=((0, 0, 0), (0.5, 0.5, 0.5)))):
        p = synth.mbp_params(S, 5.0, 16, 8, 8)
        model = synth.random_model(S, p.dim, [64, 32], 99, in_scale=0.5)
        pot = nnpot.Potential(s, p, model, skin=skin)
        pot.build_neighbors()
        longest = int(np.diff(pot.neighbor_list_host()["offsets"]).max())
        assert (longest > 128) == (skin > 0), longest
        nl = oracle.neighbors_cells(s, p.rc)
        G_ref = oracle.descriptors(p, s, nl)
        Es_ref, _, F_ref = oracle.energy_forces(p, model, s, nl)
        os.environ["NNPOT_PLAN"] = f"{wpa},{wpa},4"
        try:
            G = pot.descriptors().cpu().numpy()
            Es, _, F = [t.cpu().numpy().copy() for t in pot.energy_forces()]
            again = pot.energy_forces()[2].cpu().numpy()
        finally:
            os.environ.pop("NNPOT_PLAN", None)
        nnpot.nn_check(pot.nl)
        g = descriptor_errors(G, G_ref)
        e = float(np.abs(Es - Es_ref).max()) / s.n_atoms
        f = float(np.abs(F - F_ref).max())
        print(f"[ties] S {S} skin {skin} {wpa} waves, rows of {longest}: G {g:.2f} E/atom {e:.2e} F {f:.2e}", flush=True)
        assert g <= 1.0 and e <= E_TOL and f <= F_TOL * max(1.0, np.abs(F_ref).max())
        assert np.array_equal(F, again)
