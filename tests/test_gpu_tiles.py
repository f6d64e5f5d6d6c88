"""The distance-sorted tile passes of the mBP descriptor and its adjoint at
the sizes where their index arithmetic turns: structures of 1 to 193 atoms
that all lie within the cutoff of each other, so that an atom has 0, 1, 7, 8,
9, ... up to the limit of 192 neighbors (blocks of eight and their
remainders, one and two staging rounds of 64, the longer rows), for one, two
and several species (one species-pair block per wave, or one per half), each
angular shape's register layout and each number of waves per atom.  Then
grids whose centres are not in order, for the screening of radius terms.
Against the FP64 oracle: descriptors at their bar, forces at the force bar
relative to the largest force of these dense structures.
"""
import os

import numpy as np
import pytest

import oracle
from paper_2305_11805_amd import nnpot, synth

from helpers import E_TOL, F_TOL, descriptor_errors

pytestmark = pytest.mark.gpu

SIZES = (1, 2, 8, 9, 10, 16, 17, 18, 24, 25, 33, 40, 64, 65, 66, 72, 73, 81, 128, 129, 137, 190, 193)


def dense_batch(S, seed, side=3.4):
    rng = np.random.Generator(np.random.PCG64(seed))
    systems = []
    for m in SIZES:
        k = int(np.ceil(m ** (1 / 3)))
        site = rng.permutation(k ** 3)[:m]
        grid = np.stack([site // (k * k), site // k % k, site % k], 1) + 0.5
        pos = (grid + rng.uniform(-0.25, 0.25, (m, 3))) * (side / k)
        systems.append(synth.single(pos, rng.integers(0, S, m)))
    return synth.concat(systems)


def check(s, p, plans, seed):
    nl = oracle.neighbors_brute(s, p.rc)
    G_ref = oracle.descriptors(p, s, nl)
    scale = float(np.sqrt(p.dim) / np.sqrt(np.mean(np.sum(G_ref * G_ref, axis=1))))
    model = synth.random_model(p.n_species, p.dim, [64, 32], seed, in_scale=scale)
    Es_ref, _, F_ref = oracle.energy_forces(p, model, s, nl)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    f_max = max(1.0, float(np.abs(F_ref).max()))
    n_c = np.diff(s.atom_ptr)
    try:
        for plan in plans:
            os.environ["NNPOT_PLAN"] = plan
            rel = descriptor_errors(pot.descriptors().cpu().numpy(), G_ref)
            Es, _, F = [t.cpu().numpy() for t in pot.energy_forces()]
            e = float(np.max(np.abs(Es - Es_ref) / n_c))
            f = float(np.abs(F - F_ref).max()) / f_max
            print(f"[tiles] S {p.n_species} {p.n_theta}x{p.n_rs_ang} plan {plan}: G {rel:.2e} E/atom {e:.2e} "
                  f"F {f:.2e} of {f_max:.1f}", flush=True)
            assert rel <= 1.0 and e <= E_TOL and f <= F_TOL
        nnpot.nn_check(pot.nl)
    finally:
        os.environ.pop("NNPOT_PLAN", None)


@pytest.mark.parametrize("S,nt,nq,zeta", [(1, 8, 8, 50), (2, 8, 8, 50), (3, 8, 4, 50), (4, 8, 8, 50), (5, 4, 4, 7),
                                          (1, 16, 8, 50), (3, 16, 8, 50), (2, 4, 8, 12), (1, 16, 4, 50)])
def test_neighbor_counts(S, nt, nq, zeta):
    check(dense_batch(S, 8000 + S), synth.mbp_params(S, 6.0, 16, nt, nq, zeta=float(zeta)),
          ("1,1,8", "2,2,8", "4,4,8"), 80 + S)


@pytest.mark.parametrize("S", [1, 3])
@pytest.mark.parametrize("eta", [0.0, 12.0, 60.0])
def test_centres_in_any_order(S, eta):
    p = synth.mbp_params(S, 6.0, 20, 8, 8, eta_rad=eta, eta_ang=eta)
    rng = np.random.Generator(np.random.PCG64(81))
    p.rs_ang, p.rs_rad = rng.permutation(p.rs_ang), rng.permutation(p.rs_rad)
    s = synth.bulk_system(rng, 240, 0.09, 1.2, [240 // S] * S)
    check(s, p, ("1,1,8", "2,2,8"), 81)
