"""The per-structure energy sums around the edges of their block (one wave up
to 64 atoms, 256 threads, 16 terms a thread in flight): structures of isolated
atoms, whose energies differ by species only.  The sum of the call's own
per-atom energies in FP64, in another order, to 1e-12 of its size (n terms
of 2^-53 relative rounding each, n at most 8300)."""
import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1, 63, 64, 65, 0, 127, 128, 129, 255, 256, 257], [4095, 4096, 4097, 1], [8300]])
@pytest.mark.parametrize("forces", [False, True])
def test_energy_sums(sizes, forces):
    rng = np.random.Generator(np.random.PCG64(600 + sizes[0]))
    parts = []
    for n in sizes:
        g = np.arange(n)
        x = np.stack([g % 32, g // 32 % 32, g // 1024], axis=1) * 10.0 + 5.0
        parts.append(synth.single(x, rng.integers(0, 4, n), cell=np.eye(3) * 400.0))
    p = synth.mbp_params(4, 4.0, 16, 8, 4)
    pot = nnpot.Potential(synth.concat(parts), p, synth.random_model(4, p.dim, [64, 32], 94, in_scale=3.0))
    pot.build_neighbors()
    Es, E_atom = [t.cpu().numpy().astype(np.float64) for t in pot.energy_forces(forces=forces)[:2]]
    nnpot.nn_check(pot.nl)
    at = np.concatenate([[0], np.cumsum(sizes)])
    ref = np.array([E_atom[a:b].sum() for a, b in zip(at, at[1:])])
    size = np.array([np.abs(E_atom[a:b]).sum() for a, b in zip(at, at[1:])])
    assert np.all(np.abs(Es - ref) <= 1e-12 * size)
