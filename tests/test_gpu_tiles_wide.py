"""The tile forward of 16x8 bins with two waves an atom, where the atom count
chooses whether they share the triplets (up to 1536 atoms), or the angle terms
with four (up to 2048) or five waves per SIMD: the dense structures of
test_gpu_tiles.py and further ones that make up each count, for one, two and
several species and both exponents' code, against the FP64 oracle at its bars."""
import numpy as np
import pytest

from paper_2305_11805_amd import synth

from test_gpu_tiles import check, dense_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,S,zeta", [(1536, 1, 50), (1537, 1, 50), (1536, 2, 7), (2048, 2, 50), (2049, 1, 7),
                                      (2049, 2, 50), (2048, 3, 50)])
def test_sixteen_by_eight(n, S, zeta):
    s = dense_batch(S, 8100 + S)
    more = dense_batch(S, 8200 + S)
    rng = np.random.Generator(np.random.PCG64(8300 + n))
    parts, left = [s], n - s.n_atoms
    for a, b in zip(more.atom_ptr, more.atom_ptr[1:]):  # whole structures while they fit
        if b - a <= left:
            parts.append(synth.single(more.pos[a:b], more.species[a:b]))
            left -= int(b - a)
    parts += [synth.single(np.zeros((1, 3)), rng.integers(0, S, 1)) for _ in range(left)]
    s = synth.concat(parts)
    assert s.n_atoms == n
    check(s, synth.mbp_params(S, 6.0, 16, 16, 8, zeta=float(zeta)), ("2,2,8",), 86 + S)
