"""The row offsets of a list at the edges of their scan: one block up to 8192
atoms, tiles of 1024 beyond (a ragged last one, more than 64 of them), for one
structure and for a batch.  Rows of a chain of atoms 1 A apart with a cutoff
of 2.5 A have two entries at the ends of a structure, three beside them, four
inside (fewer in the shortest), so the offsets are known exactly."""
import numpy as np
import pytest

from paper_2305_11805_amd import nnpot, synth

pytestmark = pytest.mark.gpu


def chain(n):
    return np.stack([np.arange(n) + 5.0, np.full(n, 5.0), np.full(n, 5.0)], axis=1)


def lengths(n):
    k = np.arange(n)
    return np.minimum(k, 2) + np.minimum(n - 1 - k, 2)


@pytest.mark.parametrize("sizes", [[8191], [8192], [8193], [9216], [66563], [7] * 1171, [33] * 2048, [5000, 1, 4000]])
def test_offsets(sizes):
    p = synth.mbp_params(1, 2.5, 4, 4, 4)
    s = synth.concat([synth.single(chain(n), np.zeros(n, np.int32), cell=np.diag([n + 10.0, 10.0, 10.0]))
                      for n in sizes])
    pot = nnpot.Potential(s, p)
    pot.build_neighbors()
    ref = np.concatenate([[0], np.cumsum(np.concatenate([lengths(n) for n in sizes]))])
    assert np.array_equal(pot.offsets.cpu().numpy(), ref)
    nbr = pot.nbr.cpu().numpy()[:ref[-1]]
    row = np.repeat(np.arange(s.n_atoms), np.diff(ref))
    assert np.abs(nbr - row).max() == 2 and np.array_equal(nbr[pot.rev.cpu().numpy()[:ref[-1]]], row)
