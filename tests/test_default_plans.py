"""The default launch rules on the host (nn_launch_plan reads no device memory, so
the structs carry placeholder device pointers): waves per atom of the mBP passes
by the angular shape, the species and the atom count."""
import ctypes as C
import os

import pytest

from paper_2305_11805_amd import nnpot, synth


@pytest.fixture(autouse=True)
def built(monkeypatch):
    if not os.path.exists(nnpot.LIB_PATH):
        pytest.skip("libnnpot.so is not built")
    monkeypatch.delenv("NNPOT_PLAN", raising=False)
    monkeypatch.delenv("NN_AUTOTUNE_CACHE", raising=False)
    nnpot.nn_autotune_reset()


def default_plan(S, nt, nq, n, per_atom=60):
    params, keep = nnpot.make_params(synth.mbp_params(S, 5.0, 16, nt, nq))
    a = [C.c_void_p(0x10000 * k) for k in range(1, 16)]
    s = nnpot.nn_system(n, 1, a[0].value, a[1].value, a[2].value, a[3].value, a[4].value)
    nl = nnpot.nn_nlist(per_atom * n, a[5].value, a[6].value, a[7].value, a[8].value, a[9].value, a[10].value, None, 5.0)
    m = nnpot.nn_model()
    m.n_species = S
    D = nnpot.nn_descriptor_dim(params)
    for q in m.mlp[:S]:
        q.n_layers = 3
        q.width[0], q.width[1], q.width[2], q.width[3] = D, 64, 32, 1
        q.act[0] = q.act[1] = nnpot.ACT["gaussian"]
        q.act[2] = nnpot.ACT["linear"]
        for l in range(3):
            q.W[l], q.b[l] = a[11].value, a[12].value
    return nnpot.nn_launch_plan(s, nl, params, m, 0)


# 16x8 bins hold few waves per SIMD: at 2048 atoms two waves an atom fill one
# round, a few more start another, and many are best served by two
@pytest.mark.parametrize("n,waves", [(16, (4, 4)), (768, (4, 4)), (1024, (2, 4)), (1856, (2, 4)), (1857, (2, 2)),
                                     (2048, (2, 2)), (2049, (2, 4)), (2560, (2, 4)), (2561, (2, 2)), (4096, (2, 2)), (12288, (2, 2)), (12289, (1, 2)), (16384, (1, 2))])
def test_sixteen_angle_terms(n, waves):
    assert default_plan(1, 16, 8, n) == (*waves, 1)


@pytest.mark.parametrize("nt,nq,last", [(4, 4, 4096), (4, 8, 4096), (8, 4, 4096), (8, 8, 8192)])
@pytest.mark.parametrize("S", [1, 2, 4])
def test_where_four_adjoint_waves_end(S, nt, nq, last):
    assert default_plan(S, nt, nq, last)[1] == 4 and default_plan(S, nt, nq, last + 1)[1] == 2


def test_several_species_of_sixteen_angle_terms():
    assert [default_plan(4, 16, 8, n)[0] for n in (16, 600, 1024, 8192)] == [2] * 4
