"""Which kernel an FP32 MLP plan takes: NNPOT_PLAN's m = 1 the row blocks at any
size, so that small systems can check them against the FP64 oracle (here the
256-128 shape: energies, forces, the weight gradient, the same bits on every
run), and the default rules blocks of 16 atoms up to 8192."""
import json
import os
import re

import numpy as np
import pytest

import oracle
from paper_2305_11805_amd import nnpot, synth

from helpers import E_TOL, F_TOL

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class plan:
    def __init__(self, value):
        self.value = value

    def __enter__(self):
        os.environ["NNPOT_PLAN"] = self.value

    def __exit__(self, *a):
        os.environ.pop("NNPOT_PLAN", None)


def bulk(n, S, hidden, act="gaussian", seed=620):
    rng = np.random.Generator(np.random.PCG64(seed + n))
    counts = [n // S] * S
    counts[0] += n - sum(counts)
    s = synth.bulk_system(rng, n, 0.09, 1.2, counts)
    p = synth.mbp_params(S, 4.5, 16, 8, 4)
    return s, p, synth.random_model(S, p.dim, hidden, 99, act=act, in_scale=3.0)


@pytest.mark.parametrize("n", [701, 8192, 8193])
@pytest.mark.parametrize("hidden,tile", [([64, 32], 4), ([128, 128], 4), ([256, 128], 8)])
def test_forced_and_default_kernels(hidden, tile, n):
    s, p, model = bulk(n, 2, hidden)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    nnpot.nn_autotune_reset()
    default = pot.energy_forces()[1].clone()
    f, a, m = pot.launch_plan()
    assert m == 1
    with plan(f"{f},{a},{tile}"):
        tiles = pot.energy_forces()[1].clone()
    with plan(f"{f},{a},1"):
        rows = pot.energy_forces()[1].clone()
    nnpot.nn_check(pot.nl)
    assert (default == (tiles if n <= 8192 else rows)).all()
    assert not (rows == tiles).all()  # other instructions, other rounding
    assert float((rows - tiles).abs().max()) <= 1e-5 * float(tiles.abs().max())


@pytest.mark.parametrize("act", ["gaussian", "tanh"])
@pytest.mark.parametrize("S,n", [(1, 432), (2, 701)])
def test_256_128_row_blocks_match_oracle(S, n, act):
    s, p, model = bulk(n, S, [256, 128], act)
    nl = oracle.neighbors_cells(s, p.rc)
    Es_ref, _, F_ref = oracle.energy_forces(p, model, s, nl)
    T = synth.energy_targets(7, s.n_structs)
    _, Es_l, flat = oracle.energy_loss_grad(p, model, s, nl, T)
    ref = oracle.unflatten_grads(model, flat)
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    with plan("1,1,1"):
        runs = []
        for _ in range(2):
            Es, _, F = [t.cpu().numpy().copy() for t in pot.energy_forces()]
            _, g = pot.grad(2.0 * (Es_l - T) / s.n_structs, positions=False)
            runs.append([Es, F] + [t.cpu().numpy().copy() for net in g for pair in net for t in pair])
    nnpot.nn_check(pot.nl)
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
    e = float(np.abs(Es - Es_ref).max()) / s.n_atoms
    f = float(np.abs(F - F_ref).max())
    worst = 0.0
    for r, g in zip((t for net in ref for pair in net for t in pair), runs[0][2:]):
        worst = max(worst, np.abs(g.reshape(r.shape) - r).max() / max(np.abs(r).max(), 1e-12))
    print(f"[mlp plans] 256-128 {act} S {S}: E/atom {e:.2e} F {f:.2e} gradient {worst:.2e}", flush=True)
    assert e <= E_TOL and f <= F_TOL and worst <= 1e-4


@pytest.mark.parametrize("hidden", [[64, 32], [128, 128], [256, 128]])
def test_tuning_below_the_row_blocks(hidden):
    """Up to 8192 atoms plan value 1 is the tile kernel's 4 waves (8 for
    256-128): tuning does not weigh that kernel against itself, and its choice
    holds for the whole class."""
    rng = np.random.Generator(np.random.PCG64(621))
    s = synth.bulk_system(rng, 701, 0.09, 1.2, [701])
    p = synth.mbp_params(1, 4.5, 16, 8, 4)
    pot = nnpot.Potential(s, p, synth.random_model(1, p.dim, hidden, 99, in_scale=3.0))
    pot.build_neighbors()
    try:
        for _ in range(4):
            assert pot.autotune()[2] in {64: (1,), 128: (1, 8), 256: (1, 4)}[hidden[0]]
    finally:
        nnpot.nn_autotune_reset()


@pytest.mark.parametrize("before", ["absent", "current", "other", "unnamed"])
def test_plan_file_names_its_kernels(before, tmp_path, monkeypatch):
    """What nn_autotune writes: plans of other kernels go, the same kernels' and
    those of a file that names none stay, and such a file stays without a name."""
    own = int(re.search(r"#define NN_PLAN_KERNELS (\d+)", open(os.path.join(ROOT, "include", "nnpot.h")).read()).group(1))
    path = tmp_path / "plans.json"
    entry = {"key": [20, 1, 1, 8, 4, 16, 64, 32, 0], "plan": [1, 1, 4]}
    first = {"current": [{"kernels": own}], "other": [{"kernels": own + 1}], "unnamed": []}
    if before != "absent":
        path.write_text("[\n" + ",\n".join(json.dumps(e) for e in first[before] + [entry]) + "\n]\n")
    monkeypatch.setenv("NN_AUTOTUNE_CACHE", str(path))
    s, p, model = bulk(432, 1, [64, 32])
    nnpot.nn_autotune_reset()
    pot = nnpot.Potential(s, p, model)
    pot.build_neighbors()
    pot.autotune()
    nnpot.nn_autotune_reset()
    out = json.loads(path.read_text())
    assert (out[0] == {"kernels": own}) == (before != "unnamed")
    assert (entry in out) == (before in ("current", "unnamed"))
    assert sum("key" in e for e in out) == 1 + (before in ("current", "unnamed"))
