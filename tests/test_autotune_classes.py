"""The shape classes of tuned plans on the host: the FP32 MLP's kernel changes past
8192 atoms, so a plan tuned on one side of it is not used on the other.  And the
kernels that a plan file names."""
import json
import os
import re

import pytest

from test_autotune_cache import KEY, QUERY, ROOT, built, write  # noqa: F401
import test_autotune_cache

CLASSES = [(4095, 12), (4096, 13), (8191, 13), (8192, 13), (8193, 14), (16383, 14), (16384, 15), (32768, 16)]


@pytest.mark.parametrize("n,n_log2", CLASSES)
def test_class_of_an_atom_count(n, n_log2, tmp_path, monkeypatch):
    monkeypatch.setattr(test_autotune_cache, "QUERY",
                        QUERY.replace("nn_system(192,", f"nn_system({n},").replace("nn_nlist(4000,", f"nn_nlist({20 * n},"))
    path = str(tmp_path / "plans.json")
    lines = []
    for b in range(1, 20):
        key = [b] + KEY[1:]
        plan = [2, 4, 8] if b == n_log2 else [1, 1, 4]
        lines.append('{"key": %s, "plan": %s}' % (json.dumps(key), json.dumps(plan)))
    write(path, lines)
    assert test_autotune_cache.query({"NN_AUTOTUNE_CACHE": path})["plan"] == [2, 4, 8]


@pytest.mark.parametrize("kernels,used", [(0, True), (1, False), (-1, False)])
def test_plans_of_other_kernels_are_not_used(kernels, used, tmp_path):
    """A file names the kernels its plans were tuned on, as an offset from this
    library's here."""
    path = str(tmp_path / "plans.json")
    own = int(re.search(r"#define NN_PLAN_KERNELS (\d+)", open(os.path.join(ROOT, "include", "nnpot.h")).read()).group(1))
    write(path, ['{"kernels": %d}' % (own + kernels), '{"key": %s, "plan": [2, 4, 8]}' % json.dumps(KEY)])
    assert test_autotune_cache.query({"NN_AUTOTUNE_CACHE": path})["plan"] == ([2, 4, 8] if used else [0, 0, 1])
