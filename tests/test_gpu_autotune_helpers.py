"""The autotuner and the forms with helper wavefronts, which have no number in the
schedule table: an entry left by a batch of many clusters does not survive tuning
a batch of few, in the table and through the cache."""
import json

import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict, settle, to_dev
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts

pytestmark = pytest.mark.gpu

KEYS = ("xyz", "energy", "gnorm", "iters", "evals", "status")


@pytest.mark.parametrize("n,cls,count", [(38, 0, 8), (98, 1, 8), (38, 0, 700)])
def test_tuning_few_clusters_brings_the_rule_back(tmp_path, n, cls, count):
    off, x = random_starts([n] * count, 9985 + n)
    b, xd = to_dev(off, x)
    kind = lj.SCHED_MIN_CLASS[cls]
    p = lj.lbfgs_params(max_iter=50)
    cache = tmp_path / "sched.json"
    cache.write_text(json.dumps({"fp64": {"min_class": {str(n): {str(cls): 0}}}}))
    announce(f"autotune helpers {count} x LJ{n}")
    settle(None)
    rule = lj.minimize_forms(b, "fp64")[cls]
    assert rule in (16, 17)
    want = host_dict(lj.minimize(b, xd, p, "fp64"))
    try:
        lj.load_schedules(str(cache))
        assert lj.minimize_forms(b, "fp64")[cls] in (0, 32)
        res = lj.autotune(b, xd, "fp64", cache=str(cache))
        assert cls not in res["min_class"]
        assert lj.get_schedule(kind, "fp64", n)[0] == -1
        assert lj.minimize_forms(b, "fp64")[cls] == rule
        lj.load_schedules(str(cache))
        assert lj.minimize_forms(b, "fp64")[cls] == rule
        got = host_dict(lj.minimize(b, xd, p, "fp64"))
    finally:
        lj.set_schedule(kind, "fp64", n, -1)
        lj.set_schedule(lj.SCHED_EVAL, "fp64", n, *lj.eval_shape_default(n))
    for key in KEYS:
        assert np.array_equal(want[key], got[key]), key
