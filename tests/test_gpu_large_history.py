"""GPU parity of the large-cluster minimiser (L-BFGS history in memory) at the
numbers of stored pairs around its read-ahead and its kept pairs, and at team
sizes with empty slots and wavefronts."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 9, 10])
@pytest.mark.parametrize("shape", [0, 1, 2])
def test_history_in_memory_fp64_bitwise(m, shape):
    sizes = [257, 520, 300]
    off, x = random_starts(sizes, 9500)
    b = lj.ClusterBatch(off)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(m=m, max_iter=14)
    announce(f"history in memory fp64 m={m} shape={shape} sizes={sizes}")
    try:
        lj.set_schedule(lj.SCHED_MIN_LARGE, "fp64", 0, shape)
        r = host_dict(lj.minimize(b, xd, p, "fp64"))
    finally:
        lj.set_schedule(lj.SCHED_MIN_LARGE, "fp64", 0, 1)
    ro = O.minimize(off, x, oracle_params(p))
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status"):
        assert np.array_equal(r[key], ro[key]), key


@pytest.mark.parametrize("n", [257, 511, 513, 960, 961])
def test_large_morse_fp64_bitwise(n):
    off, x = random_starts([n, n - 1], 9600 + n)
    b = lj.ClusterBatch(off, pair="morse", rho=6.0)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(max_iter=6)
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS["morse"], 6.0
    announce(f"large morse fp64 n={n}")
    r = host_dict(lj.minimize(b, xd, p, "fp64"))
    ro = O.minimize(off, x, op)
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status"):
        assert np.array_equal(r[key], ro[key]), key
