"""GPU parity of the FP64 minimiser with helper wavefronts, which the built-in
rule takes for calls of few clusters: every output equals the oracle's bit for
bit, at every size its segments and tiles can be cut at."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu

KEYS = ("xyz", "energy", "gnorm", "iters", "evals", "status")


# one tile (every N up to 64), two tiles (65 .. 128 beside smaller ones), the
# smallest batch; m below and at the history's capacity
@pytest.mark.parametrize("sizes", [list(range(65)), [65, 128, 1, 127, 0, 96, 66, 98, 20, 126, 113],
                                   [20]], ids=["tile1", "tile2", "single"])
@pytest.mark.parametrize("pair,m", [("lj", 10), ("lj", 3), ("lj", 0), ("morse", 10)])
def test_helper_wavefronts_fp64_bitwise(sizes, pair, m):
    off, x = random_starts(sizes, 9100 + len(sizes))
    x = x.copy()
    if len(sizes) > 60 and pair == "lj":
        o = off[40]
        x[:, o + 7] = x[:, o + 30]  # coincident atoms in different segments
        o = off[2]
        x[:, o + 1] = x[:, o] + [1e7, 0.0, 0.0]  # a far-apart pair
    b = lj.ClusterBatch(off, pair=pair, rho=6.0)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(m=m, max_iter=60 if m == 0 else 400)
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS[pair], 6.0
    announce(f"helper wavefronts fp64 {pair} m={m} clusters={b.num} max_n={b.max_n}")
    r = host_dict(lj.minimize(b, xd, p, "fp64"))
    ro = O.minimize(off, x, op)
    for key in KEYS:
        assert np.array_equal(r[key], ro[key], equal_nan=True), key


@pytest.mark.parametrize("m", [0, 2, 10])
def test_two_wavefronts_per_cluster_fp64_bitwise(m):
    """More clusters than four wavefronts each have SIMDs for: two per cluster,
    every N of the class among them, and coincident atoms."""
    sizes = list(range(65)) + [20, 21, 38, 44, 45, 64] * 80
    off, x = random_starts(sizes, 9150)
    x = x.copy()
    o = off[40]
    x[:, o + 7] = x[:, o + 30]
    b = lj.ClusterBatch(off)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(m=m, max_iter=12 if m == 0 else 60)
    announce(f"two wavefronts per cluster fp64 m={m} clusters={b.num} max_n={b.max_n}")
    r = host_dict(lj.minimize(b, xd, p, "fp64"))
    ro = O.minimize(off, x, oracle_params(p))
    for key in KEYS:
        assert np.array_equal(r[key], ro[key], equal_nan=True), key
