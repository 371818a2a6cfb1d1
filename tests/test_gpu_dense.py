"""GPU parity of the minimiser kernels that run two wavefronts per SIMD with half
of the L-BFGS history in LDS: bit for bit the oracle (FP64), and the FP64 polish
from the recorded switch points (mixed), at the numbers of stored pairs around
the split and at the edges of the size classes."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts, uniform_sizes
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu

# enough clusters that the built-in rule takes these kernels
TWO_WAVES = [65, 128, 127] + list(uniform_sizes(697, 65, 128, 9701))
THREE_WAVES = [129, 192, 191, 13, 70] + list(uniform_sizes(295, 129, 192, 9702))
FOUR_WAVES = [256, 193, 255] + list(uniform_sizes(277, 190, 256, 9703))


@pytest.mark.parametrize("sizes", [TWO_WAVES, THREE_WAVES, FOUR_WAVES],
                         ids=["class1", "class2x3", "class2x4"])
@pytest.mark.parametrize("pair,precision,m", [("lj", "fp64", 1), ("lj", "fp64", 5),
                                              ("lj", "fp64", 6), ("lj", "fp64", 10),
                                              ("lj", "mixed", 4), ("lj", "mixed", 10),
                                              ("morse", "fp64", 10), ("morse", "mixed", 7)])
def test_split_history_kernels(sizes, pair, precision, m):
    off, x = random_starts(sizes, 9710 + len(sizes))
    b = lj.ClusterBatch(off, pair=pair, rho=6.0)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(m=m, max_iter=14)
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS[pair], 6.0
    announce(f"split history {pair} {precision} m={m} clusters={b.num} max_n={b.max_n}")
    r = host_dict(lj.minimize(b, xd, p, precision, switch_point=precision == "mixed"))
    ro = O.minimize(off, r["xyz_switch"] if precision == "mixed" else x, op)
    for key in ("xyz", "energy", "gnorm", "status"):
        assert np.array_equal(r[key], ro[key]), key
    if precision == "fp64":
        assert np.array_equal(r["iters"], ro["iters"]) and np.array_equal(r["evals"], ro["evals"])


@pytest.mark.parametrize("m", [1, 4, 5, 6, 10])
@pytest.mark.parametrize("pair", ["lj", "morse"])
def test_split_history_one_wavefront_equals_register_history(m, pair):
    """Class 0, mixed: the two-wavefronts-per-SIMD kernel gives every output of
    the one-wavefront-per-SIMD kernel, whose history is in registers."""
    sizes = list(range(65)) + [38] * 40
    off, x = random_starts(sizes, 9720)
    b = lj.ClusterBatch(off, pair=pair, rho=6.0)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(m=m, max_iter=150)
    out = []
    try:
        for shape in (0, 4):
            announce(f"split history class 0 mixed {pair} m={m} shape={shape}")
            lj.set_schedule(lj.SCHED_MIN_CLASS[0], "mixed", b.max_n, shape)
            out.append(host_dict(lj.minimize(b, xd, p, "mixed", switch_point=True)))
    finally:
        lj.set_schedule(lj.SCHED_MIN_CLASS[0], "mixed", b.max_n, -1)
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status", "xyz_switch"):
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key
