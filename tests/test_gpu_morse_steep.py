"""Steep Morse ranges and pairs almost on top of each other: the energy stays
finite while the force factor's quotient overflows, and then the FP64 gradient
is the oracle's infinity.  Every kernel form, bit for bit the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu

# around the least distance of the short forms (2^-140 = 7.2e-43) and far below
CLOSE = [1e-20, 7e-43, 8e-43, 1e-60, 1e-80, 1e-90, 1e-100]


def close_pairs(n, seed):
    """One cluster per separation, its first two atoms that far apart."""
    off, x = random_starts([n] * len(CLOSE), seed)
    x = x.copy()
    for b, d in enumerate(CLOSE):
        x[:, off[b]] = 0.0
        x[:, off[b] + 1] = np.array([3.0, 2.0, 1.0]) / np.sqrt(14.0) * d
    return off, x


@pytest.mark.parametrize("rho", [6.0, 240.0, 248.0, 280.0, 300.0])
@pytest.mark.parametrize("n", [2, 13, 38, 64, 100, 200, 300])
def test_energy_grad_of_close_pairs(n, rho):
    off, x = close_pairs(n, 9860 + n)
    b = lj.ClusterBatch(off, pair="morse", rho=rho)
    announce(f"morse close pairs energy_grad n={n} rho={rho}")
    E, g = lj.energy_grad(b, torch.from_numpy(x).cuda(), "fp64")
    Eo, go = O.energy_grad(off, x, pair="morse", rho=rho)
    assert np.all(np.isfinite(Eo)) and (rho < 280.0 or np.any(np.isinf(go)))
    assert np.array_equal(host(E), Eo)
    assert np.array_equal(host(g), go, equal_nan=True)


# forced shapes, and None: the built-in rule (helper wavefronts from 32 atoms on)
@pytest.mark.parametrize("n,shape", [(13, 0), (13, 1), (13, 3), (30, 2), (38, 0), (38, 4),
                                     (38, None), (60, 0), (100, None), (100, 0), (140, 1)])
def test_minimisers_of_close_pairs(n, shape):
    off, x = close_pairs(n, 9880 + n)
    b = lj.ClusterBatch(off, pair="morse", rho=300.0)
    p = lj.lbfgs_params(max_iter=20)
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS["morse"], 300.0
    c = 0 if n <= 64 else 1 if n <= 128 else 2
    announce(f"morse close pairs minimise n={n} shape={shape}")
    try:
        if shape is not None:
            lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", n, shape)
        r = host_dict(lj.minimize(b, torch.from_numpy(x).cuda(), p, "fp64"))
    finally:
        lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", n, -1)
    ro = O.minimize(off, x, op)
    assert np.any(ro["status"] == lj.NONFINITE)
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status"):
        assert np.array_equal(r[key], ro[key], equal_nan=True), key
