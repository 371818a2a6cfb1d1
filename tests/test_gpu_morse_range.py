"""The FP64 Morse terms without the general square root's and division's fix-up
steps serve pair distances inside a range; a wavefront with a pair outside it
repeats its sums by the general forms.  Pairs on both sides of the range's
edges, coincident atoms, and ranges rho outside the short forms' own: every
kernel form, bit for bit the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu


def edge_batch(sizes, rho, seed):
    """Random starts; in clusters 1, 2, ... one atom moved to a distance at, just
    below and above e^-400, to e^-708 and beyond it, next to another atom (1e-160
    and 1e-200 away, coincident), or far off."""
    off, x = random_starts(sizes, seed)
    x = x.copy()
    r400, r708 = 1.0 + 400.0 / rho, 1.0 + 708.0 / rho
    moves = [r400, r400 * (1 - 1e-6), r400 * (1 + 1e-6), r400 * 1.2, r708 * (1 - 1e-9),
             r708 * 1.01, 1e-160, 1e-200, 0.0, 1e150]
    for b, d in enumerate(moves, start=1):
        if b < len(sizes) and sizes[b] >= 2:
            o = off[b]
            x[:, o + 1] = 0.0
            x[:, o] = [d, 0.0, 0.0]
    return off, x


@pytest.mark.parametrize("rho", [6.0, 14.0, 1.0e-4, 0.5, 400.0])
@pytest.mark.parametrize("n", [2, 13, 38, 64, 100, 200, 300])
def test_energy_grad_at_the_edges(n, rho):
    off, x = edge_batch([n] * 11, rho, 9800 + n)
    b = lj.ClusterBatch(off, pair="morse", rho=rho)
    announce(f"morse range energy_grad n={n} rho={rho}")
    E, g = lj.energy_grad(b, torch.from_numpy(x).cuda(), "fp64")
    Eo, go = O.energy_grad(off, x, pair="morse", rho=rho)
    assert np.array_equal(host(E), Eo, equal_nan=True)
    assert np.array_equal(host(g), go, equal_nan=True)


@pytest.mark.parametrize("n,shape", [(13, 1), (13, 3), (13, 7), (30, 0), (30, 2), (38, 0), (38, 4),
                                     (60, 0), (60, None), (100, None), (100, 0), (140, 1)])
def test_minimisers_at_the_edges(n, shape):
    off, x = edge_batch([n] * 11, 6.0, 9850 + n)
    b = lj.ClusterBatch(off, pair="morse", rho=6.0)
    p = lj.lbfgs_params(max_iter=25)
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS["morse"], 6.0
    c = 0 if n <= 64 else 1 if n <= 128 else 2
    announce(f"morse range minimise n={n} shape={shape}")
    try:
        if shape is not None:
            lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", n, shape)
        r = host_dict(lj.minimize(b, torch.from_numpy(x).cuda(), p, "fp64"))
    finally:
        lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", n, -1)
    ro = O.minimize(off, x, op)
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status"):
        assert np.array_equal(r[key], ro[key], equal_nan=True), key


@pytest.mark.parametrize("sizes,prec", [([13] * 1500, "fp64"), ([30] * 1100, "fp64"),
                                        ([17, 32, 25] * 500, "fp64"), ([24] * 512, "fp64"),
                                        ([32] * 512, "fp64"), ([31] * 512, "fp64"),
                                        ([45, 46, 48] * 400, "fp64"),
                                        ([13] * 8200, "mixed"), ([30] * 1100, "mixed")])
def test_chosen_form_is_the_plain_one(sizes, prec):
    """The form the built-in rule takes for many Morse clusters, against the
    one-cluster-per-wavefront form, on all outputs."""
    off, x = random_starts(sizes, 9900 + len(sizes))
    b = lj.ClusterBatch(off, pair="morse", rho=6.0)
    p = lj.lbfgs_params(max_iter=30)
    xd = torch.from_numpy(x).cuda()
    announce(f"morse rule {len(sizes)} of up to {max(sizes)} {prec}")
    r = host_dict(lj.minimize(b, xd, p, prec))
    try:
        lj.set_schedule(lj.SCHED_MIN_CLASS[0], prec, max(sizes), 1 if max(sizes) <= 16 else 0)
        plain = host_dict(lj.minimize(b, xd, p, prec))
    finally:
        lj.set_schedule(lj.SCHED_MIN_CLASS[0], prec, max(sizes), -1)
    for key in ("xyz", "energy", "gnorm", "iters", "evals", "status"):
        assert np.array_equal(r[key], plain[key], equal_nan=True), key
