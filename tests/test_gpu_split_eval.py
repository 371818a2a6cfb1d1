"""GPU parity of the evaluation of a few large clusters over many workgroups:
bit for bit the one-workgroup evaluation (which the other tests hold against
the oracle), and in FP64 the oracle, at the edges of tiles, chunks and shapes."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import announce, host
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts

pytestmark = pytest.mark.gpu


def one_workgroup(b, xd, precision, sigma, epsilon):
    """lj_energy_grad_batch without scratch memory."""
    E = torch.empty(b.num, dtype=torch.float64, device="cuda")
    g = torch.full_like(xd, float("nan"))
    assert lj.lib().lj_energy_grad_batch(
        C.byref(b.desc(sigma=sigma, epsilon=epsilon)), C.c_void_p(xd.data_ptr()),
        C.c_void_p(E.data_ptr()), C.c_void_p(g.data_ptr()), lj.precision_code(precision),
        C.c_void_p(torch.cuda.current_stream().cuda_stream)) == lj.OK
    return E, g


# odd and even tile counts, a last tile of one atom, every built-in shape above
# 256 atoms (8 x 1, 16 x 1, 16 x 2, 16 x 4), and clusters far below the largest
@pytest.mark.parametrize("sizes", [[257], [449, 0, 1, 33, 300], [512, 511, 20, 64], [1000, 65],
                                   [1025, 40, 31], [2048], [2049, 700], [4096, 4033]],
                         ids=lambda s: str(s[0]))
@pytest.mark.parametrize("pair,precision", [("lj", "fp64"), ("lj", "mixed"), ("morse", "fp64"),
                                            ("morse", "mixed")])
def test_spread_evaluation_equals_one_workgroup(sizes, pair, precision):
    off, x = random_starts(sizes, 9300 + sizes[0], side=[1.3 * max(n, 1) ** (1 / 3) for n in sizes])
    b = lj.ClusterBatch(off, pair=pair, rho=6.0)
    announce(f"spread evaluation {pair} {precision} sizes={sizes}")
    for scale in (1.0, 1.7):
        xd = torch.from_numpy(x).cuda() * scale
        nb = lj.lib().lj_energy_grad_workspace_bytes(C.byref(b.desc()), lj.precision_code(precision))
        assert (nb > 0) == (precision == "fp64" or max(sizes) > 448)
        E, g = lj.energy_grad(b, xd, precision, sigma=scale, epsilon=1.25)
        E1, g1 = one_workgroup(b, xd, precision, scale, 1.25)
        assert np.array_equal(host(E), host(E1), equal_nan=True)
        assert np.array_equal(host(g), host(g1), equal_nan=True)
        Ee, _ = lj.energy_grad(b, xd, precision, grad=False, sigma=scale, epsilon=1.25)
        assert np.array_equal(host(Ee), host(E1), equal_nan=True)
    if precision == "fp64" and max(sizes) <= 1025:
        E, g = lj.energy_grad(b, torch.from_numpy(x).cuda(), "fp64")
        Eo, go = O.energy_grad(off, x, pair=pair, rho=6.0)
        assert np.array_equal(host(E), Eo) and np.array_equal(host(g), go)


def test_spread_evaluation_of_coincident_atoms():
    """Out-of-range pair distances repeat the tiles they touch with the IEEE
    division: coincident atoms in different tiles, and a pair far apart."""
    sizes = [300, 520]
    off, x = random_starts(sizes, 9400, side=[12.0, 13.0])
    x = x.copy()
    x[:, 10] = x[:, 200]
    x[0, off[1] + 5] += 1.0e160
    b = lj.ClusterBatch(off)
    xd = torch.from_numpy(x).cuda()
    announce("spread evaluation of coincident atoms")
    E, g = lj.energy_grad(b, xd, "fp64")
    Eo, go = O.energy_grad(off, x)
    assert not np.isfinite(Eo[0]) and np.isfinite(Eo[1])
    assert np.array_equal(host(E), Eo, equal_nan=True)
    assert np.array_equal(host(g), go, equal_nan=True)
