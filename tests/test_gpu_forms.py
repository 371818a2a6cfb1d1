"""The kernel forms that the built-in rule takes: helper wavefronts up to the
limits of a call that has the device on the null stream, up to a quarter of them
on a stream of the caller's, and the same results either way."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu

FOUR, TWO, DENSE = 16, 17, 32
KEYS = ("xyz", "energy", "gnorm", "iters", "evals", "status")


def batch(n, count, pair="lj"):
    return lj.ClusterBatch(np.arange(count + 1) * n, pair=pair)


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def test_helper_limits():
    c, side = cus(), torch.cuda.Stream()
    for n, count, pair, cls, alone, beside in [
            (38, 8, "lj", 0, FOUR, FOUR), (38, c // 2, "lj", 0, FOUR, FOUR),
            (38, c // 2 + 1, "lj", 0, FOUR, TWO), (38, c, "lj", 0, FOUR, TWO),
            (38, c + 1, "lj", 0, FOUR, 0), (38, 2 * c, "lj", 0, FOUR, 0),
            (38, 2 * c + 1, "lj", 0, TWO, 0), (38, 4 * c, "lj", 0, TWO, 0),
            (38, 4 * c + 1, "lj", 0, 4, 4),
            (38, c // 2, "morse", 0, FOUR, FOUR), (38, c // 2 + 1, "morse", 0, FOUR, 0),
            (38, 2 * c + 1, "morse", 0, 0, 0),
            (98, c // 4, "lj", 1, FOUR, FOUR), (98, c // 4 + 1, "lj", 1, FOUR, 0),
            (98, c, "lj", 1, FOUR, 0), (98, c + 1, "lj", 1, 0, 0), (98, 4 * c, "lj", 1, DENSE, DENSE),
            (19, 8, "lj", 0, 0, 0), (13, 8, "lj", 0, 1, 1)]:
        b = batch(n, count, pair)
        assert lj.minimize_forms(b, "fp64")[cls] == alone, (n, count, pair)
        assert lj.minimize_forms(b, "fp64", stream=side)[cls] == beside, (n, count, pair)
        mixed = lj.minimize_forms(b, "mixed")
        assert mixed == lj.minimize_forms(b, "mixed", stream=side) and FOUR not in mixed
    assert lj.minimize_forms(batch(98, 8), "fp64")[2:] == [-1, -1]


def test_small_and_uneven_clusters_take_two_wavefronts():
    """Below 28 atoms, and below 32 where most clusters are much smaller, the form
    with one hand-over is the faster at every count."""
    def form(sizes):
        off = np.concatenate([[0], np.cumsum(sizes)])
        return lj.minimize_forms(lj.ClusterBatch(off), "fp64")[0]

    c = cus()
    for count in (8, c, 2 * c):
        assert form([20] * count) == form([27] * count) == TWO
        assert form([28] * count) == form([13] * (count - 1) + [32]) == FOUR
        assert form([13] * (count - 1) + [20]) == form([13] * (count - 1) + [31]) == TWO
        assert form([13] * (count - 1) + [19]) == 0


@pytest.mark.parametrize("sizes", [[20] * 5 + [27, 21, 26], [13] * 300 + [31, 2, 0, 1], [24] * 500],
                         ids=["20to27", "13and31", "24"])
def test_two_wavefronts_for_small_clusters_bitwise(sizes):
    off, x = random_starts(sizes, 9995)
    b = lj.ClusterBatch(off)
    p = lj.lbfgs_params()
    announce(f"two wavefronts small clusters={b.num} max_n={b.max_n}")
    assert lj.minimize_forms(b, "fp64")[0] == TWO
    r = host_dict(lj.minimize(b, torch.from_numpy(x).cuda(), p, "fp64"))
    ro = O.minimize(off, x, oracle_params(p))
    for key in KEYS:
        assert np.array_equal(r[key], ro[key]), key


@pytest.mark.parametrize("n,share,pair", [(38, 1.2, "lj"), (38, 3, "lj"), (98, 0.4, "lj"),
                                          (38, 0.8, "morse")])
def test_same_results_on_either_kind_of_stream(n, share, pair):
    count, side = int(share * cus()), torch.cuda.Stream()
    off, x = random_starts([n] * count, 9990 + n)
    b = lj.ClusterBatch(off, pair=pair)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(max_iter=60)
    announce(f"forms {pair}{n} x {count}")
    assert lj.minimize_forms(b, "fp64") != lj.minimize_forms(b, "fp64", stream=side)
    alone = host_dict(lj.minimize(b, xd, p, "fp64"))
    beside = host_dict(lj.minimize(b, xd, p, "fp64", stream=side))
    for key in KEYS:
        assert np.array_equal(alone[key], beside[key]), key
