"""The kernel forms that the built-in rule takes: helper wavefronts up to limits
that are divided by the number of caller streams among the last larger calls, and
the same results whatever the form."""
import numpy as np
import pytest
import torch

from gpu_util import announce, host_dict, settle
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


@pytest.mark.parametrize("streams", [1, 2, 3, 5])
def test_helper_limits(streams):
    c, calls = cus(), min(streams, 4)
    side = [None] + [torch.cuda.Stream() for _ in range(streams - 1)]
    settle(*side)
    for n, pair, cls, form, limit, beyond in [
            (38, "lj", 0, FOUR, 2 * c, TWO), (38, "lj", 0, TWO, 4 * c, None),
            (38, "morse", 0, FOUR, 2 * c, 0), (98, "lj", 1, FOUR, c, None)]:
        for count in (1, limit // 4, limit // calls):
            if form == TWO and count * calls <= 2 * c:
                continue
            for stream in side:
                assert lj.minimize_forms(batch(n, count, pair), "fp64", stream)[cls] == form
        over = lj.minimize_forms(batch(n, limit // calls + 1, pair), "fp64")[cls]
        assert over == beyond or (beyond is None and over not in (FOUR, TWO))
    for n, count, pair, cls, form in [(98, 4 * c, "lj", 1, DENSE), (38, 4 * c + 1, "lj", 0, 4),
                                      (19, 8, "lj", 0, 0), (13, 8, "lj", 0, 1)]:
        assert lj.minimize_forms(batch(n, count, pair), "fp64")[cls] == form
        assert not {FOUR, TWO} & set(lj.minimize_forms(batch(n, count, pair), "mixed"))
    assert lj.minimize_forms(batch(98, 8), "fp64")[2:] == [-1, -1]


def test_the_rule_forgets_other_streams():
    """One caller on a stream of its own has the limits of one call; one call, and
    small calls, on other streams are not counted."""
    c, side, b = cus(), torch.cuda.Stream(), batch(38, 2 * cus())
    settle(None, side)
    assert lj.minimize_forms(b, "fp64", side)[0] == TWO
    settle(side)
    assert lj.minimize_forms(b, "fp64", side)[0] == FOUR
    off, x = random_starts([2] * (c // 4 + 1), 1)
    lj.minimize(lj.ClusterBatch(off), torch.from_numpy(x).cuda(), None, "fp64")
    assert lj.minimize_forms(b, "fp64", side)[0] == FOUR
    off, x = random_starts([2] * (c // 4), 1)
    few = lj.ClusterBatch(off)
    for _ in range(8):
        lj.minimize(few, torch.from_numpy(x).cuda(), None, "fp64")
    torch.cuda.synchronize()
    assert lj.minimize_forms(b, "fp64", side)[0] == FOUR


def test_small_and_uneven_clusters_take_two_wavefronts():
    """Below 28 atoms, and below 32 where most clusters are much smaller, the form
    with one hand-over is the faster at every count."""
    def form(sizes):
        off = np.concatenate([[0], np.cumsum(sizes)])
        return lj.minimize_forms(lj.ClusterBatch(off), "fp64")[0]

    settle(None)
    c = cus()
    for count in (8, c, 2 * c):
        assert form([20] * count) == form([27] * count) == TWO
        assert form([28] * count) == form([13] * (count - 1) + [32]) == FOUR
        assert form([13] * (count - 1) + [20]) == form([13] * (count - 1) + [31]) == TWO
        assert form([13] * (count - 1) + [19]) == 0


@pytest.mark.parametrize("sizes", [[20] * 5 + [27, 21, 26], [13] * 300 + [31, 2, 0, 1], [24] * 500,
                                   list(range(65)) + [20, 38, 45, 64] * 120],
                         ids=["20to27", "13and31", "24", "0to64"])
def test_two_wavefronts_bitwise(sizes):
    off, x = random_starts(sizes, 9995)
    b = lj.ClusterBatch(off)
    p = lj.lbfgs_params()
    announce(f"two wavefronts clusters={b.num} max_n={b.max_n}")
    settle(None)
    assert lj.minimize_forms(b, "fp64")[0] == TWO
    r = host_dict(lj.minimize(b, torch.from_numpy(x).cuda(), p, "fp64"))
    ro = O.minimize(off, x, oracle_params(p))
    for key in KEYS:
        assert np.array_equal(r[key], ro[key]), key


@pytest.mark.parametrize("n,share,pair", [(38, 1.2, "lj"), (38, 3, "lj"), (98, 0.4, "lj"),
                                          (38, 0.8, "morse")])
def test_same_results_beside_other_calls(n, share, pair):
    count, side = int(share * cus()), [torch.cuda.Stream() for _ in range(4)]
    off, x = random_starts([n] * count, 9990 + n)
    b = lj.ClusterBatch(off, pair=pair)
    xd = torch.from_numpy(x).cuda()
    p = lj.lbfgs_params(max_iter=60)
    announce(f"forms {pair}{n} x {count}")
    settle(side[0])
    form = lj.minimize_forms(b, "fp64", side[0])
    alone = host_dict(lj.minimize(b, xd, p, "fp64", stream=side[0]))
    settle(*side)
    assert lj.minimize_forms(b, "fp64", side[0]) != form
    for out in [lj.minimize(b, xd, p, "fp64", stream=s) for s in side]:
        beside = host_dict(out)
        for key in KEYS:
            assert np.array_equal(alone[key], beside[key]), key
