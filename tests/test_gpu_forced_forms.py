"""Kernel forms that the built-in rule gives to other batches than it used to, each
forced or checked by lj.minimize_forms before its results are compared: the
unique-pair Morse kernel, class 1 on both sides of the limits of its forms, and
the batches by which the other files mean to reach a form."""
import numpy as np
import pytest
import torch

import test_gpu_dense
from gpu_util import announce, host, host_dict, settle, to_dev
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts
from test_gpu_minimize import oracle_params

pytestmark = pytest.mark.gpu

FOUR, TWO, DENSE = 16, 17, 32
KEYS = ("xyz", "energy", "gnorm", "iters", "evals", "status")


def same(r, ro):
    for key in KEYS:
        assert np.array_equal(r[key], ro[key], equal_nan=True), key


def forced(c, b, shape, x, p):
    """FP64 minimisation with class c in the given shape."""
    try:
        lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", b.max_n, shape)
        assert lj.minimize_forms(b, "fp64")[c] & ~DENSE == shape
        return host_dict(lj.minimize(b, torch.from_numpy(np.ascontiguousarray(x)).cuda(), p, "fp64"))
    finally:
        lj.set_schedule(lj.SCHED_MIN_CLASS[c], "fp64", b.max_n, -1)


# every size beside larger ones (the matrix holds 40 atoms, the ordered loop serves
# 41 .. 44), and each size that the matrix can be made for
@pytest.mark.parametrize("sizes", [list(range(45))] + [[n, n - 1, 2, n] for n in range(33, 42)],
                         ids=lambda s: f"{len(s)}x{max(s)}")
@pytest.mark.parametrize("rho", [6.0, 3.0])
def test_unique_pair_morse_kernel_bitwise(sizes, rho):
    off, x = random_starts(sizes, 9700 + len(sizes) + max(sizes))
    b = lj.ClusterBatch(off, pair="morse", rho=rho)
    p = lj.lbfgs_params()
    op = oracle_params(p)
    op.pair, op.rho = lj.PAIRS["morse"], rho
    announce(f"unique-pair morse sizes={sizes[:4]}.. max_n={b.max_n} rho={rho}")
    same(forced(0, b, 0, x, p), O.minimize(off, x, op))


@pytest.mark.parametrize("count,below,above", [("cus", FOUR, 0), ("640", 0, DENSE)])
def test_class1_forms_on_both_sides_of_a_limit(count, below, above):
    """Helper wavefronts | one wavefront per SIMD | two: the clusters that a batch
    and one with one more cluster share give the same outputs."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    count = cus if count == "cus" else 10 * cus // 4  # 2 wavefronts each, 1.25 per SIMD
    sizes = [65 + (k * 37) % 64 for k in range(count)] + [65]
    off, x = random_starts(sizes, 9710)
    p = lj.lbfgs_params(max_iter=40)
    settle(None)
    out = []
    for k, form in ((count, below), (count + 1, above)):
        b, xd = to_dev(off[:k + 1], np.ascontiguousarray(x[:, :off[k]]))
        announce(f"class 1 form {form} clusters={k}")
        assert lj.minimize_forms(b, "fp64")[1] == form
        out.append(host_dict(lj.minimize(b, xd, p, "fp64")))
    for key in KEYS:
        a = out[1][key][:, :off[count]] if key == "xyz" else out[1][key][:count]
        assert np.array_equal(out[0][key], a), key


@pytest.mark.parametrize("shape", [0, 1, None])
def test_class1_beside_a_larger_cluster_fp64_bitwise(shape):
    sizes = [65, 100, 128, 80, 13, 127, 96, 70, 129]
    off, x = random_starts(sizes, 4242)
    b, xd = to_dev(off, x)
    p = lj.lbfgs_params()
    announce(f"class 1 beside 129 atoms shape={shape}")
    if shape is None:
        assert lj.minimize_forms(b, "fp64")[:2] == [FOUR, FOUR]
        r = host_dict(lj.minimize(b, xd, p, "fp64"))
    else:
        r = forced(1, b, shape, x, p)
    same(r, O.minimize(off, x, oracle_params(p)))


def test_batches_of_the_other_files_reach_their_forms():
    def forms(sizes, precision="fp64", pair="lj"):
        off = np.concatenate([[0], np.cumsum(sizes)])
        return lj.minimize_forms(lj.ClusterBatch(off, pair=pair), precision)

    settle(None)
    for precision in ("fp64", "mixed"):  # half of the history in LDS
        assert forms(test_gpu_dense.TWO_WAVES, precision)[1] & DENSE
        assert forms(test_gpu_dense.THREE_WAVES, precision)[2] == DENSE + 1
        assert forms(test_gpu_dense.FOUR_WAVES, precision)[2] == DENSE
    for pair in ("lj", "morse"):  # helper wavefronts
        assert forms(list(range(65)), pair=pair)[0] == FOUR
        assert forms([65, 128, 1, 127, 0, 96], pair=pair)[:2] == [FOUR, FOUR]
    assert forms([20])[0] == TWO
    assert forms(list(range(65)) + [20, 21, 38, 44, 45, 64] * 80)[0] == TWO
    assert forms([32] * 512, pair="morse")[0] == FOUR and forms([31] * 512, pair="morse")[0] == 0


@pytest.mark.parametrize("pair,rho", [("lj", 6.0), ("morse", 6.0), ("morse", 14.0),
                                      ("morse", 250.0)])
def test_sampled_pair_terms_equal_the_oracle(pair, rho):
    """The reciprocal, root and quotient without their scaling and fix-up steps, one
    pair per cluster: 3e5 squared distances over 80 binary orders, among them
    mantissas next to 1 and 2 and whole powers of two."""
    rng = np.random.Generator(np.random.Philox(key=np.uint64(2510 + int(rho))))
    num = 300_000
    near = np.ldexp(1.0, -rng.integers(30, 53, num)) * rng.choice([-1.0, 1.0, 0.0], num)
    m = np.where(rng.random(num) < 0.5, rng.uniform(1.0, 2.0, num), 1.0 + near)
    r = m * np.exp2(rng.uniform(-20, 20, num).round() if pair == "lj"
                    else rng.uniform(-20, 2, num).round())
    d = rng.normal(size=(3, num))
    d = np.where(rng.random(num) < 0.5, d / np.sqrt((d * d).sum(0)),
                 np.array([1.0, 0.0, 0.0])[:, None])
    x = np.zeros((3, 2 * num))
    x[:, 1::2] = d * r
    off = np.arange(num + 1, dtype=np.int32) * 2
    b = lj.ClusterBatch(off, pair=pair, rho=rho)
    announce(f"sampled pair terms {pair} rho={rho}")
    E, g = lj.energy_grad(b, torch.from_numpy(x).cuda(), "fp64")
    Eo, go = O.energy_grad(off, x, pair=pair, rho=rho)
    assert np.array_equal(host(E), Eo) and np.array_equal(host(g), go)
