"""The schedule table's pair-kernel shapes and the evaluation over many workgroups:
an entry does not keep a call of a few large clusters from being spread, unless
its sums have another order; without scratch memory every entry's own kernel
runs."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import announce, host, to_dev
from oracle import oracle as O
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts

pytestmark = pytest.mark.gpu


def spread_bytes(b, precision):
    return lj.lib().lj_energy_grad_workspace_bytes(C.byref(b.desc()), lj.precision_code(precision))


def one_workgroup(b, xd, precision):
    E = torch.empty(b.num, dtype=torch.float64, device="cuda")
    g = torch.empty_like(xd)
    assert lj.lib().lj_energy_grad_batch(C.byref(b.desc()), xd.data_ptr(), E.data_ptr(),
                                         g.data_ptr(), lj.precision_code(precision),
                                         None) == lj.OK
    return host(E), host(g)


def restore(precision, max_n):
    lj.set_schedule(lj.SCHED_EVAL, precision, max_n, *lj.eval_shape_default(max_n))


@pytest.mark.parametrize("pair,precision,max_n,shape,spread", [
    ("lj", "fp64", 1000, (8, 2), True), ("lj", "fp64", 1500, (16, 4), True),
    ("lj", "mixed", 1000, (8, 2), True), ("lj", "mixed", 1500, (8, 4), True),
    ("lj", "mixed", 1500, (16, 4), False), ("morse", "mixed", 1500, (16, 4), True)])
def test_entries_and_spreading(pair, precision, max_n, shape, spread):
    off, x = random_starts([max_n, 900], 9970, side=[1.3 * max_n ** (1 / 3), 12.6])
    b, xd = to_dev(off, x)
    b.pair = pair
    announce(f"schedule entry {shape} {pair} {precision} max_n={max_n}")
    before = [host(t) for t in lj.energy_grad(b, xd, precision)]
    try:
        lj.set_schedule(lj.SCHED_EVAL, precision, max_n, *shape)
        assert (spread_bytes(b, precision) > 0) == spread
        now = [host(t) for t in lj.energy_grad(b, xd, precision)]
        plain = one_workgroup(b, xd, precision)
    finally:
        restore(precision, max_n)
    for p, q, r in zip(before, now, plain):
        assert np.array_equal(q, r)  # with and without scratch memory, under the entry
        if spread:
            assert np.array_equal(p, q)


@pytest.mark.parametrize("sizes", [[1000, 700, 13], [1500, 900], [300, 257]])
def test_every_entry_without_scratch_memory_fp64(sizes):
    """Each shape's one-workgroup kernel against the oracle."""
    off, x = random_starts(sizes, 9975 + sizes[0])
    b, xd = to_dev(off, x)
    Eo, go = O.energy_grad(off, x)
    shapes = [(w, a) for w in (1, 2, 4, 8, 16) for a in (1, 2, 4)
              if b.max_n <= 64 * w * a <= 4096]
    assert len(shapes) >= 2
    try:
        for w, a in shapes:
            announce(f"one workgroup W={w} A={a} sizes={sizes}")
            lj.set_schedule(lj.SCHED_EVAL, "fp64", b.max_n, w, a)
            E, g = one_workgroup(b, xd, "fp64")
            assert np.array_equal(E, Eo) and np.array_equal(g, go), (w, a)
    finally:
        restore("fp64", b.max_n)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_autotune_times_the_spread_form(precision):
    """A tuned batch of many clusters leaves a single one spread; a tuned batch
    that is spread reports a time below the one-workgroup kernel's."""
    off, x = random_starts([1100] * 200, 9980)
    many, xm = to_dev(off, x)
    few, xf = to_dev(off[:2], np.ascontiguousarray(x[:, :1100]))
    announce(f"autotune spread {precision}")
    want = [host(t) for t in lj.energy_grad(few, xf, precision)]
    try:
        lj.autotune(many, xm, precision)
        assert spread_bytes(many, precision) == 0
        shape = lj.get_schedule(lj.SCHED_EVAL, precision, 1100)
        same_order = precision == "fp64" or shape != (16, 4)
        assert (spread_bytes(few, precision) > 0) == same_order
        if same_order:
            for p, q in zip(want, lj.energy_grad(few, xf, precision)):
                assert np.array_equal(p, host(q))
        restore(precision, 1100)
        ms = lj.autotune(few, xf, precision)["eval"][2]
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        one_workgroup(few, xf, precision)
        e1.record()
        torch.cuda.synchronize()
        assert 0 < ms < e0.elapsed_time(e1)
    finally:
        restore(precision, 1100)
