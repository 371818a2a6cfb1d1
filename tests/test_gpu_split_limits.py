"""The evaluation over many workgroups where offsets and the descriptor's max_n
disagree (a cluster above max_n is evaluated if it fits the launch shape, else
its energy is NaN), and at tile counts that do not fill the launch shape: bit for
bit the one-workgroup evaluation."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_util import announce, host, to_dev
from paper_2510_25938_amd import lj
from paper_2510_25938_amd.inputs import random_starts

pytestmark = pytest.mark.gpu


def evaluate(b, desc, xd, precision, spread):
    prec = lj.precision_code(precision)
    nb = lj.lib().lj_energy_grad_workspace_bytes(C.byref(desc), prec) if spread else 0
    assert (nb > 0) == spread
    ws = torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda")
    E = torch.full((b.num,), 7.0, dtype=torch.float64, device="cuda")
    g = torch.full_like(xd, 5.0)
    assert lj.lib().lj_energy_grad_batch_ws(C.byref(desc), xd.data_ptr(), E.data_ptr(),
                                            g.data_ptr(), prec, ws.data_ptr(), nb, None) == lj.OK
    return host(E), host(g)


@pytest.mark.parametrize("pair", ["lj", "morse"])
@pytest.mark.parametrize("precision,sizes,max_n", [
    ("fp64", [500, 300, 40, 320, 0], 300),      # 5 of 8 tiles, and a cluster of 8
    ("fp64", [600, 300, 40, 320, 0, 9], 300),   # one that does not fit
    ("fp64", [300] * 40 + [257], 300),
    ("fp64", [1281, 2048, 700], 1400),          # 22 of 32 tiles, and a cluster of 32
    ("mixed", [500, 449, 40, 500, 0], 449),
    ("mixed", [1281, 2048, 700], 1400),
    ("mixed", [600, 449, 40, 449, 0, 3], 449)])
def test_spread_evaluation_and_max_n(precision, sizes, max_n, pair):
    off, x = random_starts(sizes, 9960 + max_n, side=[1.3 * max(n, 1) ** (1 / 3) for n in sizes])
    b, xd = to_dev(off, x)
    b.pair = pair
    desc = b.desc(max_n=max_n)
    announce(f"spread evaluation {pair} {precision} sizes={sizes[:6]} max_n={max_n}")
    E, g = evaluate(b, desc, xd, precision, True)
    E1, g1 = evaluate(b, desc, xd, precision, False)
    assert np.array_equal(E, E1, equal_nan=True) and np.array_equal(g, g1)
    w, a = lj.eval_shape_default(max_n)
    assert np.array_equal(np.isnan(E), np.array(sizes) > 64 * w * a)
