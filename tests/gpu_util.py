"""Helpers shared by the GPU parity tests (no method arithmetic here)."""
import sys

import numpy as np
import torch

from paper_2510_25938_amd import lj

DEV = "cuda"


def announce(msg):
    """Name the case on stdout before a GPU step (flushed)."""
    sys.stdout.write(f"[gpu-case] {msg}\n")
    sys.stdout.flush()


def to_dev(off, xyz):
    batch = lj.ClusterBatch(off, device=DEV)
    return batch, torch.from_numpy(np.ascontiguousarray(xyz)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return None if t is None else t.cpu().numpy()


def host_dict(d):
    torch.cuda.synchronize()
    return {k: (None if v is None else v.cpu().numpy()) for k, v in d.items()}


def settle(*streams):
    """Lets the built-in rule see calls on these streams only (None: the current
    stream): eight calls just large enough to count."""
    num = torch.cuda.get_device_properties(0).multi_processor_count // 4 + 1
    off = np.arange(num + 1) * 2
    x = np.zeros((3, 2 * num))
    x[0, 1::2] = 1.1
    batch, xd = to_dev(off, x)
    for k in range(8):
        lj.minimize(batch, xd, lj.lbfgs_params(max_iter=1), "fp64",
                    stream=streams[k % len(streams)])
    torch.cuda.synchronize()


U32 = 2.0 ** -24
