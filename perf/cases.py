"""Performance cases of the Lennard-Jones / Morse cluster library.

Each case is one call (or one short run of calls) that a program makes through
the public entry points of paper_2510_25938_amd.lj:

  kind "eval"  energy_grad: energies and gradients of a ragged batch;
  kind "min"   minimize: the L-BFGS minimisation of a ragged batch of starts;
  kind "bh"    BasinHopping.step: `steps` basin-hopping steps of all chains.

Sizes: `count` clusters (chains for "bh") of lo .. hi atoms, uniform on the
integers and the same for every seed, which draws the coordinates (and the
random stream of a chain).  Evaluations get compact jittered fcc balls, the
structures an energy call meets during a search; minimisations get random cube
starts, as the benchmark's workloads do; chains start from minimised
structures.
"""
import math

import numpy as np
import torch

from paper_2510_25938_amd import inputs, lj

PAIR_FLOP = 27  # one unique pair: distance, pair term, force, both accumulations


def listed():
    return [
        # one small cluster, energy and gradient: the latency of a single call
        # (an external optimiser or a check of one structure)
        _eval("eval_lj13_x1_fp64", 1, 13, 13, "fp64"),
        # the batched pair kernel on large clusters (the pair-kernel benchmark)
        _eval("eval_lj1000_x256_mixed", 256, 1000, 1000, "mixed"),
        # a few structures near the largest supported size, odd sizes
        _eval("eval_lj2999_3001_x3_fp64", 3, 2999, 3001, "fp64"),
        # the eight candidates of one step, an odd size of the middle class,
        # minimised by themselves in the default precision
        _min("min_lj98_x8_fp64", 8, 98, 98, "fp64"),
        # the headline batch, mixed precision with polish, and in FP64
        _min("min_lj38_x1024_mixed", 1024, 38, 38, "mixed"),
        _min("min_lj38_x1024_fp64", 1024, 38, 38, "fp64"),
        # the same batch with the Morse pair
        _min("min_morse38_x1024_fp64", 1024, 38, 38, "fp64", pair="morse", rho=6.0),
        # many small clusters (LJ13 candidates of many chains)
        _min("min_lj13_x16384_fp64", 16384, 13, 13, "fp64"),
        # a ragged batch over three size classes
        _min("min_uneven13_150_x4096_mixed", 4096, 13, 150, "mixed"),
        # large clusters, 500 iterations without polish
        _min("min_lj1000_x256_mixed", 256, 1000, 1000, "mixed", max_iter=500, polish=0),
        # the paper's own run: one LJ13 chain with 8 candidates per step
        _bh("bh_lj13_x1_c8_fp64", 1, 13, 13, 8, 40, "fp64"),
        # many adaptive chains of uneven size
        _bh("bh_38_75_x512_c8_mixed", 512, 38, 75, 8, 2, "mixed"),
    ]


def draw(rng):
    kind = rng.choice(["eval", "eval", "min", "min", "min", "bh"])
    precision = rng.choice(["fp64", "mixed"])
    pair, rho = ("morse", rng.choice([3.0, 6.0, 10.0])) if rng.random() < 0.2 else ("lj", 0.0)
    if kind == "eval":
        hi = _log_int(rng, 2, 4096)
        lo = hi if rng.random() < 0.5 else max(2, hi // rng.choice([2, 4, 10]))
        most = max(1.0, 1.2e8 / (hi * hi))
        count = _log_int(rng, 1, int(min(16384, most)))
        return _eval(None, count, lo, hi, precision, pair, rho, grad=rng.random() < 0.8)
    if kind == "min":
        hi = _log_int(rng, 2, 1000)
        lo = hi if rng.random() < 0.5 else max(2, hi // rng.choice([2, 4, 10]))
        cap = 10000 if hi <= 256 else 100
        most = max(1.0, (8.0e6 if hi <= 256 else 3.0e7) / (hi * hi))
        count = _log_int(rng, 1, int(min(16384, most)))
        return _min(None, count, lo, hi, precision, pair, rho, max_iter=cap,
                    polish=1 if hi <= 256 else rng.choice([0, 1]))
    hi = _log_int(rng, 4, 128)
    lo = hi if rng.random() < 0.5 else max(4, hi // 2)
    cands = rng.choice([1, 2, 4, 8, 8, 16])
    count = _log_int(rng, 1, int(max(1, min(1024, 4.0e6 / (hi * hi * cands)))))
    steps = 8 if hi <= 40 else 2
    return _bh(None, count, lo, hi, cands, steps, precision, pair, rho)


def prepare(case, seed):
    pair = {"pair": case["pair"], "rho": case["rho"]}
    if case["kind"] == "eval":
        off, x = _ball_batch(case, seed)
        return {"case": case, "batch": lj.ClusterBatch(off, **pair), "xyz": _device(x)}
    off, x = inputs.random_starts(_sizes(case), seed)
    batch = lj.ClusterBatch(off, **pair)
    xyz = _device(x)
    if case["kind"] == "min":
        params = lj.lbfgs_params(max_iter=case["max_iter"], polish=case["polish"])
        return {"case": case, "batch": batch, "xyz": xyz, "params": params}
    # basin hopping: the chains' start minima and the chain object
    params = lj.lbfgs_params()
    start = lj.minimize(batch, xyz, params, "fp64")
    bh = lj.BasinHopping(batch, start["xyz"], start["energy"],
                         lj.bh_params(cands=case["cands"], kT=0.8, seed=seed), params,
                         case["precision"], step0=0.4, trace_steps=case["steps"])
    return {"case": case, "batch": batch, "bh": bh, "xyz": start["xyz"], "energy": start["energy"],
            "stream": torch.cuda.Stream()}


def run(state):
    case = state["case"]
    if case["kind"] == "eval":
        E, g = lj.energy_grad(state["batch"], state["xyz"], case["precision"], grad=case["grad"])
        return (E, g) if case["grad"] else (E,)
    if case["kind"] == "min":
        r = lj.minimize(state["batch"], state["xyz"], state["params"], case["precision"])
        return tuple(r[k] for k in ("xyz", "energy", "gnorm", "iters", "evals", "status"))
    return _search(state)


def _search(state):
    """A search of `steps` steps from the chains' start minima (a program that
    restarts its search puts the chain state back to the start).  Steps run on
    a stream of the caller's, where the library replays its step graph."""
    bh, steps = state["bh"], state["case"]["steps"]
    s, cur = state["stream"], torch.cuda.current_stream()
    s.wait_stream(cur)
    with torch.cuda.stream(s):
        bh.xyz_cur.copy_(state["xyz"])
        bh.xyz_best.copy_(state["xyz"])
        bh.e_cur.copy_(state["energy"])
        bh.e_best_acc.copy_(state["energy"])
        bh.e_best_seen.fill_(float("inf"))
        bh.step_size.fill_(0.4)
        bh.win_accepts.zero_()
        bh.step_index.zero_()
        bh.step(steps, stream=s)
    cur.wait_stream(s)
    trace = [bh.trace[k] for k in ("e_trial", "accepted", "e_best", "e_best_acc", "e_cur", "step",
                                   "polish_status")]
    return (bh.xyz_cur, bh.e_cur, bh.step_size, bh.win_accepts, bh.step_index, bh.e_best_seen,
            bh.e_best_acc, bh.xyz_best, *trace)


def work(case):
    """Bytes: coordinates in, results out.  Flops: the pair terms of the
    evaluations a search of this size takes (about 48 sqrt(N) per
    minimisation) and, for the minimiser, the two-loop recursion and updates
    of each iteration (10 stored pairs)."""
    sizes = np.arange(case["lo"], case["hi"] + 1, dtype=np.float64)
    n = float(sizes.mean())
    pairs = float((sizes * (sizes - 1) / 2).mean())
    count = case["count"]
    if case["kind"] == "eval":
        out = 24.0 * n if case["grad"] else 0.0
        return {"bytes": int(count * (24.0 * n + out + 8)), "flops": int(count * PAIR_FLOP * pairs)}
    iters = min(48.0 * math.sqrt(n), float(case["max_iter"]))
    per_min = iters * (PAIR_FLOP * pairs + 300.0 * n)
    if case["kind"] == "min":
        return {"bytes": int(count * (48.0 * n + 28)), "flops": int(count * per_min)}
    runs = count * case["cands"] * case["steps"]
    return {"bytes": int(count * 96.0 * n + 40 * count * case["steps"]),
            "flops": int(runs * per_min)}


def exact(case, seed):
    """Energies and gradients in 64 bits from the pair potential's definition;
    None for searches, whose path has no value of its own to compare with."""
    if case["kind"] != "eval":
        return None
    off, x = _ball_batch(case, seed)
    xyz = _device(x)
    grad = torch.zeros_like(xyz)
    energy = torch.zeros(len(off) - 1, dtype=torch.float64, device=xyz.device)
    groups = {}
    for b, n in enumerate(np.diff(off)):
        groups.setdefault(int(n), []).append(b)
    for n, members in groups.items():
        chunk = max(1, 8_000_000 // (n * n))
        for k in range(0, len(members), chunk):
            bs = torch.tensor(members[k:k + chunk], device=xyz.device)
            starts = torch.tensor(off[members[k:k + chunk]].astype(np.int64), device=xyz.device)
            at = starts[:, None] + torch.arange(n, device=xyz.device)
            e, g = _pair_sums(xyz[:, at], case["pair"], case["rho"])
            energy[bs] = e
            grad[:, at] = g
    return (energy, grad) if case["grad"] else (energy,)


def _pair_sums(x, pair, rho):
    """x [3][clusters][n] -> energies [clusters], gradients [3][clusters][n]."""
    n = x.shape[2]
    d = x[:, :, :, None] - x[:, :, None, :]
    r2 = (d * d).sum(0)
    diag = torch.eye(n, dtype=torch.bool, device=x.device)
    if pair == "lj":
        q = torch.where(diag, 0.0, 1.0 / torch.where(diag, 1.0, r2))
        s6 = q ** 3
        v = 4.0 * (s6 * s6 - s6)
        f = q * (24.0 * s6 - 48.0 * s6 * s6)
    else:
        r = torch.where(diag, 1.0, r2).sqrt()
        t = torch.where(diag, 0.0, torch.exp(rho * (1.0 - r)))
        v = t * (t - 2.0)
        f = -2.0 * rho * t * (t - 1.0) / r
    return 0.5 * v.sum((1, 2)), (f * d).sum(3)


def _case(kind, name, count, lo, hi, precision, pair, rho, **more):
    case = {"kind": kind, "count": count, "lo": lo, "hi": hi, "precision": precision,
            "pair": pair, "rho": rho, **more}
    if name is not None:
        case["name"] = name
    return case


def _eval(name, count, lo, hi, precision, pair="lj", rho=0.0, grad=True):
    return _case("eval", name, count, lo, hi, precision, pair, rho, grad=grad)


def _min(name, count, lo, hi, precision, pair="lj", rho=0.0, max_iter=10000, polish=1):
    return _case("min", name, count, lo, hi, precision, pair, rho, max_iter=max_iter, polish=polish)


def _bh(name, count, lo, hi, cands, steps, precision, pair="lj", rho=0.0):
    return _case("bh", name, count, lo, hi, precision, pair, rho, cands=cands, steps=steps,
                 max_iter=10000)


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _sizes(case):
    if case["lo"] == case["hi"]:
        return np.full(case["count"], case["lo"], dtype=np.int64)
    return inputs.uniform_sizes(case["count"], case["lo"], case["hi"], inputs.SEED_BASE + 3)


def _device(x):
    return torch.from_numpy(x).to("cuda")


def _ball_batch(case, seed):
    """Compact clusters: the n fcc sites nearest to a random point of the cell,
    at the pair's nearest-neighbour distance, each site jittered."""
    sizes = _sizes(case)
    rng = np.random.Generator(np.random.Philox(key=np.uint64(seed)))
    k = int(math.ceil((0.75 * int(sizes.max()) / math.pi / 4.0) ** (1.0 / 3.0))) + 2
    cell = np.arange(-k, k + 1, dtype=np.float64)
    grid = np.stack(np.meshgrid(cell, cell, cell, indexing="ij"), axis=-1).reshape(-1, 1, 3)
    basis = np.array([[0, 0, 0], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
    sites = (grid + basis).reshape(-1, 3) * (1.09 if case["pair"] == "lj" else 1.0) * math.sqrt(2.0)
    # a handful of ball centres serve the whole batch; the jitter is its own
    balls = [sites[np.argsort(((sites - c) ** 2).sum(1), kind="stable")[:int(sizes.max())]] - c
             for c in rng.random((8, 3))]
    off = inputs.offsets_from_sizes(sizes)
    xyz = np.concatenate([balls[b % 8][:n] for b, n in enumerate(sizes)])
    xyz = xyz + rng.uniform(-0.08, 0.08, xyz.shape)
    return off, np.ascontiguousarray(xyz.T)
