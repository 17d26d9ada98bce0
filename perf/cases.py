"""Performance cases: what programs do with this library, over the range of sizes and options they do it at.

A case is a dict of plain values.  Its "form" says which calls a pass makes:

  epochs    a problem kept by the program and past its warm-up; a pass runs the
            epoch schedule "tours" (run_tours and merge_epoch for each entry)
  graph     the same through a captured epoch, replayed "replays" times
  estimate  one whole small problem: create, run the schedule, read c_n
  batch     several kept problems, one batched launch and their merges a pass
  job       a mix of problems created, chained on the device in one launch
            (run_job) and read out
  serve     a server kept by the program; a pass submits jobs and steps the
            server until all of them are done

Walks are grown from parameters, so a case's inputs are its problems' seeds.
Outputs are the merged state itself (pooled sums, sample counts, tours and the
per-sequence counters, which hold the trajectory digests) where the program
keeps going on the device, and the estimates where it reads them.
"""
import math
import random

import numpy as np
import torch

from paper_2002_03000_amd import ParallelFlatPERM, run_job
from paper_2002_03000_amd.sampler import Batch, Server


def listed():
    return [
        # plain flatPERM: one sequence, square lattice, walks of 20 steps: a
        # single wave's latency, and the estimates read after every epoch
        {"name": "plain square", "form": "epochs", "dim": 2, "n_max": 20, "N": 1, "tours": "1000", "read": True},
        # the smallest epochs: launches and host work count, so a program
        # replays them from a captured graph
        {"name": "small graph", "form": "graph", "dim": 2, "n_max": 50, "N": 200, "tours": "1", "replays": 8},
        # one small problem from its parameters to its estimates
        {"name": "small cubic from start", "form": "estimate", "dim": 3, "n_max": 40, "N": 96, "tours": "1,1,2,3"},
        # the square-lattice problem of the benchmark, one steady epoch
        {"name": "square 4096 x 500", "form": "epochs", "dim": 2, "n_max": 500, "N": 4096, "tours": "64"},
        # the cubic-lattice problem of the benchmark (its launch option
        # included), one steady epoch: the largest call
        {"name": "cubic 16384 x 1000", "form": "epochs", "dim": 3, "n_max": 1000, "N": 16384, "tours": "32",
         "sums_global": True},
        # Algorithm 1 (independent sequences), ragged sizes
        {"name": "independent 999 x 121", "form": "epochs", "dim": 2, "n_max": 121, "N": 999, "tours": "16",
         "mode": "independent"},
        # the end-to-end distance beside the weights, with the error estimate on
        {"name": "observables 500 x 250", "form": "epochs", "dim": 3, "n_max": 250, "N": 500, "tours": "16",
         "observables": True, "group_stats": True},
        # plain Rosenbluth sampling of long cubic walks (sums in global memory,
        # 64-bit occupancy keys)
        {"name": "rosenbluth 256 x 6000", "form": "epochs", "dim": 3, "n_max": 6000, "N": 256, "tours": "2",
         "mode": "rosenbluth"},
        # cubic walks past the short key format, two short epochs a pass
        {"name": "cubic 300 x 1500", "form": "epochs", "dim": 3, "n_max": 1500, "N": 300, "tours": "8,8"},
        # ragged problems of both lattices sharing batched launches
        {"name": "batch of 8", "form": "batch", "mix": 8, "count": 8, "n_lo": 60, "n_hi": 600, "N_lo": 20,
         "N_hi": 1000, "T": 8},
        # a mix of fresh problems chained on the device
        {"name": "job of 24", "form": "job", "mix": 24, "count": 24, "n_lo": 64, "n_hi": 700, "N_lo": 64,
         "N_hi": 512, "T": 16},
        # jobs served until their tour cap
        {"name": "serve 12 jobs", "form": "serve", "mix": 12, "count": 12, "n_lo": 50, "n_hi": 400, "N_lo": 256,
         "N_hi": 256, "T": 16},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(["epochs"] * 5 + ["graph", "estimate", "batch", "job", "serve"])
    dim = rng.choice([2, 3])
    if form == "epochs":
        mode = rng.choice(["shared"] * 4 + ["independent", "rosenbluth"])
        case = {"form": form, "dim": dim, "mode": mode}
        # (longer square walks, and longer sequences on their own, spend
        # seconds in their warm-up)
        longest = 6000 if (mode, dim) == ("rosenbluth", 3) else 2000 if dim == 3 else 800
        case["n_max"] = _log_uniform(rng, 20, 120 if mode == "independent" else longest)
        # no more work than the largest listed case, in all and along one sequence
        T = min(_log_uniform(rng, 1, 64), max(1, 32000 // case["n_max"]))
        top = max(1, min(1000 if mode == "independent" else 16384, int(1.5e8 / (T * case["n_max"]))))
        case["N"] = _log_uniform(rng, 1, top)
        case["tours"] = str(T)
        if mode != "independent" and rng.random() < 0.2:
            case["observables"] = True
        if rng.random() < 0.3:
            case["group_stats"] = True
        if rng.random() < 0.3:
            case["sums_global"] = True
        if rng.random() < 0.3:
            case["read"] = True
        return case
    if form == "graph":
        return {"form": form, "dim": dim, "n_max": _log_uniform(rng, 20, 200), "N": _log_uniform(rng, 16, 2000),
                "tours": str(rng.randint(1, 4)), "replays": rng.randint(1, 12)}
    if form == "estimate":
        return {"form": form, "dim": dim, "n_max": _log_uniform(rng, 20, 300), "N": _log_uniform(rng, 16, 400),
                "tours": rng.choice(["1,1,2", "1,1,2,3", "1,1,2,4"])}
    lo = _log_uniform(rng, 40, 200)
    case = {"form": form, "mix": rng.randrange(1 << 30), "count": rng.randint(4, 24), "n_lo": lo,
            "n_hi": lo + _log_uniform(rng, 20, 400), "N_lo": 256, "N_hi": 256, "T": 16}
    if form != "serve":
        case["N_lo"] = _log_uniform(rng, 16, 128)
        case["N_hi"] = case["N_lo"] + _log_uniform(rng, 16, 500)
        case["T"] = rng.randint(2, 16)
    return case


def _tours(case):
    return [int(t) for t in case["tours"].split(",")]


def _warm_up(T):
    """Epochs of 1, 1, 2, 4, ... tours up to T in all, as the workloads begin."""
    head = [1]
    while 2 * sum(head) <= T:
        head.append(sum(head))
    if sum(head) < T:
        head.append(T - sum(head))
    return head


def _mix(case):
    """The problems of a mix: (dim, n_max, N, T) each, the same for every seed."""
    rng = random.Random(case["mix"])
    return [(rng.choice([2, 3]), rng.randint(case["n_lo"], case["n_hi"]),
             _log_uniform(rng, case["N_lo"], case["N_hi"]), rng.randint(max(1, case["T"] // 2), case["T"]))
            for _ in range(case["count"])]


def _problem(case, seed):
    return ParallelFlatPERM(case["dim"], case["n_max"], case["N"], seed, mode=case.get("mode", "shared"),
                            group_stats=case.get("group_stats", False), observables=case.get("observables", False),
                            sums_global=case.get("sums_global", False))


def _epoch(problem, tours):
    problem.run_tours(tours)
    problem.merge_epoch()


def _state(problem):
    names = ["G", "HG", "MG", "t", "stats"]
    if problem.layout.obs_G:
        names.append("obs_G")
    if problem.cfg.flags & 1:      # group sums of the error estimate
        names += ["gsum", "gtours"]
    return {name: problem.view(name) for name in names}


def _estimates(problems):
    read = [p.estimates() for p in problems]
    return {"log_cn": np.concatenate([r[0] for r in read]), "hist": np.concatenate([r[1] for r in read]),
            "tours": np.array([r[2] for r in read])}


def prepare(case, seed):
    form = case["form"]
    state = {"case": case, "seed": seed}
    if form in ("epochs", "graph"):
        p = state["problem"] = _problem(case, seed)
        if p.mode != "rosenbluth":
            for T in _warm_up(max(_tours(case))):
                _epoch(p, T)
        if form == "graph":
            state["graph"] = p.epoch_graph(_tours(case)[0])
    elif form == "batch":
        mix = _mix(case)
        state["problems"] = [ParallelFlatPERM(d, n, N, seed, stream_id=i) for i, (d, n, N, _) in enumerate(mix)]
        state["tours"] = [T for _, _, _, T in mix]
        state["batch"] = Batch(len(mix))
        for p, T in zip(state["problems"], state["tours"]):
            for t in _warm_up(T):
                _epoch(p, t)
    elif form == "serve":
        state["server"] = Server(1 << 28, 16384)
    return state


def run(state):
    case, form = state["case"], state["case"]["form"]
    if form == "epochs":
        p = state["problem"]
        for T in _tours(case):
            _epoch(p, T)
        return dict(_state(p), **_estimates([p])) if case.get("read") and p.mode != "independent" else _state(p)
    if form == "graph":
        for _ in range(case["replays"]):
            state["graph"].launch()
        return _state(state["problem"])
    if form == "estimate":
        p = _problem(case, state["seed"])
        for T in _tours(case):
            _epoch(p, T)
        return _estimates([p])
    if form == "batch":
        state["batch"].run_tours(state["problems"], state["tours"])
        for p in state["problems"]:
            p.merge_epoch()
        names = ("G", "HG", "MG", "stats")
        return {name: torch.cat([p.view(name).reshape(-1) for p in state["problems"]]) for name in names}
    if form == "job":
        mix = _mix(case)
        problems = [ParallelFlatPERM(d, n, N, state["seed"], stream_id=i) for i, (d, n, N, _) in enumerate(mix)]
        run_job(problems, [_warm_up(T) + [T] for _, _, _, T in mix])
        return _estimates(problems)
    server = state["server"]
    ids = [server.submit(d, n, N, state["seed"], T, 4 * N * T, stream_id=i)
           for i, (d, n, N, T) in enumerate(_mix(case))]
    while sum(server.counts()[:2]):
        server.step()
    results = [server.result(j) for j in ids]
    infos = [server.info(j) for j in ids]
    for j in ids:
        server.release(j)
    return {"log_cn": np.concatenate([r[0] for r in results]), "hist": np.concatenate([r[1] for r in results]),
            "counts": np.array([[i["epochs"], i["tours"], i["steps"]] for i in infos])}


def _problems(case):
    """(dim, n_max, N, tours per sequence, mode) of every problem of a pass."""
    if "mix" not in case:
        tours = sum(_tours(case)) * case.get("replays", 1)
        return [(case["dim"], case["n_max"], case["N"], tours, case.get("mode", "shared"))]
    times = {"batch": 1, "job": 2, "serve": 4}[case["form"]]
    return [(d, n, N, T * times, "shared") for d, n, N, T in _mix(case)]


def work(case):
    """Bytes: the pooled sums and counts read and written, every sequence's
    counters read and written.  Operations: about one sample per length and
    tour (a flat histogram; a Rosenbluth walk is trapped after 71 steps on the
    square and about 3950 on the cubic lattice), each 157 (square) or 171
    (cubic) 32-bit operations of the method."""
    nbytes = flops = 0.0
    for dim, n_max, N, tours, mode in _problems(case):
        rows = N if mode == "independent" else 1
        nbytes += 2 * (24 * rows * (n_max + 1) + 88 * N)
        steps = n_max if mode != "rosenbluth" else min(n_max, 71 if dim == 2 else 3950)
        flops += N * tours * steps * (157 if dim == 2 else 171)
    return {"bytes": nbytes, "flops": flops}


# ---- the method in plain Python, for the smallest problems ---------------------


def _philox(counter, key):
    """Philox4x32-10 blocks (Salmon et al., SC'11) of uint64 counter arrays."""
    x0, x1, x2, x3 = counter
    k0, k1 = key
    low = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * x0, np.uint64(0xCD9E8D57) * x2
        x0, x1, x2, x3 = (p1 >> s32) ^ x1 ^ np.uint64(k0), p1 & low, (p0 >> s32) ^ x3 ^ np.uint64(k1), p0 & low
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x0, x1, x2


def _draws(key, s, t):
    """The random numbers of tour t of sequence s: (first word, 53-bit uniform) per event."""
    first = 0
    while True:
        k = np.arange(first, first + 256, dtype=np.uint64)
        zero = np.zeros_like(k)
        b0, b1, b2 = _philox((k, zero, zero + np.uint64(t), zero + np.uint64(s)), key)
        u = ((b1 >> np.uint64(5)) * np.uint64(1 << 26) + (b2 >> np.uint64(6))).astype(np.float64) * 2.0 ** -53
        yield from zip(b0.tolist(), u.tolist())
        first += 256


def _tour(dim, n_max, N, draws, G, MG, L, H, m):
    """One tour of one sequence: L and H are its sums and counts of the epoch,
    G and MG the pooled sums and tours (doubles: short walks stay in range)."""
    steps = [tuple(sign if a == axis else 0 for a in range(dim)) for axis in range(dim) for sign in (1, -1)]
    seen = float(MG + N * m)
    path, on = [(0,) * dim], {(0,) * dim}
    pending = []                      # (length, weight, copies left, end)
    W, decide = 1.0, False
    while True:
        n, end = len(path) - 1, path[-1]
        free = [q for q in (tuple(x + y for x, y in zip(end, d)) for d in steps) if q not in on]
        back = not free
        if free:
            b0, u = next(draws)
            if decide:
                total = G[n] + N * L[n]
                r = (W * seen) / total
                if r >= 1.0:
                    c = math.floor(r)
                    if not (r == c or u < (c + 1.0) - r):
                        c += 1
                    if c > 1:
                        W /= c
                        pending.append([n, W, c - 1])
                elif u < r:
                    W = total / seen
                else:
                    back = True
            if not back:
                site = free[b0 * len(free) >> 32]
                W *= len(free)
                path.append(site)
                on.add(site)
                n += 1
                L[n] += W
                H[n] += 1
                decide = True
                back = n == n_max
        if back:
            if not pending:
                return
            top = pending[-1]
            n, W = top[0], top[1]
            top[2] -= 1
            if not top[2]:
                pending.pop()
            on.difference_update(path[n + 1:])
            del path[n + 1:]
            decide = False


def exact(case, seed):
    """The estimates of one small problem run from its start, in plain Python."""
    if case["form"] != "estimate":
        return None
    dim, n_max, N, tours, _ = _problems(case)[0]
    if N * tours * n_max > 3e5:
        return None
    key = (seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF)
    G, HG, MG = np.zeros(n_max + 1), np.zeros(n_max + 1, dtype=np.uint64), 0
    run_so_far = 0
    for T in _tours(case):
        rows = []
        g = G.tolist()
        for s in range(N):
            L, H = [0.0] * (n_max + 1), [0] * (n_max + 1)
            for i in range(T):
                L[0] += 1.0
                H[0] += 1
                _tour(dim, n_max, N, _draws(key, s, run_so_far + i), g, MG, L, H, i + 1)
            rows.append(np.array(L))
            HG += np.array(H, dtype=np.uint64)
        run_so_far += T
        # the merge: an aligned pairwise tree over sequences
        rows += [np.zeros(n_max + 1)] * ((1 << max(0, N - 1).bit_length()) - N)
        while len(rows) > 1:
            rows = [rows[i] + rows[i + 1] for i in range(0, len(rows), 2)]
        G = G + rows[0]
        MG += N * T
    with np.errstate(divide="ignore"):
        return {"log_cn": np.log(G) - math.log(MG), "hist": HG, "tours": np.array([MG])}
