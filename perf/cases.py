"""Measured cases of the TT-cross library: what a user's program does with it.

Each case is a plain dict: "kind" says which entry points it goes through, the
rest are sizes and options.  The kinds:

  solve  one problem: TTCross.run, then its ranks and cores, the cores copied
         into a GPU buffer of the program's (tt_cross_get_cores with
         on_device), and, with "points", TTCross.tt_eval at that many
         multi-indices
  batch  many small problems together: batch_run, then every problem's cores
         copied one after the other into one GPU buffer
  serve  a list of requests submitted at once to a Server and waited for, with
         each request's stats and cores read back into one host buffer
  tteval TTCross.tt_eval of a solved problem at m multi-indices on the GPU
  error  TTCross.sampled_error of a solved problem over R samples
  fneval fn_eval: the generating function at m multi-indices, which lie on the
         GPU or, with "host", in a numpy array

Handles, servers and index arrays are made in prepare(), as a program keeps
them between calls.  The seed chooses the sample entries a solve starts from
(and so its first pivot), the indices, and the parameters of drawn problem
lists.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2407_11290_amd import (FN_BIMAXWELL, FN_HILBERT, FN_MAXWELL, FN_MAXWELL_2D2V, FN_MAXWELL_3D3V,
                                  PIVOT_GREEDY, PIVOT_ROOK, PREC_AUTO, PREC_FP64)
from paper_2407_11290_amd._lib import check, load
from paper_2407_11290_amd.api import Server, TTCross, batch_run, fn_eval
from paper_2407_11290_amd.workloads import batch_mix, served_trace

FNS = {"hilbert": FN_HILBERT, "bimaxwell": FN_BIMAXWELL, "maxwell": FN_MAXWELL, "maxwell2d2v": FN_MAXWELL_2D2V,
       "maxwell3d3v": FN_MAXWELL_3D3V}


def _text(sizes):
    """Mode sizes (or prescribed ranks) as a case holds them: "64x64x64"."""
    return "x".join(str(x) for x in sizes)


def _sizes(text):
    return [int(x) for x in text.split("x")] if text else []


def _solve(name, fn, n, eps, **more):
    case = {"name": name, "kind": "solve", "fn": fn, "n": _text(n), "eps": eps, "grid": 2, "caps": "",
            "rook": False, "fp64": True, "r_max": 64, "points": 0}
    case.update(more)
    if not name:
        del case["name"]
    return case


def listed():
    return [
        # the smallest solve: a 3D tensor of 32^3 entries in one block, where launches and waits are the time
        _solve("solve_small", "hilbert", [32] * 3, 1e-10, grid=1),
        # the benchmark's workload: 6D Hilbert, 64 points a mode, 2^6 subtensor blocks, to eps in FP64
        _solve("solve_hilbert6d", "hilbert", [64] * 6, 1e-8),
        # the phase-space workload: eps that the precision policy sweeps in FP32, with its sampled-error check
        _solve("solve_maxwell6d_fp32", "maxwell", [128] * 6, 1e-6, fp64=False),
        # odd modes and uneven blocks, two Maxwellians in FP64, and the result evaluated at a program's own points
        _solve("solve_ragged_points", "bimaxwell", [37, 101, 75, 53, 89], 1e-9, grid=3, points=10007),
        # the paper's Table 6 at n = 1000 and its prescribed ranks: superblocks of several hundred MB
        _solve("solve_hilbert3d_n1000", "hilbert", [1000] * 3, 0.0, caps="25x25"),
        # the paper's largest kinetic tensor (Table 5) at its shape and prescribed ranks
        _solve("solve_maxwell3d3v", "maxwell3d3v", [800, 400] * 3, 0.0, caps="10x5x30x5x20"),
        # superblocks beyond device memory: Alg. 1 inside every block on residual factors
        _solve("solve_rook_n20000", "hilbert", [20000] * 3, 1e-8, rook=True, caps="20x20"),
        # the mixed batch of the batched workload: 512 uneven problems in one call
        {"name": "batch_512", "kind": "batch", "count": 512, "eps": 1e-6},
        # served solves, a burst of requests at both accuracies
        {"name": "serve_128", "kind": "serve", "count": 128, "slots": 64, "budget_gib": 32},
        # the finished TT read at a million points
        {"name": "tt_eval_1m", "kind": "tteval", "fn": "hilbert", "n": _text([64] * 6), "eps": 1e-8, "m": 1000000},
        # Sec. 5's error over a million entries of a solved tensor
        {"name": "error_1m", "kind": "error", "fn": "maxwell", "n": _text([128] * 6), "eps": 1e-6, "m": 1000000},
        # bulk element access of the phase-space tensor in the FP32 of FP32 sweeps
        {"name": "fn_eval_16m", "kind": "fneval", "fn": "maxwell", "n": _text([128] * 6), "m": 1 << 24, "fp32": True,
         "host": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "rook", "batch", "serve", "tteval", "error", "fneval"])
    if kind == "solve":
        fixed = rng.random() < 0.3
        # prescribed ranks: tensors whose residuals stay far from rounding at them
        fn = rng.choice(["hilbert", "maxwell2d2v", "maxwell3d3v"] if fixed else
                        ["hilbert", "hilbert", "bimaxwell", "maxwell", "maxwell2d2v", "maxwell3d3v"])
        d = {"maxwell": 6, "maxwell2d2v": 4, "maxwell3d3v": 6}.get(fn) or rng.randint(3, 6)
        hi = 1200 if d == 3 else 300 if d == 4 else 150
        n = [_log_int(rng, 30 if fixed else 12, hi) for _ in range(d)]
        if rng.random() < 0.4:
            n = [n[0]] * d
        return _solve("", fn, n, 0.0 if fixed else 10.0 ** rng.uniform(-9.0, -3.0), grid=rng.randint(1, 3),
                      caps=_text(rng.randint(2, 7) for _ in range(d - 1)) if fixed else "",
                      fp64=rng.random() < 0.6, r_max=rng.choice([16, 32, 40]),
                      points=_log_int(rng, 10, 50000) if rng.random() < 0.3 else 0)
    if kind == "rook":
        return _solve("", "hilbert", [_log_int(rng, 100, 10000) for _ in range(3)], 10.0 ** rng.uniform(-8.0, -4.0),
                      rook=True, r_max=32, grid=rng.randint(1, 3))
    if kind == "batch":
        return {"kind": "batch", "count": _log_int(rng, 3, 400), "eps": 10.0 ** rng.uniform(-7.0, -4.0)}
    if kind == "serve":
        return {"kind": "serve", "count": _log_int(rng, 4, 100), "slots": rng.choice([8, 32, 64]), "budget_gib": 24}
    if kind in ("tteval", "error"):
        fn = rng.choice(["hilbert", "bimaxwell", "maxwell"])
        d = 6 if fn == "maxwell" else rng.randint(3, 6)
        return {"kind": kind, "fn": fn, "n": _text(_log_int(rng, 16, 130) for _ in range(d)),
                "eps": 10.0 ** rng.uniform(-9.0, -4.0), "m": _log_int(rng, 100, 1000000)}
    fn = rng.choice(["hilbert", "bimaxwell", "maxwell", "maxwell2d2v", "maxwell3d3v"])
    d = {"maxwell": 6, "maxwell2d2v": 4, "maxwell3d3v": 6}.get(fn) or rng.randint(3, 7)
    host = rng.random() < 0.3
    return {"kind": "fneval", "fn": fn, "n": _text(_log_int(rng, 16, 500) for _ in range(d)),
            "m": _log_int(rng, 50, 100000 if host else 10000000), "fp32": rng.random() < 0.5, "host": host}


def _params(fn, seed):
    """Two Maxwellians drawn as in the batched workload; the other functions take their defaults."""
    if fn != "bimaxwell":
        return None
    rng = np.random.default_rng([7, seed])
    out = []
    for _ in range(2):
        out += [float(rng.uniform(0.5, 2.0)), *[float(x) for x in rng.uniform(-2.0, 2.0, 3)],
                float(rng.uniform(0.5, 2.0))]
    return out + [8.0]


def _indices(n, m, seed):
    rng = np.random.default_rng([11, seed])
    return np.stack([rng.integers(0, nj, m, dtype=np.int32) for nj in n], axis=1)


def _handle(case, seed):
    n = _sizes(case["n"])
    d = len(n)
    p = TTCross(n, case["eps"], FNS[case["fn"]], _params(case["fn"], seed), seed=seed,
                r_max=case.get("r_max", 64), precision=PREC_FP64 if case.get("fp64", False) else PREC_AUTO,
                grid=[case.get("grid", 2)] * d, pivot=PIVOT_ROOK if case.get("rook") else PIVOT_GREEDY)
    if case.get("caps"):
        p.set_rank_caps(_sizes(case["caps"]))
    return p


def _rank_room(case):
    """Doubles that the cores of a solve can need at most (its rank caps)."""
    n, caps = _sizes(case["n"]), _sizes(case["caps"])
    d, r = len(n), [1]
    for k in range(1, d):
        r.append(min(math.prod(n[:k]), math.prod(n[k:]), case["r_max"], caps[k - 1] if caps else case["r_max"]))
    r.append(1)
    return sum(r[k] * n[k] * r[k + 1] for k in range(d))


def _cores_into(p, buf, off):
    """The solved problem's cores G_1..G_d, concatenated, into the GPU buffer
    buf from entry off on; their length."""
    return check(load().tt_cross_get_cores(p.h, ctypes.c_void_p(buf.data_ptr() + 8 * off), buf.numel() - off, 1))


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if "n" in case:
        state["n"] = _sizes(case["n"])
    if kind == "solve":
        state["p"] = _handle(case, seed)
        state["cores"] = torch.zeros(_rank_room(case), dtype=torch.float64, device="cuda")
        if case["points"]:
            state["idx"] = torch.from_numpy(_indices(_sizes(case["n"]), case["points"], seed)).cuda()
    elif kind == "batch":
        state["ps"] = [TTCross(s.n, s.eps, s.fn_id, s.params, seed=seed + s.seed, grid=s.grid)
                       for s in batch_mix(case["count"], gen_seed=2024 + seed, eps=case["eps"])]
        state["cores"] = torch.zeros(200000 + 16000 * case["count"], dtype=torch.float64, device="cuda")
    elif kind == "serve":
        state["reqs"] = served_trace(case["count"], trace_seed=7 + seed)
        state["srv"] = Server(int(case["budget_gib"]) << 30, max_slots=case["slots"])
        state["cores"] = np.zeros(800000 + 50000 * case["count"])
    elif kind in ("tteval", "error"):
        p = _handle(case, seed)
        p.run()
        state["p"] = p
        state["seed"] = 1000 + seed
        if kind == "tteval":
            state["idx"] = torch.from_numpy(_indices(_sizes(case["n"]), case["m"], seed)).cuda()
    else:
        idx = _indices(_sizes(case["n"]), case["m"], seed)
        state["idx"] = idx if case["host"] else torch.from_numpy(idx).cuda()
        state["params"] = _params(case["fn"], seed)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        p = state["p"]
        status = p.run()
        _cores_into(p, state["cores"], 0)
        out = {"status": status, "ranks": p.ranks(), "cores": state["cores"]}
        if case["points"]:
            out["values"] = p.tt_eval(state["idx"])
        return out
    if kind == "batch":
        status, lengths, off = batch_run(state["ps"]), [], 0
        for p in state["ps"]:
            lengths.append(_cores_into(p, state["cores"], off))
            off += lengths[-1]
        return {"status": np.array(status), "lengths": np.array(lengths), "cores": state["cores"]}
    if kind == "serve":
        srv, buf, off = state["srv"], state["cores"], 0
        tickets = [srv.submit(q.n, q.eps, q.fn_id, q.params, seed=q.seed) for q in state["reqs"]]
        status, ranks = [], np.zeros((len(tickets), 8), dtype=np.int32)
        for i, t in enumerate(tickets):
            status.append(srv.wait(t)[0])
            st, cores = srv.result(t)
            srv.release(t)
            ranks[i, :len(st["ranks"])] = st["ranks"]
            buf[off:off + cores.size] = cores
            off += cores.size
        return {"status": np.array(status), "ranks": ranks, "cores": buf}
    if kind == "tteval":
        return state["p"].tt_eval(state["idx"])
    if kind == "error":
        return state["p"].sampled_error(case["m"], state["seed"])
    return fn_eval(FNS[case["fn"]], state["n"], state["idx"], state["params"], fp32=case["fp32"])


def _typical_ranks(case):
    """Ranks a solve of this kind ends with, for work()."""
    n = _sizes(case["n"])
    d = len(n)
    if case.get("caps"):
        want = _sizes(case["caps"])
    elif case["fn"] == "hilbert":
        want = [min(case.get("r_max", 64), 1 + int(1.5 * -math.log10(max(case["eps"], 1e-16))))] * (d - 1)
    else:
        want = [2] * (d - 1)
    r = [1]
    for k in range(1, d):
        r.append(int(min(want[k - 1], math.prod(n[:k]), math.prod(n[k:]))))
    return r + [1]


def _solve_work(case):
    """Cores written; a solve has to form every residual of its superblocks
    (rook: of the rows and columns of its pivots), r_k multiply-adds each."""
    n, r = _sizes(case["n"]), _typical_ranks(case)
    d = len(n)
    cores = sum(r[k] * n[k] * r[k + 1] for k in range(d))
    flops = 0
    for k in range(1, d):
        rows, cols = r[k - 1] * n[k - 1], n[k] * r[k + 1]
        looked = r[k] * (rows + cols) if case.get("rook") else rows * cols
        flops += looked * 2 * r[k]
    return {"bytes": 8 * cores, "flops": flops}


# operations of one entry: sums, products and one function call's worth of arithmetic
_FN_FLOPS = {"hilbert": 8, "bimaxwell": 40, "maxwell": 30, "maxwell2d2v": 50, "maxwell3d3v": 60}


def work(case):
    kind, m = case["kind"], case.get("m", 0)
    if kind == "solve":
        w = _solve_work(case)
        if case["points"]:
            w["bytes"] += case["points"] * (4 * len(_sizes(case["n"])) + 8)
        return w
    if kind in ("batch", "serve"):
        if kind == "batch":
            specs = batch_mix(case["count"], eps=case["eps"])
        else:
            specs = served_trace(case["count"])
        ws = [_solve_work({"n": _text(s.n), "eps": s.eps, "fn": "hilbert" if s.fn_id == FN_HILBERT else "bimaxwell",
                           "r_max": 32}) for s in specs]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    n = _sizes(case["n"])
    d = len(n)
    if kind == "fneval":
        return {"bytes": m * (4 * d + (4 if case["fp32"] else 8)), "flops": m * _FN_FLOPS[case["fn"]]}
    r = _typical_ranks(case)
    cores = sum(r[k] * n[k] * r[k + 1] for k in range(d))
    flops = m * 2 * sum(r[k] * r[k + 1] for k in range(d))
    if kind == "tteval":
        return {"bytes": m * (4 * d + 8) + 8 * cores, "flops": flops}
    return {"bytes": 8 * cores, "flops": flops + m * _FN_FLOPS[case["fn"]]}


def _entries(fn, n, idx, params):
    """The tensor's entries at 0-based indices in 64 bits (the paper's formulas)."""
    i = idx.astype(np.float64)
    d = len(n)
    if fn == "hilbert":
        return 1.0 / ((i + 1.0).sum(axis=1) + (1 - d))
    if fn == "maxwell":
        x = [i[:, j] / n[j] for j in range(3)]
        v = [-8.0 + (i[:, 3 + j] + 0.5) * (16.0 / n[3 + j]) for j in range(3)]
        rho = 1.0 + 0.5 * np.sin(2 * np.pi * x[0]) * np.cos(2 * np.pi * x[1])
        q = (v[0] - 0.3 * np.sin(2 * np.pi * x[2])) ** 2 + v[1] ** 2 + v[2] ** 2
        return rho * (2 * np.pi) ** -1.5 * np.exp(-q / 2.0)
    if fn == "bimaxwell":
        vmax = params[10]
        out = np.zeros(len(i))
        for m in range(2):
            rho, u, t = params[5 * m], params[5 * m + 1:5 * m + 4], params[5 * m + 4]
            q = np.zeros(len(i))
            for c in range(3):
                j = d - 3 + c
                q += (-vmax + (i[:, j] + 0.5) * (2.0 * vmax / n[j]) - u[c]) ** 2
            out += rho * (2 * np.pi * t) ** -1.5 * np.exp(-q / (2.0 * t))
        return out
    pre = em = ep = 0.0
    for w in range(2 if fn == "maxwell2d2v" else 3):
        x = -0.5 + (i[:, 2 * w] + 0.5) / n[2 * w]
        v = -3.0 + (i[:, 2 * w + 1] + 0.5) * (6.0 / n[2 * w + 1])
        rho, t = 1.0 + 0.875 * np.sin(2 * np.pi * x), 0.5 + 0.4 * np.sin(2 * np.pi * x)
        pre = pre + rho / (2.0 * np.sqrt(2 * np.pi * t))
        em = em + (v - 0.75) ** 2 / (2.0 * t)
        ep = ep + (v + 0.75) ** 2 / (2.0 * t)
    return pre * (np.exp(-em) + np.exp(-ep))


def exact(case, seed):
    """The tensor's own entries where a pass returns values at given indices.
    Cores have no such value (they depend on which pivots the search takes),
    nor has the sampled error of one particular approximation."""
    kind = case["kind"]
    if kind == "solve" and case["points"] and case["eps"] > 0.0:
        vals = _entries(case["fn"], _sizes(case["n"]), _indices(_sizes(case["n"]), case["points"], seed), _params(case["fn"], seed))
        return {"status": None, "ranks": None, "cores": None, "values": vals}
    if kind in ("tteval", "fneval"):
        return _entries(case["fn"], _sizes(case["n"]), _indices(_sizes(case["n"]), case["m"], seed), _params(case["fn"], seed))
    return None
