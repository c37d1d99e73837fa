"""The work that users have this framework do, as cases to be timed.

Every case goes through the package's public entry points (the ctypes binding
`sim` and the upload-once layer `api`).  The workloads are seeded and
synthetic, with the shapes of `workload/problems.py`: Gamma arrivals per model
by rate and CV, power-law or equal rates over the models, even stage latency
tables, SLO scales as multiples of the single-device latency.

Kinds of case:
  score   as_simulate_placements: placements x SLO scales over one trace
  sweep   as_simulate_jobs: one placement, jobs that each have their own trace
  stats   as_simulate_stats: a few selections with the heuristic's statistics
  batch   as_simulate_batched: the dynamic-batching simulation
  search  a whole placement search (partition, greedy, beam, fast or alg2)

All results are whole numbers or IEEE binary64 values whose operations and
order the entry points define, so every output is compared exactly.
"""
from __future__ import annotations

import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np

from paper_2302_11665_amd import api, sim
from paper_2302_11665_amd.workload import gen, problems

GIB = problems.GIB_MIB


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # One call on a toy cluster (4 models, every placement form of 4
        # devices): what a unit test or a notebook runs; launch and latency.
        dict(name="score_tiny", kind="score", models=4, groups=4, cfgs="1:1,2:1,4:1", layout="partition",
             placements=273, base=0, replicas=1, rate=20.0, exponent=0.0, cv=1.0, requests=1200, d_lo=0.1,
             d_hi=0.25, scales=1, finish=4),
        # The first step of Alg. 1 at several SLO scales: every single
        # replica of 16 models on 4 pipelines of 4 devices.
        dict(name="score_first_step", kind="score", models=16, groups=4, cfgs="4:1", layout="same",
             placements=64, base=0, replicas=-1, rate=64.0, exponent=0.0, cv=3.0, requests=38400, d_lo=0.1,
             d_hi=0.4, scales=8, finish=4),
        # A late step of Alg. 1: a selection that fills most of the memory
        # of 32 two-stage groups, and every further addition to it.
        dict(name="score_late_step", kind="score", models=32, groups=32, cfgs="2:1", layout="same",
             placements=777, base=128, replicas=-1, rate=128.0, exponent=0.0, cv=2.0, requests=76801,
             d_lo=0.05, d_hi=0.8, scales=1, finish=0),
        # Heterogeneous placements (groups of different pipeline depths, as
        # Alg. 2's remainder groups make them) at three SLO scales.
        dict(name="score_mixed", kind="score", models=24, groups=12, cfgs="1:1,2:1,4:2,8:1", layout="group",
             placements=333, base=0, replicas=3, rate=200.0, exponent=0.5, cv=4.0, requests=60001, d_lo=0.05,
             d_hi=0.4, scales=3, finish=2),
        # A quarter of an hour of heavy traffic over a thousand placements.
        dict(name="score_quarter_hour", kind="score", models=64, groups=16, cfgs="4:2", layout="same",
             placements=1000, base=0, replicas=0, rate=1000.0, exponent=0.9, cv=4.0, requests=900000,
             d_lo=0.03, d_hi=0.11, scales=1, finish=8),
        # The benchmark's size: 8192 placements over an hour at 1000 req/s.
        dict(name="score_hour", kind="score", models=64, groups=16, cfgs="4:2", layout="same",
             placements=8192, base=0, replicas=0, rate=1000.0, exponent=0.9, cv=4.0, requests=3600000,
             d_lo=0.03, d_hi=0.11, scales=1, finish=16),
        # SLO-attainment curves over rate, CV and SLO scale for a placement of
        # 32 models on 64 single devices, each grid point with its own trace.
        dict(name="sweep_devices", kind="sweep", models=32, groups=64, cfgs="1:1", mem_gb=32, rates=8, cvs=8,
             slos=8, rate=128.0, rate_lo=0.25, rate_hi=4.0, cv_hi=8.0, slo_hi=20.0, requests=38400,
             d_lo=0.05, d_hi=0.8, finish=8),
        # The same curves on 4 pipelines of 4 devices.
        dict(name="sweep_pipelines", kind="sweep", models=16, groups=4, cfgs="4:1", mem_gb=64, rates=10,
             cvs=10, slos=10, rate=64.0, rate_lo=0.25, rate_hi=4.0, cv_hi=8.0, slo_hi=20.0, requests=19200,
             d_lo=0.1, d_hi=0.4, finish=4),
        # One step of the fast heuristic run by hand: a few selections with
        # their per-model served counts and per-group busy times.
        dict(name="stats_selections", kind="stats", models=32, groups=64, cfgs="1:1", layout="same",
             placements=6, base=0, replicas=4, rate=128.0, exponent=0.0, cv=2.0, requests=76800, d_lo=0.05,
             d_hi=0.8, scales=1),
        # The dynamic-batching experiment's shape: 32 instances of one model
        # on 16 four-stage groups, 8 SLO scales, batches of up to 4.
        dict(name="batch_experiment", kind="batch", models=32, groups=16, cfgs="4:1", layout="same",
             placements=256, base=0, replicas=4, rate=128.0, exponent=0.0, cv=4.0, requests=76800,
             d_lo=0.151, d_hi=0.151, scales=8, finish=2, max_batch=4, beta=1.0),
        # A whole reduced Alg. 2: Alg. 1 on four uniform partitions of 16 devices.
        dict(name="search_partitions", kind="search", how="partition", models=16, devices=16, mem_gb=16,
             parts="4:4:1,4:2:2,8:8:1,16:4:4", w_lo=2.0, w_hi=6.0, rate=64.0, exponent=0.5, cv=2.0,
             requests=38400, d_lo=0.1, d_hi=0.4, scale=5.0, beam=1),
        # A whole run of the fast heuristic on 64 single devices.
        dict(name="search_fast", kind="search", how="fast", models=32, devices=64, mem_gb=32, parts="1:1:1",
             w_lo=1.0, w_hi=13.0, rate=128.0, exponent=0.0, cv=2.0, requests=19200, d_lo=0.05, d_hi=0.8,
             scale=5.0, beam=0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _ints(rng, lo, hi):
    return int(round(_log(rng, lo, hi)))


def _load(rng, devices, d_lo, d_hi):
    """A total rate (req/s) from light load to overload of the devices."""
    return round(rng.choice([0.2, 0.5, 0.8, 1.2]) * rng.uniform(0.8, 1.2) * devices * 2.0 / (d_lo + d_hi), 3)


def draw(rng):
    kind = rng.choice(["score", "score", "score", "sweep", "stats", "batch", "search"])
    models = _ints(rng, 2, 64)
    d_lo = round(_log(rng, 0.03, 0.2), 4)
    d_hi = round(d_lo * rng.uniform(1.0, 8.0), 4)
    cv = round(rng.uniform(1.0, 6.0), 2)
    if kind == "search":
        models = _ints(rng, 4, 20)
        devices = rng.choice([4, 8, 16])
        parts = rng.choice(["1:1:1", "2:2:1", "2:1:2", "1:1:1,2:2:1", "2:1:2,4:4:1", "1:1:1,2:2:1,4:2:2"])
        rate = _load(rng, devices, d_lo, d_hi)
        return dict(kind=kind, how=rng.choice(["partition", "greedy", "beam", "fast", "alg2"]), models=models,
                    devices=devices, mem_gb=rng.choice([8, 12, 16]), parts=parts, w_lo=2.0, w_hi=6.0, rate=rate,
                    exponent=rng.choice([0.0, 0.5]), cv=cv, requests=_ints(rng, 500, 12000),
                    d_lo=d_lo, d_hi=d_hi, scale=rng.choice([2.0, 5.0, 10.0]), beam=rng.choice([1, 2, 3]))
    groups = _ints(rng, 1, 64)
    cfgs = rng.choice(["1:1", "2:1", "4:1", "4:2", "8:1", "3:1", "1:2"])
    if kind == "sweep":
        S, k = (int(x) for x in cfgs.split(":"))
        rate = _load(rng, groups * S * k, d_lo, d_hi)
        rates, cvs, slos = (rng.randint(1, 8) for _ in range(3))
        return dict(kind=kind, models=models, groups=groups, cfgs=cfgs, mem_gb=S * k * rng.choice([16, 32]),
                    rates=rates, cvs=cvs, slos=slos, rate=rate, rate_lo=0.5, rate_hi=2.0, cv_hi=cv, slo_hi=20.0,
                    requests=_ints(rng, 200, 40000), d_lo=d_lo, d_hi=d_hi,
                    finish=rng.choice([0, 0, 1, 5]))
    layout = rng.choice(["same", "same", "group"])
    if layout == "group":
        cfgs = rng.choice(["1:1,2:1", "4:1,2:2,1:1", "8:1,4:2,3:1", "2:1,1:2,4:1,8:1"])
    width = np.mean([int(c.split(":")[0]) * int(c.split(":")[1]) for c in cfgs.split(",")])
    rate = _load(rng, groups * float(width), d_lo, d_hi)
    case = dict(kind=kind, models=models, groups=groups, cfgs=cfgs, layout=layout, base=0, rate=rate,
                exponent=rng.choice([0.0, 0.5, 0.9]), cv=cv, d_lo=d_lo, d_hi=d_hi)
    if kind == "score":
        n = _log(rng, 300, 1000000)
        scales = rng.choice([1, 1, 1, 2, 5, 8])
        jobs = _log(rng, 8, min(8192.0, 2.0e9 / n))
        case.update(placements=max(1, int(jobs / scales)), scales=scales, finish=rng.choice([0, 0, 1, 4]),
                    replicas=rng.choice([0, 1, 2, 3, 5, -1]), requests=int(n))
        if case["replicas"] == -1:
            case["base"] = _ints(rng, 1, max(2, models * groups // 8))
        case["finish"] = min(case["finish"], case["placements"] * scales)
    elif kind == "stats":
        case.update(placements=_ints(rng, 1, 64), scales=rng.choice([1, 1, 1, 3]), replicas=rng.choice([0, 1, 2, 4]),
                    requests=_ints(rng, 300, 100000))
    else:
        n = _log(rng, 300, 60000)
        scales = rng.choice([1, 4, 8])
        jobs = _log(rng, 8, min(2048.0, 1.0e8 / n))
        case.update(placements=max(1, int(jobs / scales)), scales=scales, finish=rng.choice([0, 1, 2]),
                    replicas=rng.choice([0, 1, 2, 4]), requests=int(n),
                    max_batch=rng.choice([1, 2, 4, 8, 16]), beta=rng.choice([0.0, 0.5, 1.0]))
        case["finish"] = min(case["finish"], case["placements"] * scales)
    return case


# ------------------------------------------------------------ host workloads

def _rates(case):
    return problems.c4_rates(case["models"], case["rate"], case["exponent"])


def _trace(seed, rates, cv, n):
    """The first n requests of a Gamma trace (fixed counts, so that every seed
    gives outputs of one shape)."""
    span = (n + 4.0 * max(cv, 1.0) * math.sqrt(n) + 16.0) / float(np.sum(rates))
    while True:
        t, m = gen.trace(seed, rates, cv, span)
        if len(t) >= n:
            return t[:n], m[:n]
        span *= 1.5


def _models(case, seed):
    """Single-device latencies, configurations (S, k), stage table."""
    d = problems._uniform_range(seed, gen.PURPOSE_LATENCY, case["models"], case["d_lo"], case["d_hi"])
    cfgs = [tuple(int(x) for x in c.split(":")) for c in case["cfgs"].split(",")]
    return d, cfgs, problems.stage_table(d, cfgs)


def _scales(k):
    return np.array([5.0]) if k == 1 else np.geomspace(1.0, 20.0, k)


def _perms(seed, rows, n):
    return gen.permutations(seed, gen.PURPOSE_PERMUTE, 0, rows, n)


def _layout(case, seed, cfgs, P):
    """Group configurations [P, G] and the number of groups each placement uses [P]."""
    G = case["groups"]
    if case["layout"] == "same":
        return np.zeros((P, G), np.int32), np.full(P, G)
    u = gen.uniforms(gen.key(seed, gen.PURPOSE_PERMUTE, 1 << 40), P * G).reshape(P, G)
    if case["layout"] == "group":
        return (u * len(cfgs)).astype(np.int32), np.full(P, G)
    pick = (u[:, 0] * len(cfgs)).astype(np.int32)  # "partition": G devices in equal groups
    used = np.array([max(1, G // (S * k)) for S, k in cfgs])[pick]
    return np.where(np.arange(G)[None] < used[:, None], pick[:, None], -1).astype(np.int32), used


def _masks(case, seed, used, P):
    """Hosting masks [P, M]: replicas > 0 on the first groups of seeded
    permutations, 0: replicas by rate, -1: one selection of `base` replicas
    and in placement p the p-th addition that it does not hold yet."""
    M, G, r = case["models"], case["groups"], case["replicas"]
    if r == -1:
        order = _perms(seed, 1, M * G)[0]
        held, free = order[: case["base"]], np.sort(order[case["base"]:])
        sel = np.zeros(M, np.uint64)
        for x in held:
            sel[x // G] |= np.uint64(1 << int(x % G))
        m = np.tile(sel, (P, 1))
        if len(free):
            add = free[np.arange(P) % len(free)]
            m[np.arange(P), add // G] |= np.left_shift(np.uint64(1), (add % G).astype(np.uint64))
        return m
    if r == 0:
        share = _rates(case) / case["rate"]
        reps = np.clip(np.floor(0.75 * M * share + 0.5), 1, G).astype(np.int64)
    else:
        reps = np.full(M, min(r, G), np.int64)
    perms = _perms(seed, P * M, G).reshape(P, M, G).astype(np.int64)
    host = np.zeros((P, M, G), bool)
    np.put_along_axis(host, perms, np.arange(G)[None, None] < reps[None, :, None], axis=2)
    if (used < G).any():  # fold the groups that a placement does not have onto those it has
        for p in np.nonzero(used < G)[0]:
            full = host[p]
            folded = np.zeros_like(full)
            for g in range(G):
                folded[:, g % used[p]] |= full[:, g]
            host[p] = folded
    bits = np.left_shift(np.uint64(1), np.arange(G, dtype=np.uint64))
    return (host * bits).sum(axis=2, dtype=np.uint64)


def _finish_jobs(case, jobs):
    n = min(case.get("finish", 0), jobs)
    return (np.arange(n, dtype=np.int64) * jobs // max(n, 1)).astype(np.int32)


def _problem(case, seed):
    """The workload of a score, stats or batch case as a problems.Problem."""
    d, cfgs, L = _models(case, seed)
    t, m = _trace(seed, _rates(case), case["cv"], case["requests"])
    P = case["placements"]
    gcfg, used = _layout(case, seed, cfgs, P)
    scales = _scales(case["scales"])
    return problems.Problem(case["kind"], t, m, d, np.zeros(len(d), np.int64), np.array([S for S, _ in cfgs], np.int32),
                            np.array([k for _, k in cfgs], np.int32), L, gcfg, _masks(case, seed, used, P), scales,
                            _finish_jobs(case, P * len(scales)))


def _sweep(case, seed):
    """One placement (models put on seeded permutations of the groups until
    no memory is left) and a rate x CV x SLO grid of jobs with their own traces."""
    d, cfgs, L = _models(case, seed)
    M, G = case["models"], case["groups"]
    w = problems._weights_mib(seed, M, 1.0, 13.0)
    room = np.full(G, case["mem_gb"] * GIB)
    mask = np.zeros(M, np.uint64)
    for r in range(G):
        order = _perms(seed + 1 + r, 1, M)[0]
        perm = _perms(seed + 1001 + r, 1, G)[0]
        for x, mm in enumerate(order):
            g = int(perm[x % G])
            if w[mm] <= room[g] and not (int(mask[mm]) >> g) & 1:
                mask[mm] |= np.uint64(1 << g)
                room[g] -= w[mm]
    grid = [(i, j, k) for i in range(case["rates"]) for j in range(case["cvs"]) for k in range(case["slos"])]
    step = lambda lo, hi, i, n: lo * (hi / lo) ** (i / max(n - 1, 1))  # noqa: E731
    grow = [step(case["rate_lo"], case["rate_hi"], i, case["rates"]) for i in range(case["rates"])]
    specs = [(seed * 100003 + x, [case["rate"] * grow[i] / M] * M, step(1.0, case["cv_hi"], j, case["cvs"]),
              int(case["requests"] * grow[i])) for x, (i, j, k) in enumerate(grid)]
    with ThreadPoolExecutor(min(16, os.cpu_count() or 1)) as ex:
        segs = list(ex.map(lambda s: _trace(*s), specs))
    offs = np.zeros(len(segs) + 1, np.int64)
    np.cumsum([len(s[0]) for s in segs], out=offs[1:])
    J = len(grid)
    return problems.SweepProblem(
        "sweep", np.concatenate([s[0] for s in segs]), np.concatenate([s[1] for s in segs]).astype(np.int32), offs, d,
        np.array([S for S, _ in cfgs], np.int32), L, np.zeros((1, G), np.int32), mask.reshape(1, M),
        np.zeros(J, np.int32), np.arange(J, dtype=np.int32),
        np.array([step(1.0, case["slo_hi"], k, case["slos"]) for _, _, k in grid]), _finish_jobs(case, J))


def _search(case, seed):
    d = problems._uniform_range(seed, gen.PURPOSE_LATENCY, case["models"], case["d_lo"], case["d_hi"])
    w = problems._weights_mib(seed, case["models"], case["w_lo"], case["w_hi"])
    t, m = _trace(seed, _rates(case), case["cv"], case["requests"])
    parts, cfgs = [], []
    for c, p in enumerate(case["parts"].split(",")):
        size, S, k = (int(x) for x in p.split(":"))
        cfgs.append((S, k))
        G = max(1, case["devices"] // size)
        parts.append({"group_cfg": np.full(G, c, np.int32),
                      "group_mem_mib": np.full(G, size * case["mem_gb"] * GIB, np.int64)})
    return problems.GreedyProblem("search", t, m, d, w, np.array([S for S, _ in cfgs], np.int32),
                                  np.array([k for _, k in cfgs], np.int32), problems.stage_table(d, cfgs), parts,
                                  case["scale"])


# ---------------------------------------------------------------- the passes

def prepare(case, seed):
    """Device-resident inputs and output buffers, as `api.upload` makes them."""
    import torch
    kind = case["kind"]
    if kind == "score":
        return {"case": case, "dp": api.upload(_problem(case, seed))}
    if kind == "sweep":
        return {"case": case, "ds": api.upload_sweep(_sweep(case, seed))}
    if kind in ("stats", "batch"):
        pb = _problem(case, seed)
        s = {"case": case, "dp": api.upload(pb)}
        J, M, G = pb.n_jobs, case["models"], case["groups"]
        if kind == "stats":
            s["model_served"] = torch.empty((J, M), dtype=torch.int64, device="cuda")
            s["busy"] = torch.empty((J, G), dtype=torch.float64, device="cuda")
        return s
    gp = _search(case, seed)
    dev = {k: sim.to_device(v) for k, v in (("t", gp.t), ("model", gp.model), ("d_single", gp.d_single),
                                            ("stage_lat", gp.stage_lat))}
    return {"case": case, "gp": gp, "dev": dev}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "score":
        dp = state["dp"]
        api.run(dp)
        out = {"served": dp.out_served, "attain": dp.out_attain, "digest": dp.out_digest}
        if dp.out_finish is not None:
            out["finish"] = dp.out_finish
        return out
    if kind == "sweep":
        ds = state["ds"]
        api.run_sweep(ds)
        out = {"served": ds.out_served, "attain": ds.out_attain, "digest": ds.out_digest}
        if ds.out_finish is not None:
            out["finish"] = ds.out_finish
        return out
    if kind == "stats":
        dp = state["dp"]
        sim.as_simulate_stats(dp.t, dp.model, dp.d_single, dp.cfg_stages, dp.stage_lat, dp.group_cfg, dp.host_mask,
                              dp.slo_scale, dp.out_served, dp.out_digest, state["model_served"], state["busy"])
        return {"served": dp.out_served, "digest": dp.out_digest, "model_served": state["model_served"],
                "busy": state["busy"]}
    if kind == "batch":
        dp = state["dp"]
        sim.as_simulate_batched(dp.t, dp.model, dp.d_single, dp.cfg_stages, dp.stage_lat, dp.group_cfg, dp.host_mask,
                                dp.slo_scale, case["max_batch"], case["beta"], dp.out_served, dp.out_digest,
                                dp.finish_jobs if len(dp.finish_jobs) else None, dp.out_finish, queue_cap=1 << 20)
        out = {"served": dp.out_served, "digest": dp.out_digest}
        if dp.out_finish is not None:
            out["finish"] = dp.out_finish
        return out
    gp, dev = state["gp"], state["dev"]
    args = (dev["t"], dev["model"], dev["d_single"], gp.cfg_stages, dev["stage_lat"], gp.weight_mib)
    how = case["how"]
    if how == "partition":
        r = sim.as_partition_search(*args, gp.partitions, gp.slo_scale)
        return {"best": r["best_mask"].view(np.int64), "served": r["best_served"], "partition": r["best_partition"],
                "parts": np.array(r["part_served"], np.int64)}
    if how == "alg2":
        devices = gp.cfg_stages * gp.cfg_k
        r = sim.as_placement_search(*args, devices, case["devices"], 2, case["mem_gb"] * GIB, 0.2, 4.0, 2, case["beam"],
                                    gp.slo_scale)
        cells = np.full((2, 2 + 64 + case["models"]), -1, np.int64)  # up to two buckets
        for b, x in enumerate(r["buckets"]):
            cells[b, :2] = x["served"], x["devices"]
            cells[b, 2:2 + len(x["group_cfg"])] = x["group_cfg"]
            cells[b, 66:] = x["mask"].view(np.int64)
        return {"served": r["served"], "buckets": cells,
                "counts": np.array([r["n_bucket_configs"], r["n_device_splits"], r["n_kept_splits"], r["n_problems"]])}
    part = gp.partitions[0]
    args = args + (part["group_cfg"], part["group_mem_mib"], gp.slo_scale)
    if how == "greedy":
        r = sim.as_greedy_placement(*args)
    elif how == "beam":
        r = sim.as_beam_placement(*args, case["beam"])
    else:
        r = sim.as_fast_placement(*args)
    steps = np.full((4096, 3), -1, np.int64)
    steps[: len(r["steps"])] = np.array(r["steps"], np.int64).reshape(-1, 3)
    return {"best": r["best_mask"].view(np.int64), "served": r["best_served"], "n_steps": r["n_steps"], "steps": steps}


def tolerance(case):
    return "exact"


# ------------------------------------------------------------------ its work

def work(case):
    """Bytes: the trace, the placements and the outputs once each (a search:
    the trace once).  Operations: per simulated request that has a host, the
    comparisons of its hosts' free times, a max and an add per stage, the
    deadline and its test, in binary64."""
    M = case["models"]
    n = float(case["requests"])
    if case["kind"] == "search":
        flops, steps = 0.0, 0.0
        w = 512.0 * (case["w_lo"] + case["w_hi"])
        for p in case["parts"].split(","):
            size, S, k = (int(x) for x in p.split(":"))
            G = max(1, case["devices"] // size)
            reps = G * min(M, size * case["mem_gb"] * GIB / w)  # replicas that fit = steps taken
            H = reps / (2.0 * M)
            cand = 1.0 if case["how"] == "fast" else M * G / 2.0 * (case["beam"] if case["how"] == "beam" else 1)
            flops += reps * cand * n * min(1.0, H) * (max(H - 1, 0) + 2 * S + 2)
            steps += reps
        return {"bytes": 12.0 * n + 20.0 * steps, "flops": flops}
    cfgs = [tuple(int(x) for x in c.split(":")) for c in case["cfgs"].split(",")]
    S = float(np.mean([s for s, _ in cfgs]))
    G = case["groups"]
    if case["kind"] == "sweep":
        J = case["rates"] * case["cvs"] * case["slos"]
        grow = [case["rate_lo"] * (case["rate_hi"] / case["rate_lo"]) ** (i / max(case["rates"] - 1, 1))
                for i in range(case["rates"])]
        n *= float(np.mean(grow))
        H = min(G, G * min(M, case["mem_gb"] / 7.0) / M)
        ev = J * n * min(1.0, H)
        return {"bytes": 12.0 * J * n + 48.0 * J + 8.0 * min(case["finish"], J) * n,
                "flops": ev * (max(H - 1, 0) + 2 * S + 2)}
    P, K = case["placements"], case["scales"]
    J = P * K
    share = _rates(case) / case["rate"]
    if case["replicas"] == -1:
        H = np.full(M, (case["base"] + 1) / M)
    elif case["replicas"] == 0:
        H = np.clip(np.floor(0.75 * M * share + 0.5), 1, G)
    else:
        H = np.full(M, float(min(case["replicas"], G)))
    hosted = np.minimum(1.0, H)
    ops = float((share * hosted * (np.maximum(H - 1, 0) + 2 * S + 2)).sum())
    out = 32.0 * J + 8.0 * case.get("finish", 0) * n + (J * (M + G) * 8.0 if case["kind"] == "stats" else 0.0)
    return {"bytes": 12.0 * n + P * (8.0 * M + 4.0 * G) + out, "flops": J * n * ops}


# ---------------------------------------------------- the definition in numpy

def _simulate(t, m, d, L, gcfg, host, scale, rows, stats):
    """All jobs at once, request by request.  t, m: [n] or [n, J] (m = -1: no
    request); gcfg [J, G]; host bool [J, M, G]; scale [J]."""
    J, G = gcfg.shape
    S = L.shape[2]
    F = np.zeros((J, G, S))
    ar = np.arange(J)
    served = np.zeros(J, np.int64)
    fin = np.full((len(rows), len(t)), np.nan)
    slow = L.max(axis=2)
    busy, ms = np.zeros((J, G)), np.zeros((J, len(d)), np.int64)
    cfg = np.maximum(gcfg, 0)
    for i in range(len(t)):
        ti, mi = np.broadcast_to(t[i], J), np.broadcast_to(m[i], J)
        there = mi >= 0
        mi = np.maximum(mi, 0)
        h = host[ar, mi] & there[:, None]
        hosted = h.any(axis=1)
        g = np.where(h, F[:, :, 0], np.inf).argmin(axis=1)
        g = np.where(hosted, np.where(h[ar, g], g, h.argmax(axis=1)), 0)
        lat = L[mi, cfg[ar, g]]
        f, fs = ti, np.empty((J, S))
        for s in range(S):
            f = np.maximum(f, F[ar, g, s]) + lat[:, s]
            fs[:, s] = f
        ok = hosted & ~(f > ti + scale * d[mi])
        F[ar[ok], g[ok]] = fs[ok]
        served += ok
        if stats:
            busy[ar[ok], g[ok]] += slow[mi[ok], cfg[ar[ok], g[ok]]]
            ms[ar[ok], mi[ok]] += 1
        for r, j in enumerate(rows):
            if there[j]:
                fin[r, i] = f[j] if ok[j] else (-1.0 if hosted[j] else -2.0)
    return served, fin, ms, busy


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("score", "sweep", "stats"):
        return None  # whole numbers (search), or events out of trace order (batch)
    n, G = float(case["requests"]), case["groups"]
    J = case["placements"] * case["scales"] if kind != "sweep" else case["rates"] * case["cvs"] * case["slos"]
    if kind == "sweep":
        n *= case["rate_hi"]
    if n * (2.0e-4 + J * (G + case["models"] / 8) * 2.0e-8) > 12.0:
        return None
    if kind == "sweep":
        sp = _sweep(case, seed)
        lens = np.diff(sp.seg_offsets)
        J, n = len(lens), int(lens.max())
        t, m = np.zeros((n, J)), np.full((n, J), -1, np.int64)
        for j in range(J):
            a, b = sp.seg_offsets[j], sp.seg_offsets[j + 1]
            t[: b - a, j], m[: b - a, j] = sp.t[a:b], sp.model[a:b]
        gcfg, mask, scale, rows = np.repeat(sp.group_cfg, J, 0), np.repeat(sp.host_mask, J, 0), sp.job_scale, sp.finish_jobs
        d, L, total = sp.d_single, sp.stage_lat, lens
    else:
        sp = _problem(case, seed)
        K = len(sp.slo_scale)
        t, m, d, L, rows, total = sp.t, sp.model, sp.d_single, sp.stage_lat, sp.finish_jobs, len(sp.t)
        gcfg, mask, scale = np.repeat(sp.group_cfg, K, 0), np.repeat(sp.host_mask, K, 0), np.tile(sp.slo_scale, len(sp.group_cfg))
    host = ((mask[:, :, None] >> np.arange(G, dtype=np.uint64)) & np.uint64(1)).astype(bool)
    served, fin, ms, busy = _simulate(t, m, d, L, gcfg, host, scale, rows, kind == "stats")
    if kind == "stats":
        return {"served": served, "digest": None, "model_served": ms, "busy": busy}
    out = {"served": served, "attain": np.where(total > 0, served / np.maximum(total, 1), 0.0), "digest": None}
    if len(rows):
        stride = int(lens[rows].max()) if kind == "sweep" else len(t)
        out["finish"] = fin[:, :stride]
    return out
