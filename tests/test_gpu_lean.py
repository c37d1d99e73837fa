"""The group-per-lane kernels (sim_lean.hpp) against the oracle where their
layout can go wrong: chunk and batch remainders, requests left out because no
job of the wavefront hosts them, several jobs per wavefront with a last
wavefront that is not full, exact ties, groups of different configurations,
unbounded deadlines, rows and statistics.  Bit-exact, so no tolerance."""
import dataclasses

import numpy as np
import pytest

import oracle
from gpu_common import compare, kernels_run, oracle_problem, say

pytestmark = pytest.mark.gpu


def _problem(seed, n, G, P, scales, M=9, cfgs=((1, 1), (2, 1), (4, 1)), hosts=3, burst=False, big=False):
    from paper_2302_11665_amd.workload import problems
    r = np.random.default_rng(seed)
    d = r.uniform(0.05, 0.4, M)
    if burst:
        d[:] = 0.125  # dyadic: equal arrivals give equal free times
    L = problems.stage_table(d, list(cfgs))
    if big:
        L *= 1e306  # finish times overflow to infinity
    t = np.sort(r.uniform(0.0, max(n, 1) * 0.02, n))
    if burst:
        t = np.floor(t * 4.0) / 4.0
    m = r.integers(0, M, n).astype(np.int32)
    gcfg = r.integers(-1, len(cfgs), (P, G)).astype(np.int32)
    mask = np.zeros((P, M), np.uint64)
    for p in range(P):
        live = [g for g in range(G) if gcfg[p, g] >= 0]
        for mm in range(M):
            if live and r.uniform() < 0.7:
                for g in r.choice(live, min(len(live), int(r.integers(1, hosts + 1))), replace=False):
                    mask[p, mm] |= np.uint64(1 << int(g))
    J = P * len(scales)
    return problems.Problem("lean", t, m, d, np.zeros(M, np.int64), np.array([s for s, _ in cfgs], np.int32),
                            np.array([k for _, k in cfgs], np.int32), L, gcfg, mask, np.array(scales),
                            np.unique(np.array([0, J // 2, J - 1], np.int32))[: J if n else 0])  # an empty row has no memory


def _check(api, pb, label, jobs=None):
    say(label)
    res = api.simulate_problem(pb)
    jobs = list(range(pb.n_jobs)) if jobs is None else jobs
    compare(res, oracle_problem(pb, jobs, pb.finish_jobs.tolist()), len(pb.t), label)


@pytest.fixture
def api(monkeypatch):
    from paper_2302_11665_amd import api as a
    monkeypatch.setenv("ALPASERVE_PATH", "shared")
    return a


@pytest.mark.parametrize("n", [0, 1, 7, 8, 9, 63, 64, 65, 129, 500])
@pytest.mark.parametrize("G", [1, 5, 16, 33])
def test_remainders(api, n, G):
    _check(api, _problem(n * 100 + G, n, G, 6, [0.0, 2.0, np.inf]), f"n={n} G={G}")


@pytest.mark.parametrize("G,hosts,cfgs", [(2, 2, ((8, 1),)), (4, 4, ((1, 1), (3, 1))), (8, 8, ((2, 1),)),
                                          (16, 16, ((1, 1),)), (32, 20, ((1, 1), (2, 1))), (64, 40, ((1, 1),))])
def test_exact_ties(api, G, hosts, cfgs):
    """Bursts of equal arrivals and dyadic latencies: free times tie in every bit."""
    _check(api, _problem(G, 700, G, 5, [4.0, 40.0], cfgs=cfgs, hosts=hosts, burst=True), f"ties G={G}")


@pytest.mark.parametrize("stages", [1, 4])
@pytest.mark.parametrize("G", [33, 64])
def test_minimum_across_rows_of_lanes(api, G, stages):
    """Wavefronts of one job (33 to 64 groups): model m on group m alone, on one
    group of each 16, or on the first and the last group, with ties between them."""
    pb = _problem(G + stages, 900, G, 3, [1.5, 6.0], M=G, cfgs=((stages, 1),), burst=True)
    gcfg = np.zeros_like(pb.group_cfg)
    mask = np.zeros_like(pb.host_mask)
    for m in range(G):
        mask[0, m] = np.uint64(1 << m)
        mask[1, m] = np.uint64(sum(1 << g for g in range(m % 16, G, 16)))
        mask[2, m] = np.uint64(1 | 1 << (G - 1))
    _check(api, dataclasses.replace(pb, group_cfg=gcfg, host_mask=mask), f"rows of lanes G={G} stages={stages}")


@pytest.mark.parametrize("G,P", [(1, 4100), (4, 1500), (16, 2051), (32, 1537), (64, 1100)])
def test_several_jobs_per_wavefront(api, G, P):
    """More jobs than SIMDs: several per wavefront, the last wavefront part empty."""
    pb = _problem(P, 150, G, P, [3.0])
    _check(api, pb, f"G={G} P={P}", sorted({*range(0, P, 41), *range(P - 70, P), *pb.finish_jobs.tolist()}))


@pytest.mark.parametrize("G,P,per_simd,mixes", [
    (1, 1, 1.01, True), (1, 5, 2.3, False), (4, 1, 3.1, True), (4, 3, 3.2, True), (6, 2, 4.5, True), (12, 1, 9.0, True),
    (16, 7, 5.0, True), (32, 1, 1.5, True), (32, 2, 3.0, False), (33, 1, 1.2, False)])
def test_many_scales_on_few_placements(api, G, P, per_simd, mixes):
    """Few placements at many SLO scales: wavefronts of one scale would hold one
    job a placement, so they take jobs of several scales (never 64 lanes, which
    hold one job, nor where a placement's jobs fill the wavefronts anyway)."""
    import torch
    K = int(per_simd * 4 * torch.cuda.get_device_properties(0).multi_processor_count) // P
    scales = np.geomspace(0.2, 30.0, K)
    scales[K // 3], scales[K // 2] = 0.0, np.inf
    pb = _problem(G * 10 + P, 137, G, P, scales.tolist())
    names = kernels_run(lambda: api.simulate_problem(pb))
    assert any("shared_kernel" in n and n.count("true") == 1 for n in names) == mixes, sorted(names)
    _check(api, pb, f"G={G} P={P} K={K}", sorted({*range(0, P * K, 7), *range(P * K - 70, P * K), K // 3, K // 2,
                                                  *pb.finish_jobs.tolist()}))


@pytest.mark.parametrize("G,P,scales,rows", [
    (1, 4100, [3.0], [0, 1, 2, 63, 64, 4099]), (4, 3001, [2.0], [5, 1, 2998, 3000, 6]), (16, 2051, [4.0], [2, 3, 0, 1, 2050]),
    (16, 2049, [1.0, 6.0], [1, 3, 4096, 4097, 0]), (5, 1, np.geomspace(0.5, 20.0, 2100).tolist(), [0, 1, 7, 2099, 1050]),
    (32, 2100, [2.0], [1, 0, 2099]), (64, 1500, [2.0], [1499, 3, 0])])
def test_rows_of_jobs_that_share_a_wavefront(api, G, P, scales, rows):
    """Rows of several jobs of one wavefront, of its first and its last job, of a
    job that hosts less than the others, in any order, at one and at many scales."""
    pb = _problem(G + P, 200, G, P, scales, hosts=2)
    pb = dataclasses.replace(pb, finish_jobs=np.array(rows, np.int32))
    J = P * len(scales)
    _check(api, pb, f"rows G={G} P={P} K={len(scales)}", sorted({*range(0, J, 97), *rows}))


def test_rows_do_not_lengthen_full_launches(api):
    """Two wavefronts on every SIMD: a few rows are written by the wavefronts that
    simulate their jobs anyway (wavefronts of their own took 1.4 times the time)."""
    import torch
    P = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    pb = _problem(3, 5000, 64, P, [2.0], cfgs=((1, 1),))
    best = []
    for fin in ([], [0, P // 3, P // 2, P - 1]):
        dp = api.upload(dataclasses.replace(pb, finish_jobs=np.array(fin, np.int32)))
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            api.run(dp)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        best.append(min(t))
    say("rows on full SIMDs: ms without and with", best)
    assert best[1] < 1.2 * best[0], best


def test_infinite_finish_times(api):
    _check(api, _problem(5, 300, 12, 4, [1.0, np.inf], big=True), "infinite finish times")


@pytest.mark.parametrize("G,P,K,table", [
    (3, 30, 1, {}), (16, 2100, 1, {}), (16, 1030, 3, {}), (24, 9, 3, {}), (64, 5, 2, {}),
    (1, 3, 2, dict(M=64, cfgs=tuple((8, k) for k in range(1, 33))))])  # the largest table
def test_statistics(api, G, P, K, table):
    import torch
    from paper_2302_11665_amd import sim
    pb = dataclasses.replace(_problem(G + P, 333, G, P, [1.0, 2.5, np.inf][:K], **table), finish_jobs=np.zeros(0, np.int32))
    dp = api.upload(pb)
    M, J = len(pb.d_single), pb.n_jobs
    ms = torch.empty((J, M), dtype=torch.int64, device="cuda")
    busy = torch.empty((J, G), dtype=torch.float64, device="cuda")
    say(f"statistics G={G} P={P} K={K}")
    sim.as_simulate_stats(dp.t, dp.model, dp.d_single, dp.cfg_stages, dp.stage_lat, dp.group_cfg, dp.host_mask,
                          dp.slo_scale, dp.out_served, dp.out_digest, ms, busy)
    served, dg = dp.out_served.cpu().numpy(), sim.u64(dp.out_digest)
    ms, busy = ms.cpu().numpy(), busy.cpu().numpy()
    lib = oracle.lib()
    for j in sorted({*range(0, J, max(1, J // 60)), J - 1}):
        p, k = divmod(j, K)
        s, d, om, ob = lib.simulate_job_stats(pb.t, pb.model, pb.d_single, pb.cfg_stages, pb.stage_lat,
                                              pb.group_cfg[p], pb.host_mask[p], pb.slo_scale[k])
        assert (served[j], tuple(int(x) for x in dg[j])) == (s, d), j
        assert np.array_equal(ms[j], om) and busy[j].tobytes() == ob.tobytes(), j


@pytest.mark.parametrize("G", [1, 4, 16, 32, 64])
def test_segments(api, G):
    """Jobs with segments of their own: empty, short and long ones, rows shorter
    than the segment, jobs that name nothing."""
    import torch
    from paper_2302_11665_amd import sim
    pb = _problem(G, 900, G, 3, [1.0])
    offs = np.array([0, 0, 1, 8, 72, 200, 900])
    t = np.concatenate([np.sort(pb.t[a:b]) - (pb.t[a] if b > a else 0) for a, b in zip(offs[:-1], offs[1:])])
    place = np.array([0, 1, 2, 0, 1, 2, 0, 7, 1], np.int32)
    seg = np.array([0, 1, 2, 3, 4, 5, 5, 1, 9], np.int32)
    sc = np.array([1.0, 2.0, 3.0, 2.0, np.inf, 2.5, 0.0, 1.0, 1.0])
    fin, stride = np.array([5, 0, 3], np.int32), 300
    d = sim.to_device
    served = torch.empty(9, dtype=torch.int64, device="cuda")
    dg = torch.empty((9, 2), dtype=torch.int64, device="cuda")
    out = torch.full((3, stride), float("nan"), dtype=torch.float64, device="cuda")
    say(f"segments G={G}")
    sim.as_simulate_jobs(d(t), d(pb.model), d(offs), d(pb.d_single), pb.cfg_stages, d(pb.stage_lat), d(pb.group_cfg),
                         d(pb.host_mask), d(sim.jobs_to_bytes(place, seg, sc)), served, None, dg, fin, out, stride)
    served, dg, out = served.cpu().numpy(), sim.u64(dg), out.cpu().numpy()
    lib = oracle.lib()
    for j in range(9):
        if place[j] >= 3 or seg[j] >= 6:
            assert served[j] == 0 and not dg[j].any()
            continue
        a, b = offs[seg[j]], offs[seg[j] + 1]
        s, g, f = lib.simulate_job(t[a:b], pb.model[a:b], pb.d_single, pb.cfg_stages, pb.stage_lat,
                                   pb.group_cfg[place[j]], pb.host_mask[place[j]], sc[j], want_finish=True)
        assert (served[j], tuple(int(x) for x in dg[j])) == (s, g), j
        if j in fin:
            row, k = out[list(fin).index(j)], min(b - a, stride)
            assert row[:k].tobytes() == f[:k].tobytes() and np.isnan(row[k:]).all(), j


@pytest.mark.parametrize("G,hosts,rate", [(3, 3, 0.02), (16, 4, 0.02), (40, 12, 0.02), (6, 2, 0.2)])
@pytest.mark.parametrize("segments", [2, 9, 10, 40])
def test_fix_ups(api, monkeypatch, G, hosts, rate, segments):
    """The speculative kernels' fix-ups: cold segment starts, saved states every
    64 requests, fewer and more segments than rounds (the last jobs then whole);
    busy groups, whose runs meet late or never, and idle ones."""
    monkeypatch.setenv("ALPASERVE_PATH", "spec")
    monkeypatch.setenv("ALPASERVE_SPEC_SEGMENTS", str(segments))
    monkeypatch.setenv("ALPASERVE_SPEC_WARMUP", "0")
    monkeypatch.setenv("ALPASERVE_SPEC_CKPT", "64")
    monkeypatch.setenv("ALPASERVE_SPEC_CAP", str(1 << 40))
    pb = _problem(G * 100 + segments, 6000, G, 70, [2.0], hosts=hosts)
    pb.t *= rate / 0.02
    _check(api, pb, f"fix-ups G={G} segments={segments}", sorted({*range(0, 70, 3), *pb.finish_jobs.tolist()}))
