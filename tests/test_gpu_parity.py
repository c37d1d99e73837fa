"""GPU parity: the HIP path (through the C-ABI) against the CPU oracle on the
same seeded inputs, bit-exact.  Sizes are chosen so the oracle finishes in
seconds while the GPU runs still span several LDS chunks, ragged tails, every
lanes-per-job shape and every padded stage count."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import compare, kernels_run, oracle_problem, say  # noqa: E402
from oracle_pins import random_case  # noqa: E402

pytestmark = pytest.mark.gpu


# kernel selections the library offers (environment variables read per call):
# the group-per-lane kernels, the general LDS-staged kernel
# with one or two groups per lane, and the segment-speculative kernels
NEVER_GIVE_UP = {"ALPASERVE_SPEC_CAP": str(1 << 40)}
VARIANTS = {
    "shared": {"ALPASERVE_PATH": "shared"},
    "lds": {"ALPASERVE_PATH": "lds", "ALPASERVE_GPL": "1"},
    "lds_gpl2": {"ALPASERVE_PATH": "lds", "ALPASERVE_GPL": "2"},
    # one lane per job over trace segments run at once and reconciled: the
    # default segment count, an odd count, and 64 segments (short and empty
    # segments whose states never meet: many reconciliation rounds).  A cap on
    # one re-run's requests replaces the fix-ups' own limits, which would leave
    # most of these short traces to the fallback kernels.
    "spec": {"ALPASERVE_PATH": "spec"},
    "spec_seg7": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "7", **NEVER_GIVE_UP},
    "spec_seg64": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "64", **NEVER_GIVE_UP},
    # no warm-up: every segment starts from the empty state
    "spec_seg7_cold": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "7", "ALPASERVE_SPEC_WARMUP": "0",
                       **NEVER_GIVE_UP},
    # a warm-up shorter than a segment
    "spec_seg16_warm100": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "16",
                           "ALPASERVE_SPEC_WARMUP": "100", **NEVER_GIVE_UP},
    # saved states every 64 requests: re-runs stop at the first one they meet
    "spec_seg5_ck64": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "5", "ALPASERVE_SPEC_WARMUP": "0",
                       "ALPASERVE_SPEC_CKPT": "64", **NEVER_GIVE_UP},
    # re-runs give up after 64 requests without meeting the old results (cold
    # segments rarely meet that soon): the group-per-lane kernels launched behind
    # the pipeline, gated on that flag, produce the results
    "spec_seg7_giveup": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "7", "ALPASERVE_SPEC_WARMUP": "0",
                         "ALPASERVE_SPEC_CAP": "64"},
    # cold segments under the fix-ups' own limits
    "spec_seg7_cold_limits": {"ALPASERVE_PATH": "spec", "ALPASERVE_SPEC_SEGMENTS": "7", "ALPASERVE_SPEC_WARMUP": "0"},
}


@pytest.fixture(scope="module")
def gpu_api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2302_11665_amd import api, sim
    say("library:", sim.as_version())
    return api


@pytest.fixture(params=sorted(VARIANTS))
def gpu(request, gpu_api, monkeypatch):
    for k in ("ALPASERVE_PATH", "ALPASERVE_GPL", "ALPASERVE_SPEC_SEGMENTS", "ALPASERVE_SPEC_WARMUP",
              "ALPASERVE_SPEC_CKPT", "ALPASERVE_SPEC_CAP"):
        monkeypatch.delenv(k, raising=False)
    for k, v in VARIANTS[request.param].items():
        monkeypatch.setenv(k, v)
    say("variant", request.param)
    return gpu_api


def test_variants_reach_the_kernels_they_name(gpu_api, monkeypatch):
    """The variants that are there for the fix-ups finish on them, and the one
    that is there for the fallback ends on the kernels behind the gate."""
    from paper_2302_11665_amd.workload import problems
    pb = problems.c4_heavy(duration=60.0, n_placements=64, n_finish=2)
    for name, env in sorted(VARIANTS.items()):
        if env.get("ALPASERVE_PATH") != "spec" or "ALPASERVE_SPEC_CAP" not in env:
            continue
        with monkeypatch.context() as mp:
            for k, v in env.items():
                mp.setenv(k, v)
            times = kernels_run(lambda: gpu_api.simulate_problem(pb))
        gated = sum(t for n, t in times.items() if "shared_kernel" in n)
        say("variant", name, "gated kernels", round(gated, 1), "us")
        assert any("spec_pass0" in n for n in times) and (gated > 1000.0) == (name == "spec_seg7_giveup"), (name, times)


def test_c1_all_placements(gpu):
    from paper_2302_11665_amd.workload import problems
    pb = problems.c1_tiny()
    say("c1_tiny", pb.n_jobs, len(pb.t))
    res = gpu.simulate_problem(pb)
    compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), len(pb.t), "c1")


def test_c2_greedy_step(gpu):
    from paper_2302_11665_amd.workload import problems
    pb = problems.c2_greedy_step()
    say("c2_greedy_step", pb.n_jobs, len(pb.t))
    res = gpu.simulate_problem(pb)
    compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), len(pb.t), "c2")


def test_c4_reduced_all_jobs(gpu):
    from paper_2302_11665_amd.workload import problems
    pb = problems.c4_heavy(duration=45.0, n_placements=600, n_finish=7)
    say("c4 reduced", pb.n_jobs, len(pb.t))
    res = gpu.simulate_problem(pb)
    compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), len(pb.t), "c4 reduced")


def test_c4_reduced_no_rows(gpu):
    """The same jobs with no per-request output rows: on the speculative path
    the digest step then runs as a dispatch of its own (with rows it shares
    the output-row dispatch)."""
    import dataclasses
    from paper_2302_11665_amd.workload import problems
    pb = problems.c4_heavy(duration=45.0, n_placements=600, n_finish=7)
    pb = dataclasses.replace(pb, finish_jobs=np.zeros(0, np.int32))
    say("c4 reduced, no rows", pb.n_jobs, len(pb.t))
    res = gpu.simulate_problem(pb)
    compare(res, oracle_problem(pb), len(pb.t), "c4 reduced no rows")


def test_c3_candidate_steps_every_partition(gpu):
    """Greedy-step job sets of every partition of the 64-device workload:
    single-replica candidates from the empty selection, and candidates on top
    of a random memory-feasible partial selection (2 minutes of trace)."""
    from paper_2302_11665_amd.workload import problems
    gp = problems.c3_greedy(duration=120.0)
    rng = np.random.default_rng(3)
    M = len(gp.d_single)
    for pi, part in enumerate(gp.partitions):
        G = len(part["group_cfg"])
        cands = [(m, g) for m in range(M) for g in range(G)]
        pick = rng.choice(len(cands), size=min(96, len(cands)), replace=False)
        base = np.zeros(M, np.uint64)
        used = np.zeros(G, np.int64)
        for _ in range(G * 2):  # random partial selection within memory
            m, g = int(rng.integers(M)), int(rng.integers(G))
            if used[g] + gp.weight_mib[m] <= part["group_mem_mib"][g]:
                base[m] = np.uint64(int(base[m]) | (1 << g))
                used[g] += gp.weight_mib[m]
        masks = []
        for q, k in enumerate(pick):
            m, g = cands[k]
            row = (base.copy() if q % 2 else np.zeros(M, np.uint64))
            row[m] = np.uint64(int(row[m]) | (1 << g))
            masks.append(row)
        pb = problems.Problem(f"c3_step_{pi}", gp.t, gp.model, gp.d_single, gp.weight_mib, gp.cfg_stages,
                              gp.cfg_k, gp.stage_lat, np.tile(part["group_cfg"], (len(masks), 1)),
                              np.array(masks, np.uint64), np.array([gp.slo_scale]),
                              np.array([0, len(masks) - 1], np.int32))
        say("c3 partition", pi, part["label"], pb.n_jobs)
        res = gpu.simulate_problem(pb)
        compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), len(pb.t), f"c3 p{pi}")


def _random_problem(rng, G, S, n, P, K, M=None, mixed=True, max_hosts=4):
    """Random problem with exactly G groups, up to S stages, mixed configs;
    a hosted model has 1..max_hosts hosting groups."""
    from paper_2302_11665_amd.workload.problems import Problem
    M = M or int(rng.integers(1, 9))
    C = int(rng.integers(1, 5)) if mixed else 1
    cfg_stages = rng.integers(1, S + 1, C).astype(np.int32)
    cfg_stages[0] = S
    L = rng.uniform(0.01, 0.3, (M, C, S))
    gaps = rng.exponential(0.02, n)
    gaps[rng.random(n) < 0.2] = 0.0
    t = np.cumsum(gaps)
    model = rng.integers(0, M, n).astype(np.int32)
    gcfg = rng.integers(0, C, (P, G)).astype(np.int32)
    gcfg[rng.random((P, G)) < 0.1] = -1
    gcfg[:, 0] = np.maximum(gcfg[:, 0], 0)
    masks = np.zeros((P, M), np.uint64)
    for p in range(P):
        for m in range(M):
            if rng.random() < 0.15:
                continue  # unhosted model
            k = int(rng.integers(1, min(G, max_hosts) + 1))
            valid = [g for g in range(G) if gcfg[p, g] >= 0]
            for g in rng.choice(valid, size=min(k, len(valid)), replace=False):
                masks[p, m] = np.uint64(int(masks[p, m]) | (1 << int(g)))
    d = L[:, 0, :].sum(axis=1) * rng.uniform(0.5, 1.5, M)
    scales = np.array(sorted(rng.choice([0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 5.0, np.inf], size=K, replace=False)))
    J = P * K
    fin = np.unique(rng.integers(0, J, size=min(3, J))).astype(np.int32)
    return Problem("random", t, model, d, np.zeros(M, np.int64), cfg_stages, np.ones(C, np.int32), L,
                   gcfg, masks, scales, fin)


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 11, 16, 17, 32, 33, 64])
def test_random_shapes_every_width(gpu, G):
    rng = np.random.default_rng(100 + G)
    for S in (1, 3, 8):
        n = int(rng.choice([1, 63, 64, 65, 2047, 2049, 4500]))
        P = int(rng.integers(1, 40))
        K = int(rng.integers(1, 4))
        pb = _random_problem(rng, G, S, n, P, K)
        say("random", G, S, n, P, K)
        res = gpu.simulate_problem(pb)
        compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), n, f"random G={G} S={S} n={n}")


@pytest.mark.parametrize("G", [3, 9, 16, 32, 64])
def test_random_many_hosts(gpu, G):
    """Models on up to every group: the dispatch over more than two hosts
    (the further hosts read in one batch, the winning row read again) and
    over more than eight (the loop past the batch), with unhosted models
    beside them."""
    rng = np.random.default_rng(700 + G)
    for S in (1, 4):
        for mixed in (False, True):
            n = int(rng.choice([65, 2049, 5000]))
            pb = _random_problem(rng, G, S, n, int(rng.integers(1, 24)), 2, M=int(rng.integers(2, 12)),
                                 mixed=mixed, max_hosts=G)
            say("many hosts", G, S, n, mixed)
            res = gpu.simulate_problem(pb)
            compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), n, f"many hosts G={G} S={S} n={n}")


@pytest.mark.parametrize("G", [4, 16])
def test_full_depth_mixed_configs(gpu, G):
    """Every configuration equally deep but with latencies of its own, groups
    of one job on different configurations: the reconciliation rounds'
    per-lane latency rows with no stage past any group's depth (the
    cold-start and forced-segment variants re-run most segments)."""
    rng = np.random.default_rng(900 + G)
    for S in (1, 2, 4):
        n = int(rng.choice([2049, 6000]))
        pb = _random_problem(rng, G, S, n, int(rng.integers(8, 40)), 2, mixed=True)
        pb.cfg_stages[:] = S
        say("full depth mixed", G, S, n, len(pb.cfg_stages))
        res = gpu.simulate_problem(pb)
        compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), n, f"full depth G={G} S={S} n={n}")


def test_tiny_cases_like_the_brute_force_pins(gpu):
    """The random tiny problems the oracle's brute-force pin uses, one call each."""
    from paper_2302_11665_amd.workload.problems import Problem
    rng = np.random.default_rng(2024)
    for k in range(40):
        t, model, prob, sigma = random_case(rng, dyadic=(k % 2 == 0))
        G = len(prob["group_cfg"])
        pb = Problem("tiny", np.asarray(t, float), model, prob["d_single"], np.zeros(len(prob["d_single"]), np.int64),
                     prob["cfg_stages"], np.ones(len(prob["cfg_stages"]), np.int32), prob["stage_lat"],
                     prob["group_cfg"].reshape(1, G), prob["host_mask"].reshape(1, -1), np.array([sigma]),
                     np.array([0], np.int32))
        res = gpu.simulate_problem(pb)
        compare(res, oracle_problem(pb, finish_jobs=[0]), len(t), f"tiny {k}")


def test_empty_trace_and_zero_jobs(gpu):
    from paper_2302_11665_amd.workload.problems import Problem
    rng = np.random.default_rng(1)
    pb = _random_problem(rng, 4, 2, 10, 5, 2)
    pb.t = pb.t[:0]
    pb.model = pb.model[:0]
    pb.finish_jobs = np.zeros(0, np.int32)
    res = gpu.simulate_problem(pb)
    assert np.all(res["served"] == 0) and np.all(res["attain"] == 0.0)
    assert np.all(res["digest"] == 0)


def test_deterministic_repeat(gpu_api):
    gpu = gpu_api
    from paper_2302_11665_amd.workload import problems
    pb = problems.c2_greedy_step(duration=120.0)
    dp = gpu.upload(pb)
    gpu.run(dp)
    a = gpu.results(dp)
    gpu.run(dp)
    b = gpu.results(dp)
    assert np.array_equal(a["served"], b["served"]) and np.array_equal(a["digest"], b["digest"])
    for j in a["finish"]:
        assert a["finish"][j].tobytes() == b["finish"][j].tobytes()


def test_validate_catches_bad_data(gpu_api):
    import torch
    from paper_2302_11665_amd import sim
    from paper_2302_11665_amd.workload import problems
    pb = problems.c1_tiny(duration=5.0)
    d = sim.to_device
    args = [d(pb.t), d(pb.model), d(pb.d_single), pb.cfg_stages, d(pb.stage_lat), d(pb.group_cfg),
            d(pb.host_mask), d(pb.slo_scale)]
    sim.as_validate(*args)
    bad_t = pb.t.copy()
    bad_t[3], bad_t[4] = bad_t[4], bad_t[3] + 1.0
    cases = {
        0: d(bad_t),
        1: d(np.where(np.arange(len(pb.model)) == 2, 7, pb.model).astype(np.int32)),
        6: d(np.array([-1.0])),
    }
    for idx, arr in cases.items():
        a2 = list(args)
        a2[idx if idx != 6 else 7] = arr
        with pytest.raises(sim.SimError) as ei:
            sim.as_validate(*a2)
        assert ei.value.code == sim.AS_E_INVALID_DATA
    hm = pb.host_mask.copy()
    hm[0, 0] = np.uint64(1 << 5)  # group 5 does not exist
    a2 = list(args)
    a2[6] = d(hm)
    with pytest.raises(sim.SimError):
        sim.as_validate(*a2)
    torch.cuda.synchronize()


def test_c4_full_size_sampled(gpu_api):
    """The benchmark workload at full size (8192 placements x 3.6 M requests) in
    the benchmark's launch configuration; the oracle recomputes 4 jobs of every
    block of 64 consecutive jobs (a wavefront's jobs on the speculative
    kernels, 512 in all, each over the whole trace) and all 16 per-request
    output rows."""
    from paper_2302_11665_amd.workload import problems
    pb = problems.c4_heavy()
    say("c4 full", pb.n_jobs, len(pb.t))
    res = gpu_api.simulate_problem(pb)
    rng = np.random.default_rng(44)
    jobs = set()
    for b in range(0, pb.n_jobs, 64):
        jobs |= set((b + rng.choice(min(64, pb.n_jobs - b), 4, replace=False)).tolist())
    fins = [int(x) for x in pb.finish_jobs]
    jobs = sorted(jobs | set(fins))
    assert len(jobs) >= 512
    say("c4 full: oracle on", len(jobs), "jobs")
    compare(res, oracle_problem(pb, jobs=jobs, finish_jobs=fins), len(pb.t), "c4 full sampled")


def test_c4_full_size_spec_sampled(gpu_api, monkeypatch):
    """The benchmark workload at full size on the segment-speculative kernels
    (default segment count): oracle samples as above, and every job's served
    count and digest equal to those of the shared-trace kernel (itself checked
    against the oracle in the test above)."""
    from paper_2302_11665_amd.workload import problems
    pb = problems.c4_heavy()
    monkeypatch.setenv("ALPASERVE_PATH", "spec")
    say("c4 full spec", pb.n_jobs, len(pb.t))
    res = gpu_api.simulate_problem(pb)
    rng = np.random.default_rng(45)
    jobs = sorted(set(rng.choice(pb.n_jobs, 6, replace=False).tolist()) | {int(pb.finish_jobs[0]),
                                                                           int(pb.finish_jobs[-1])})
    fins = [int(pb.finish_jobs[0]), int(pb.finish_jobs[-1])]
    compare(res, oracle_problem(pb, jobs=jobs, finish_jobs=fins), len(pb.t), "c4 full spec sampled")
    monkeypatch.setenv("ALPASERVE_PATH", "shared")
    ref = gpu_api.simulate_problem(pb)
    assert np.array_equal(res["served"], ref["served"])
    assert np.array_equal(np.asarray(res["digest"]), np.asarray(ref["digest"]))
    for f in range(len(pb.finish_jobs)):
        j = int(pb.finish_jobs[f])
        assert res["finish"][j].tobytes() == ref["finish"][j].tobytes(), j


def test_maximum_sizes(gpu):
    """64 models, 64 groups, 8-stage pipelines, 8 configurations (the largest
    stage-latency table every kernel shape holds), every job of several scales,
    a ragged trace."""
    rng = np.random.default_rng(64)
    from paper_2302_11665_amd.workload.problems import Problem
    M, G, S, C, n, P = 64, 64, 8, 8, 3001, 6
    cfg_stages = rng.integers(1, S + 1, C).astype(np.int32)
    cfg_stages[0] = S
    L = rng.uniform(0.01, 0.4, (M, C, S))
    gaps = rng.exponential(0.002, n)
    gaps[rng.random(n) < 0.2] = 0.0
    t = np.cumsum(gaps)
    model = rng.integers(0, M, n).astype(np.int32)
    gcfg = rng.integers(0, C, (P, G)).astype(np.int32)
    masks = rng.integers(0, 1 << 62, (P, M)).astype(np.uint64) | rng.integers(0, 4, (P, M)).astype(np.uint64) << np.uint64(62)
    d = L[:, 0, :].sum(axis=1) * rng.uniform(0.5, 1.5, M)
    pb = Problem("maximum", t, model, d, np.zeros(M, np.int64), cfg_stages, np.ones(C, np.int32), L, gcfg, masks,
                 np.array([0.0, 2.0, np.inf]), np.array([0, 7, 17], np.int32))
    say("maximum sizes", M, G, S, C, n, P)
    res = gpu.simulate_problem(pb)
    compare(res, oracle_problem(pb, finish_jobs=pb.finish_jobs), n, "maximum sizes")


def test_table_beyond_lds_is_refused(gpu_api):
    """64 models x 32 configurations x 8 stages do not fit in any kernel's LDS:
    the call returns AS_E_LIMITS and launches nothing."""
    import torch
    from paper_2302_11665_amd import sim
    M, C, S, G = 64, 32, 8, 4
    d = sim.to_device
    L = np.full((M, C, S), 0.1)
    out = torch.zeros(1, dtype=torch.int64, device="cuda")
    with pytest.raises(sim.SimError) as ei:
        sim.as_simulate_placements(d(np.zeros(10)), d(np.zeros(10, np.int32)), d(np.ones(M)),
                                   np.full(C, S, np.int32), d(L), d(np.zeros((1, G), np.int32)),
                                   d(np.ones((1, M), np.uint64)), d(np.array([1.0])), out)
    assert ei.value.code == sim.AS_E_LIMITS
    assert int(out.cpu()[0]) == 0
