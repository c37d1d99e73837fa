// Per-job statistics of the serving simulation for the fast placement
// heuristic of Sec. 4.2 (simulate the current selection once, then place the
// model with the most unserved requests on the available group with the
// lowest utilization): besides the served count and digest, every job reports
// the served requests of each model and the busy time of each group.
//
// Both come from the group-per-lane kernels (sim_lean.hpp): on accept the
// target lane adds the model's slowest stage latency for its configuration
// (the stage that bounds a pipeline's throughput, Sec. 3.4) to its busy time,
// in trace order, and bumps the model's served counter (LDS, one writer per
// request).  A kernel of their own for several SLO scales, with its branches
// and a staged chunk that four jobs shared, took 32.5 ms for 6 placements x 3
// scales of 64 groups on 76800 requests; these take 8.4.
#include <hip/hip_runtime.h>

#include <cstring>

#include "alpaserve_sim.h"
#include "sim_internal.hpp"
#include "sim_kernel.hpp"

using namespace as_host;

extern "C" int as_simulate_stats(const as_trace_t* trace, const as_models_t* models,
                                 const as_placements_t* placements, const double* slo_scale,
                                 int32_t n_scales, int64_t* out_served, uint64_t* out_digest,
                                 int64_t* out_model_served, double* out_group_busy, void* stream) {
  KArgs ka;
  std::memset(&ka, 0, sizeof ka);
  if (!trace) return fail(AS_E_INVALID_ARG, "trace must not be NULL");
  if (trace->n < 0) return fail(AS_E_INVALID_ARG, "trace n=%lld < 0", (long long)trace->n);
  if (trace->n > 0 && (!trace->t || !trace->model))
    return fail(AS_E_INVALID_ARG, "trace arrays must not be NULL");
  int W = 1, smax = 1;
  int rc = check_common(models, placements, ka, W, smax);
  if (rc != AS_OK) return rc;
  if (n_scales < 0) return fail(AS_E_INVALID_ARG, "n_scales=%d < 0", n_scales);
  const int64_t J = (int64_t)placements->n_placements * n_scales;
  if (J > 0x7FFFFFFFLL) return fail(AS_E_LIMITS, "placements x scales = %lld jobs > 2^31-1", (long long)J);
  if (J > 0 && (!slo_scale || !out_served))
    return fail(AS_E_INVALID_ARG, "slo_scale and out_served must not be NULL");
  if (J == 0) return ok();
  hipStream_t s = (hipStream_t)stream;
  // the group-per-lane kernel with its statistics outputs
  ka.t = trace->t;
  ka.model = trace->model;
  ka.n = trace->n;
  ka.slo_scale = slo_scale;
  ka.K = n_scales;
  ka.J = (int32_t)J;
  ka.P = placements->n_placements;
  ka.out_served = out_served;
  ka.out_digest = out_digest;
  ka.out_model_served = out_model_served;
  ka.out_group_busy = out_group_busy;
  ka.n_finish = 0;
  return run_shared_stats(ka, smax, s);
}
