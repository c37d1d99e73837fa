// Job sets of the group-per-lane kernels (sim_lean.hpp) and the bounds of
// segmented jobs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alpaserve_sim.h"
#include "sim_kernel.hpp"

namespace as_dev {

// log2 of the bytes that a model record of SMAX stages has counted as in the
// limit on stage-latency tables (lean_takes in sim_api.hip).
__host__ __device__ constexpr int rec_shift(int SMAX) { return SMAX == 1 ? 5 : (SMAX <= 4 ? 6 : 7); }

// The jobs one launch (or one shape segment of a multi-shape launch) runs:
// their count, group-row stride, placement rows and outputs.
struct JobSet {
  int64_t J;
  int32_t G;
  const int32_t* group_cfg;
  const uint64_t* host_mask;
  int64_t* out_served;
  double* out_attain;
  uint64_t* out_digest;
  int64_t* out_model_served;
  double* out_group_busy;
  int32_t jw;  // jobs per wavefront, at most 64 / W
};

__device__ __forceinline__ JobSet job_set(const KArgs& a, int jw) {
  return JobSet{a.J, a.G, a.group_cfg, a.host_mask, a.out_served, a.out_attain, a.out_digest,
                a.out_model_served, a.out_group_busy, jw};
}

// Multi-shape launches: consecutive block ranges run job sets of different
// shapes (lanes per job 2^wl, padded stages 2^sl), so that the jobs of
// several shapes share one dispatch instead of queueing behind each other.
constexpr int kMaxShapeSegs = 16;
struct ShapeSeg {
  int32_t wl, sl;
  int64_t block0;  // first block of the segment
  JobSet v;
};
struct MultiSegs {
  int32_t n;
  ShapeSeg s[kMaxShapeSegs];
};

// Length and start of job j's segment: a record naming a missing placement or
// segment makes an empty job; bounds are clamped to [0, seg_off[n_segments]].
__device__ __forceinline__ void seg_job(const KArgs& a, int64_t j, int& p, double& sigma,
                                        int64_t& begin, int64_t& len) {
  const as_job_t jb = a.jobs[j];
  p = jb.placement;
  sigma = jb.slo_scale;
  begin = 0;
  len = 0;
  if (p < 0 || p >= a.P || jb.segment < 0 || jb.segment >= a.n_segments) {
    p = 0;
    return;
  }
  const int64_t total = a.seg_off[a.n_segments];
  int64_t b = a.seg_off[jb.segment], e = a.seg_off[jb.segment + 1];
  b = b < 0 ? 0 : (b > total ? total : b);
  e = e < b ? b : (e > total ? total : e);
  begin = b;
  len = e - b;
}

}  // namespace as_dev
