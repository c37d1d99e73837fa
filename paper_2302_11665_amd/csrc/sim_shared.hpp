// Group-per-lane request step on per-wavefront model records, the step of the
// speculative rounds (sim_spec.hip), and the job sets of the group-per-lane
// kernels (sim_lean.hpp).  A job owns W lanes of a wavefront, lane r of the
// job holds group r's stage free times F[0..SMAX-1] in registers.
//
// Per-wavefront model records (LDS, one per model m, built when the kernel
// starts): the wavefront's hosting lane mask for m (bit l = lane l's group
// hosts m), d_single[m], a count that is 0 when no job of the wavefront has two groups
// hosting m and otherwise the number of jobs of the wavefront hosting m, and,
// when every group of the wavefront has the same configuration, that
// configuration's stage latencies of m.  A request therefore costs one
// address computation and reads at immediate offsets of one record.
//
// Dispatch (Sec. 4.3): the target of a job is the hosting lane with the
// smallest stage-0 free time, the lowest such lane on ties.  When the record's
// count is 0, the hosting lanes are the targets.  Otherwise the minimum is
// found on the free times' IEEE bit patterns: free times are >= 0, so with the
// sign bit cleared (-0 and +0 become equal) the unsigned order of the 64-bit
// patterns is the numeric order.  The high words are reduced first with
// one-instruction DPP min steps (v_min_u32 with a DPP operand inside 16-lane
// rows, permlane swaps across rows).  If the hosting lanes holding the
// minimal high word are exactly one per hosting job (their population count
// equals the record's count), they are the targets.  Otherwise the low words
// of the tied lanes are reduced as well, and the lowest lane of each job
// holding the minimum -- the lowest set bit of every W-bit field of the
// equality mask, computed on the scalar unit -- is the target.  Projection,
// admission and counting are sim_kernel.hpp's, so the results are
// bit-identical.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alpaserve_sim.h"
#include "sim_kernel.hpp"

namespace as_dev {

// Lowest set bit of every aligned W-bit field of a 64-bit lane mask (uniform,
// scalar ALU).  Per field, -b is (~b + 1) computed without carries crossing
// field boundaries: fieldwise x + y = ((x & ~H) + (y & ~H)) ^ ((x ^ y) & H),
// H = the top bit of every field, y = L = the bottom bit of every field.
template <int W>
__device__ __forceinline__ uint64_t lowest_per_field(uint64_t b) {
  if constexpr (W == 1) {
    return b;
  } else if constexpr (W == 64) {
    return b & (~b + 1);
  } else {
    uint64_t L = 0, H = 0;
#pragma unroll
    for (int f = 0; f < 64; f += W) {
      L |= 1ull << f;
      H |= 1ull << (f + W - 1);
    }
    const uint64_t x = ~b;
    const uint64_t neg = ((x & ~H) + L) ^ ((x ^ L) & H);
    return b & neg;
  }
}

__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Unsigned minimum over each aligned W-lane segment, in every lane of it.
// Inside a 16-lane row each step is one v_min_u32 with a DPP operand; for
// W = 32 the 16-lane step swaps rows with v_permlane16_swap (its two outputs
// are the two halves of the butterfly); for W = 64 row broadcasts gather the
// minimum in lane 63, whose value is returned to every lane.
template <int W>
__device__ __forceinline__ uint32_t seg_min_u32(uint32_t x) {
  if constexpr (W >= 2) x = umin32(x, dpp_u32<kXor1>(x));
  if constexpr (W >= 4) x = umin32(x, dpp_u32<kXor2>(x));
  if constexpr (W >= 8) x = umin32(x, dpp_u32<kHalfMirror>(x));
  if constexpr (W >= 16) x = umin32(x, dpp_u32<kMirror>(x));
  if constexpr (W == 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = umin32(r[0], r[1]);
  }
  if constexpr (W == 64) {
    // fold the four row minima into lane 63 (row_bcast:15 into rows 1 and 3,
    // row_bcast:31 into rows 2 and 3; masked-off rows keep their value) and
    // read it back as a wave-uniform scalar
    x = umin32(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x142, 0xa, 0xf, false));
    x = umin32(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, 0x143, 0xc, 0xf, false));
    x = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
  }
  return x;
}

// Layout of one model record: hosting mask (u64) at 0, count (u32) at 8,
// stage latencies (SMAX doubles) at 16, SLO or d_single (double) after them;
// the record size is a power of two.
constexpr int kRecMask = 0, kRecCount = 8, kRecLat = 16;
__host__ __device__ constexpr int rec_slo(int SMAX) { return kRecLat + 8 * SMAX; }
__host__ __device__ constexpr int rec_shift(int SMAX) { return SMAX == 1 ? 5 : (SMAX <= 4 ? 6 : 7); }

// Per-lane state: group (lane mod W) of one job.
template <int SMAX>
struct SharedLane {
  double F[SMAX];
  uint64_t fin_sum, served;
};

struct SharedConst {
  const unsigned char* rec;  // this wavefront's model records (LDS)
  const double* lrow;        // stage-latency row of this lane's configuration for model 0 (LDS)
  int lshift;                // log2 of the per-model row stride (bytes) of that table
  double sigma;              // this job's scale
};

// Projection through this lane's stage chain (Sec. 3.4): fs[s] is the
// request's finish time at stage s; returns the last.
template <int SMAX>
__device__ __forceinline__ double chain(const SharedLane<SMAX>& st, double ti,
                                        const double (&L)[SMAX], double (&fs)[SMAX]) {
  double f = ti;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    fs[s] = vmax(f, st.F[s]) + L[s];
    f = fs[s];
  }
  return f;
}

// One request.  hm: the wavefront's hosting lanes; cnt: the record's count; L:
// this lane's stage latencies of the model; d: d_single of the model.
template <int W, int SMAX>
__device__ __forceinline__ void fast_step(SharedLane<SMAX>& st, const SharedConst& c, double ti,
                                          uint64_t hm, uint32_t cnt, const double (&L)[SMAX],
                                          double d, uint32_t& sr) {
  uint64_t cm = hm;  // the dispatch target of every job: one lane per job or none
  if (cnt != 0) {
    const bool hosted = __builtin_amdgcn_inverse_ballot_w64(hm);
    const uint64_t kb = (uint64_t)__double_as_longlong(st.F[0]);
    const uint32_t khi = hosted ? ((uint32_t)(kb >> 32) & 0x7fffffffu) : 0xffffffffu;
    const uint32_t mhi = seg_min_u32<W>(khi);
    const uint64_t eqhi = __builtin_amdgcn_ballot_w64(khi == mhi) & hm;
    cm = eqhi;
    if ((uint32_t)__builtin_popcountll(eqhi) != cnt) {
      // some job has two hosting lanes with the same high word: compare the
      // low words of the tied lanes
      const bool tied = __builtin_amdgcn_inverse_ballot_w64(eqhi);
      const uint32_t klo = tied ? (uint32_t)kb : 0xffffffffu;
      const uint32_t mlo = seg_min_u32<W>(klo);
      cm = lowest_per_field<W>(__builtin_amdgcn_ballot_w64(klo == mlo) & eqhi);
    }
  }
  double fs[SMAX];
  const double f = chain<SMAX>(st, ti, L, fs);
  // admission (Sec. 4.3, Sec. 3.2) and commit on the target lane
  const double deadline = ti + c.sigma * d;
  const uint64_t am = cm & __builtin_amdgcn_ballot_w64(!(f > deadline));
  const bool acc = __builtin_amdgcn_inverse_ballot_w64(am);
#pragma unroll
  for (int s = 0; s < SMAX; ++s) st.F[s] = acc ? fs[s] : st.F[s];
  st.fin_sum += acc ? (uint64_t)__double_as_longlong(f) : 0ull;
  sr = (sr << 1) | (acc ? 1u : 0u);
}

// B requests of an LDS chunk (cT: arrivals at stride 2, cO: record offsets):
// read all of their inputs first (LDS reads in flight together), then run them
// in order.  UNI: every group of the wavefront has the same configuration,
// whose stage latencies the model records hold; otherwise each lane reads its
// configuration's row.
template <int W, int SMAX, int B, bool UNI>
__device__ __forceinline__ void fast_batch(SharedLane<SMAX>& st, const SharedConst& c,
                                           const double* __restrict__ cT,
                                           const uint32_t* __restrict__ cO, uint32_t& sr) {
  double t[B], dv[B], L[B][SMAX];
  uint64_t hmv[B];
  uint32_t cnv[B], off[B];
#pragma unroll
  for (int k = 0; k < B; ++k) {
    t[k] = cT[2 * k];
    off[k] = cO[k];
  }
#pragma unroll
  for (int k = 0; k < B; ++k) {
    // records are 32-byte aligned: 16-byte loads
    const unsigned char* r = c.rec + off[k];
    const uint4 head = *(const uint4*)(r + kRecMask);  // hosting mask, count
    hmv[k] = ((uint64_t)head.y << 32) | head.x;
    cnv[k] = head.z;
    dv[k] = *(const double*)(r + rec_slo(SMAX));
    if (UNI) {
#pragma unroll
      for (int s = 0; s + 1 < SMAX; s += 2) {
        const double2 l2 = *(const double2*)(r + kRecLat + 8 * s);
        L[k][s] = l2.x;
        L[k][s + 1] = l2.y;
      }
      if (SMAX & 1) L[k][SMAX - 1] = *(const double*)(r + kRecLat + 8 * (SMAX - 1));
    } else {
      const double* lr =
          (const double*)((const char*)c.lrow + ((off[k] >> rec_shift(SMAX)) << c.lshift));
#pragma unroll
      for (int s = 0; s < SMAX; ++s) L[k][s] = lr[s];
    }
  }
#pragma unroll
  for (int k = 0; k < B; ++k) {
    // record words are the same in every lane: move them to scalar registers
    const uint64_t hm = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(hmv[k] >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)hmv[k]);
    const uint32_t cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)cnv[k]);
    fast_step<W, SMAX>(st, c, t[k], hm, cnt, L[k], dv[k], sr);
  }
}

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
