// Arguments and workspace of the segment-speculative kernels (sim_spec.hip:
// pass 0, output rows, final step; below: the fix-up of jobs whose segments
// started from a wrong estimate).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alpaserve_sim.h"
#include "sim_kernel.hpp"
#include "sim_lean.hpp"

namespace as_dev {

constexpr int kSpecMaxSeg = 1024;
constexpr int kSpecRounds = 8;  // parallel rounds before the job-by-job fix-up
constexpr uint64_t kSpecHashMul = 0x9E3779B97F4A7C15ULL;

struct SpecArgs {
  const double* t;
  const int32_t* model;
  int64_t n;
  const double* d_single;
  const double* stage_lat;
  const int32_t* group_cfg;
  const uint64_t* host_mask;
  const double* slo_scale;
  int64_t* out_served;
  double* out_attain;
  uint64_t* out_digest;
  double* out_finish;
  // workspace
  uint64_t* bitmap;     // [nw][J] accept bits, 64 requests per word
  double* st_start;     // [nseg][G*SMAX][J] start state behind each segment's results
  double* st_end;       // [nseg][G*SMAX][J] state at its end
  int64_t* seg_served;  // [nseg][J]
  uint64_t* seg_fsum;   // [nseg][J]
  double* ckpt;         // [nseg][ckps][G*SMAX][J] states every ck requests into a segment
  int64_t* ck_served;   // [nseg][ckps][J] served count of the segment before each checkpoint
  uint64_t* ck_fsum;    // [nseg][ckps][J] finish-time sum likewise
  double* xch[2];       // [nseg][G*SMAX][J] end states handed to the next round
  int2* list[2];        // [J*nseg] {job, segment} whose start state is not its predecessor's end state
  int32_t* claimed;     // [J] the last fix-up has taken the job
  int32_t* cfg_info;    // [3]: 1 when every used group has one configuration; that configuration;
                        // 1 once the fix-ups gave up (the results are then left to other kernels)
  int32_t* count;       // [kSpecRounds + 2] entries of each round's list, list q & 1 for round q + 1
  int32_t* taken;       // [kSpecRounds + 2] entries that wavefronts have taken
  unsigned long long* work;  // requests that fix-ups have simulated
  int64_t ck;           // checkpoint interval (a multiple of 64)
  int32_t ckps;         // checkpoints per segment (upper bound)
  int64_t cap;          // requests one re-run may simulate before the fix-ups give up
  int64_t budget;       // and all of them together
  int64_t budget1;      // and those of round 1, by what its entries promise so far
  int64_t pairs;        // entries of the first list beyond which they give up at once
  int64_t few, some;    // and shares of it listed again beyond which they do: none up to few
  double again_some, again;  // entries, again_some up to some, else again
  int64_t nw;
  int64_t warmup;  // requests simulated before a segment to estimate its start state
  int32_t M, C, smax_in, G, K, J, n_finish, nseg, njb;
  int32_t cfg_stages[AS_MAX_CONFIGS];
  int32_t finish_jobs[AS_MAX_FINISH];
};

// First request of segment k: a multiple of 64 (n for k = nseg).
__device__ __forceinline__ int64_t seg_bound(int64_t n, int nseg, int k) {
  return k >= nseg ? n : ((n * k / nseg) & ~(int64_t)63);
}

__device__ __forceinline__ uint64_t bits_of(double x) { return (uint64_t)__double_as_longlong(x); }

// Saved states inside a segment of requests [b, e).
__device__ __forceinline__ int spec_ckpts(int64_t b, int64_t e, int64_t ck) { return (int)((e - b - 1) / ck); }

// Fix-ups, after pass 0 has simulated every segment from an estimated start
// state.  Where a segment's start state is not its predecessor's end state, the
// segment is simulated again from that end state until the state equals, bit
// for bit, the one its results had at a saved point: from there on both runs
// take the same decisions, so the old results stand and only the prefix is
// replaced.  A run that never meets them replaces the segment, and the next
// segment is looked at again.
//
// Rounds (round_entry) take all listed segments of all jobs at once, each from
// the end state its predecessor had after the round before, so that a job
// whose runs meet slowly settles all its segments in about (requests until
// they meet) / (segment length) rounds: after kSpecRounds of them few jobs are
// left, whose segments are then fixed one after the other (spec_fix).
// Afterwards every saved state and total is exact.
//
// One job per wavefront on the group-per-lane step (sim_lean.hpp), whose
// request is the shortest chain: a round's time is its longest re-run.
// Measured: 1000 placements, 900,000 requests, 13 seeds: 12 to 79 ms a call (105
// where the fix-ups gave up; 64 segments of 14,062 requests), 48 to 205 with the
// six segments to which rounds of one segment after the other's end, each on all
// jobs' lanes, had held it; 8192 placements, 3.6 M requests, on a seed where some
// jobs' runs never meet: 735 ms, since one of them sent the whole call to the
// other kernels, -> 164 to 182.

// Counts requests that a re-run has simulated; whether that is more than the
// fix-ups may.  first: entries of the first list in round 1, else 0 (that
// round's entries promise what those taken so far have run, the ones that still
// run in part, so the promise is never too high).
__device__ __forceinline__ bool fix_spent(const SpecArgs& a, int64_t requests, int first) {
  unsigned long long all = 0;
  if ((threadIdx.x & 63) == 0) all = atomicAdd(a.work, (unsigned long long)requests);
  all = lean_uniform(all);
  if (all > (unsigned long long)a.budget) return true;
  if (first == 0) return false;
  const int taken = __hip_atomic_load(a.taken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (double)all * first > (double)a.budget1 * (taken < first ? taken : first);
}

// The re-run of one segment.  Returns 0: gave up; 1: met the old results; 2: ran
// to the end, which st.F holds.
template <int W, int SMAX, bool UNI>
__device__ __forceinline__ int fix_segment(const SpecArgs& a, const LeanWave<W, SMAX>& w, LeanLane<SMAX>& st,
                                           int job, int k, const double (&start)[SMAX], int first) {
  const int lane = threadIdx.x & 63;
  const bool mine_g = lane < a.G;  // this lane holds a group
  const int GS = a.G * SMAX;
  const int64_t J = a.J;
  const size_t own = ((size_t)k * GS + (size_t)lane * SMAX) * J + job;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    st.F[s] = start[s];
    if (mine_g) a.st_start[own + (size_t)s * J] = start[s];
  }
  st.fin = 0;
  int64_t served = 0;
  const int64_t b = seg_bound(a.n, a.nseg, k), e = seg_bound(a.n, a.nseg, k + 1);
  if (b >= e) return 2;
  const size_t ck0 = (size_t)k * a.ckps;
  const int nck = spec_ckpts(b, e, a.ck);
  const int64_t top = e - 1;
  double tn = a.t[b + lane < e ? b + lane : top];
  int mn = a.model[b + lane < e ? b + lane : top];
  for (int64_t cb = b; cb < e; cb += 64) {
    if (cb > b && (cb - b) % a.ck == 0) {
      const int jl = (int)((cb - b) / a.ck) - 1;
      const size_t j = ck0 + (size_t)jl, at = (j * GS + (size_t)lane * SMAX) * J + job, cj = j * J + job;
      bool same = true;
      if (mine_g)
#pragma unroll
        for (int s = 0; s < SMAX; ++s) same &= bits_of(a.ckpt[at + (size_t)s * J]) == bits_of(st.F[s]);
      const uint64_t fsum = seg_sum_u64<64>(st.fin);
      if (__builtin_amdgcn_ballot_w64(!same) == 0) {
        // the old results stand from here on; later running totals shift by
        // the prefix's change
        if (lane == 0) {
          const int64_t ds = served - a.ck_served[cj];
          const uint64_t df = fsum - a.ck_fsum[cj];
          a.seg_served[(size_t)k * J + job] += ds;
          a.seg_fsum[(size_t)k * J + job] += df;
          for (int j2 = jl; j2 < nck; ++j2) {
            a.ck_served[(ck0 + j2) * J + job] += ds;
            a.ck_fsum[(ck0 + j2) * J + job] += df;
          }
        }
        return 1;
      }
      if (mine_g)
#pragma unroll
        for (int s = 0; s < SMAX; ++s) a.ckpt[at + (size_t)s * J] = st.F[s];
      if (lane == 0) {
        a.ck_served[cj] = served;
        a.ck_fsum[cj] = fsum;
      }
      if (fix_spent(a, a.ck, first)) return 0;
    }
    if (cb - b >= a.cap) return 0;
    const double tv = tn;
    const int mv = mn;
    const int64_t ahead = cb + 64 + lane;
    tn = a.t[ahead < e ? ahead : top];
    mn = a.model[ahead < e ? ahead : top];
    int rank, nh;
    const bool mine = lean_mine<W, SMAX>(w, cb + lane < e, mv, rank, nh);
    uint64_t word = lean_uniform(lean_chunk<W, SMAX, UNI, false, 0>(st, w, tv, mv, mine, rank, nh));
    served += __builtin_popcountll(word);
    word = __builtin_amdgcn_ballot_w64(mine && ((word >> rank) & 1u));
    if (lane == 0) a.bitmap[(cb >> 6) * J + job] = word;
  }
  // what lies behind the last saved state, in a short segment all of it
  if (fix_spent(a, e - b - (int64_t)nck * a.ck, first)) return 0;
  const uint64_t fsum = seg_sum_u64<64>(st.fin);
  if (lane == 0) {
    a.seg_served[(size_t)k * J + job] = served;
    a.seg_fsum[(size_t)k * J + job] = fsum;
  }
  return 2;
}

// Whether the start states differ from those recorded for the segment.
template <int SMAX>
__device__ __forceinline__ bool fix_stale(const SpecArgs& a, const double* from, int job, int k,
                                          double (&start)[SMAX]) {
  const int lane = threadIdx.x & 63;
  const int GS = a.G * SMAX;
  const int64_t J = a.J;
  const size_t own = ((size_t)k * GS + (size_t)lane * SMAX) * J + job, prv = own - (size_t)GS * J;
  bool differ = false;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) {
    start[s] = lane < a.G ? from[prv + (size_t)s * J] : 0.0;
    if (lane < a.G) differ |= bits_of(a.st_start[own + (size_t)s * J]) != bits_of(start[s]);
  }
  return __builtin_amdgcn_ballot_w64(differ) != 0;
}

// One listed segment of round q; returns false when it gives up.
template <int W, int SMAX, bool UNI>
__device__ __forceinline__ bool round_entry(const SpecArgs& a, const LeanWave<W, SMAX>& w, int job, int k, int q) {
  const int lane = threadIdx.x & 63;
  double start[SMAX];
  if (!fix_stale<SMAX>(a, a.xch[(q - 1) & 1], job, k, start)) return true;
  LeanLane<SMAX> st;
  st.busy = 0.0;
  const int r = fix_segment<W, SMAX, UNI>(a, w, st, job, k, start, q == 1 ? a.count[0] : 0);
  if (r != 2) return r != 0;
  // a new end state, unless it is the old one: the next segment is listed
  const int GS = a.G * SMAX;
  const int64_t J = a.J;
  const size_t own = ((size_t)k * GS + (size_t)lane * SMAX) * J + job;
  bool differ = false;
  if (lane < a.G)
#pragma unroll
    for (int s = 0; s < SMAX; ++s) differ |= bits_of(a.st_end[own + (size_t)s * J]) != bits_of(st.F[s]);
  if (__builtin_amdgcn_ballot_w64(differ) == 0 || k + 1 >= a.nseg) return true;
  if (lane < a.G)
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      a.st_end[own + (size_t)s * J] = st.F[s];
      a.xch[q & 1][own + (size_t)s * J] = st.F[s];
    }
  if (lane == 0) a.list[q & 1][atomicAdd(a.count + q, 1)] = make_int2(job, k + 1);
  return true;
}

// All segments of a job, one after the other.
template <int W, int SMAX, bool UNI>
__device__ __forceinline__ bool fix_job(const SpecArgs& a, const LeanWave<W, SMAX>& w, int job) {
  const int lane = threadIdx.x & 63;
  LeanLane<SMAX> st;
  st.busy = 0.0;
  for (int k = 1; k < a.nseg; ++k) {
    double start[SMAX];
    if (!fix_stale<SMAX>(a, a.st_end, job, k, start)) continue;
    const int r = fix_segment<W, SMAX, UNI>(a, w, st, job, k, start, 0);
    if (r == 0) return false;
    if (r == 2 && lane < a.G) {
      const size_t own = ((size_t)k * a.G * SMAX + (size_t)lane * SMAX) * a.J + job;
#pragma unroll
      for (int s = 0; s < SMAX; ++s) a.st_end[own + (size_t)s * a.J] = st.F[s];
    }
  }
  return true;
}

// Round q = 1 .. kSpecRounds of list (q - 1) & 1; q = kSpecRounds + 1: the jobs
// of the list that is left, each whole.  Wavefronts take entries in turn.
template <int W, int SMAX>
__global__ __launch_bounds__(64) void spec_fix(const SpecArgs a, int q) {
  const int n = __builtin_amdgcn_readfirstlane(a.count[q - 1]);
  if (n == 0 || __builtin_amdgcn_readfirstlane(a.cfg_info[2]) != 0) return;
  const int lane = threadIdx.x & 63;
  bool over = q == 1 && n > a.pairs;
  if (q == 2) {
    const int first = a.count[0];
    over = first > a.few && n > (first > a.some ? a.again : a.again_some) * first;
  }
  if (over) {
    if (blockIdx.x == 0 && lane == 0) a.cfg_info[2] = 1;
    return;
  }
  extern __shared__ __align__(16) unsigned char smem[];
  double* sL = reinterpret_cast<double*>(smem);
  size_t tab = 0;
  const int lshift = lean_table<SMAX>(a, sL, tab);
  for (;;) {
    int x = 0;
    if (lane == 0) x = atomicAdd(a.taken + q - 1, 1);
    x = __builtin_amdgcn_readfirstlane(x);
    if (x >= n) return;
    const int2 en = a.list[(q - 1) & 1][x];
    const int job = __builtin_amdgcn_readfirstlane(en.x), k = __builtin_amdgcn_readfirstlane(en.y);
    if (q > kSpecRounds) {
      int c = 0;
      if (lane == 0) c = atomicExch(a.claimed + job, 1);
      if (__builtin_amdgcn_readfirstlane(c) != 0) continue;
    }
    const int p = job / a.K;
    int cfg = lane < a.G ? a.group_cfg[(int64_t)p * a.G + lane] : -1;
    if (cfg >= a.C || cfg < 0) cfg = -1;
    const uint64_t hm = (lane < a.M ? a.host_mask[(int64_t)p * a.M + lane] : 0) & __builtin_amdgcn_ballot_w64(cfg >= 0);
    const LeanWave<W, SMAX> w = lean_wave<W, SMAX>(a, a.slo_scale[job % a.K], cfg, hm, sL, lshift, smem + tab);
    bool done;
    if (lean_uni(cfg))
      done = q > kSpecRounds ? fix_job<W, SMAX, true>(a, w, job) : round_entry<W, SMAX, true>(a, w, job, k, q);
    else
      done = q > kSpecRounds ? fix_job<W, SMAX, false>(a, w, job) : round_entry<W, SMAX, false>(a, w, job, k, q);
    if (!done) {
      if (lane == 0) a.cfg_info[2] = 1;
      return;
    }
  }
}

}  // namespace as_dev
