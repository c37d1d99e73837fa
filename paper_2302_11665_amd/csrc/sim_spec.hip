// Segment-speculative simulation of a shared trace: one lane per job, the
// trace cut into segments that run at the same time.
//
// The definition (Sec. 3.4, Sec. 4.3) is a recurrence over the requests of
// one job: request i is dispatched on the stage free times F left by request
// i-1.  A job's only parallelism is its groups, which the other kernels spread
// over lanes; most of those lanes then idle on every request (a model has one
// or two hosting groups, and only the chosen group runs the stage chain).
// Here one lane carries a whole job -- every lane does useful work on every
// request -- and the missing parallelism comes from the trace instead:
//
//   pass 0   every (job, segment) estimates its start state by simulating
//            the requests just before the segment from the empty state
//            (all F = 0), then runs the segment from that estimate,
//            recording its results and the state at its end;
//   fix-ups  a segment whose recorded start state is not its predecessor's end
//            state is simulated again from there until its state equals, bit
//            for bit, the state its current results had at the same request
//            (pass 0 saves the state every few thousand requests): from there
//            on both runs take identical decisions (the state is the only
//            thing a request depends on besides its own arrival), so the old
//            results stand and only the re-run prefix is replaced.  All such
//            segments at once in a few rounds, then job by job (sim_spec.hpp);
//   final    per job: served counts and finish-time sums add up over
//            segments; the digest's ordered hash runs over the accept bitmap.
//
// After round q segments 0..q hold exact results (segment 0 starts from the
// true empty state), so nseg - 1 rounds always suffice; a round with nothing
// listed returns at once.  Bursty arrivals make the speculation cheap: two runs
// of one job from different states become identical within a few thousand
// requests, so the warm-up estimate is usually exact and little is redone.
//
// State layout: F[g][s] of a lane lives in LDS as [g][s][lane] (conflict-free
// for any per-lane g), with a spare row that unserved requests write and a
// sentinel row that stands for a missing host; each lane's hosting masks live
// in registers (a uniform model index selects one); arrivals come in chunks
// of 64, one per lane, and a request is read from its lane with readlane.
//
// Exactness: the same IEEE operations in the same order as the definition
// (v_max_f64, single v_add_f64, no FMA), so finish times are bit-identical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "alpaserve_sim.h"
#include "sim_internal.hpp"
#include "sim_kernel.hpp"
#include "sim_launch.hpp"
#include "sim_spec.hpp"

namespace as_dev {
namespace {

// Jobs per wavefront: one lane per job.  (32 jobs per wavefront halves the
// state, so a SIMD holds two wavefronts; on the 8192-placement workload that
// took 305 ms against 276: the two did not overlap enough to pay for doubling
// the instructions per job.)
constexpr int kSpecJobsPerWave = 64;

// Accept bits of a chunk: each request's bit enters at the top and moves down
// one place per request, so that after the chunk's cnt requests chunk_word
// has request r's bit at r (bits pushed before them fall out of the word).
__device__ __forceinline__ uint64_t push_bit(uint64_t w, bool bit) {
  const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
  return ((uint64_t)__builtin_amdgcn_alignbit((uint32_t)bit, hi, 1) << 32) | __builtin_amdgcn_alignbit(hi, lo, 1);
}
__device__ __forceinline__ uint64_t chunk_word(uint64_t w, int cnt) { return cnt < 64 ? w >> (64 - cnt) : w; }

// Hosting masks of one lane's placement for every model, MB bits per model,
// held in vector registers (32-dword vector values: a wavefront-uniform index
// into one lowers to indexed register moves, not memory).
typedef uint32_t u32x32 __attribute__((ext_vector_type(32)));

template <int MB>
struct LaneMasks {
  static_assert(MB == 32 || MB == 64, "32- or 64-bit hosting masks");
  using MaskT = typename std::conditional<MB == 32, uint32_t, uint64_t>::type;
  // named vectors, never an array of them: a variable first index would put
  // the registers in memory.  MB 32 uses v0-v1, MB 64 v0-v3.
  u32x32 v0, v1, v2, v3;
  __device__ __forceinline__ void put(int w, uint32_t x) {  // dword w of the masks
    if (w < 32) {
      v0[w & 31] = x;
    } else if (w < 64) {
      v1[w & 31] = x;
    } else if constexpr (MB == 64) {
      if (w < 96) {
        v2[w & 31] = x;
      } else {
        v3[w & 31] = x;
      }
    }
  }
  // bits of groups >= G are dropped (they name no state); returns whether some
  // model has more than two hosting groups
  __device__ __forceinline__ bool load(const uint64_t* row, int M, int G, bool valid) {
    v0 = v1 = (u32x32)(0u);
    if constexpr (MB == 64) v2 = v3 = (u32x32)(0u);
    bool many = false;
    if (!valid) return many;
    const uint64_t keep = G >= 64 ? ~0ull : (1ull << G) - 1;
#pragma unroll
    for (int m = 0; m < 64; ++m) {
      const uint64_t x = m < M ? row[m] & keep : 0;
      many |= __popcll(x) > 2;
      if constexpr (MB == 32) {
        put(m, (uint32_t)x);
      } else {
        put(2 * m, (uint32_t)x);
        put(2 * m + 1, (uint32_t)(x >> 32));
      }
    }
    return many;
  }
  // m is wavefront-uniform; one indexed register move per vector read (the
  // empty asm keeps the compiler from selecting whole vectors first)
  __device__ __forceinline__ MaskT get(int m) const {
    if constexpr (MB == 32) {
      uint32_t lo = v0[m & 31], hi = v1[m & 31];
      asm volatile("" : "+v"(lo), "+v"(hi));
      return m < 32 ? lo : hi;
    } else {
      const int e = (2 * m) & 31;
      uint32_t lo, hi;
      if (m < 16) {
        lo = v0[e];
        hi = v0[e + 1];
      } else if (m < 32) {
        lo = v1[e];
        hi = v1[e + 1];
      } else if (m < 48) {
        lo = v2[e];
        hi = v2[e + 1];
      } else {
        lo = v3[e];
        hi = v3[e + 1];
      }
      asm volatile("" : "+v"(lo), "+v"(hi));
      return (uint64_t)lo | ((uint64_t)hi << 32);
    }
  }
};

template <typename T>
__device__ __forceinline__ int ctz_any(T x) {
  if constexpr (sizeof(T) == 4) {
    return (int)__builtin_ctz(x);
  } else {
    return (int)__builtin_ctzll(x);
  }
}

// Index of the lowest set bit, -1 when there is none (v_ffbl_b32 returns
// all ones for zero; the asm keeps the compiler from assuming x != 0).
template <typename T>
__device__ __forceinline__ int lowest_or_m1(T x) {
  if constexpr (sizeof(T) == 4) {
    int r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
  } else {
    return x ? (int)__builtin_ctzll(x) : -1;
  }
}

// Per-wavefront LDS: the model table, per-lane group configurations when
// groups differ, then the state.
//   uniform configuration c0:  T[m] = {L[m][c0][0..SMAX-1], d_single[m]}
//   otherwise:                 L[m][c][0..SMAX-1], D[m] = d_single[m], cfg[g][lane]
template <int SMAX, bool UCFG>
struct SpecLds {
  double* T;      // UCFG: [M][SMAX + 1]; else L: [M][C][SMAX]
  double* D;      // !UCFG: [M]
  uint16_t* cfg;  // !UCFG: [G][JPW] = c
  double* F;      // rows -1 .. G of [SMAX][JPW]; row -1 is a sentinel, row G is written, never read
};

// jpw: jobs per wavefront (lanes at or above it hold no job).  The state has
// a spare row past the G groups: a request that commits nothing writes
// there, so that the commit is a store without a branch.  Before the groups
// sits a sentinel row -1 whose stage-0 free time is +inf: a lane that has no
// (or no further) hosting group reads it as its host, and it never wins the
// dispatch.
__host__ __device__ constexpr size_t spec_lds_bytes(int M, int C, int G, int SMAX, bool ucfg, int jpw) {
  return (ucfg ? (size_t)M * (SMAX + 1) * 8 : (size_t)M * C * SMAX * 8 + (size_t)M * 8 + (size_t)G * jpw * 2) +
         (size_t)(G + 2) * SMAX * jpw * 8;
}

__device__ __forceinline__ double readlane_f64(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}

template <int SMAX, bool UCFG, int JPW>
__device__ __forceinline__ SpecLds<SMAX, UCFG> spec_tables(const SpecArgs& a, double* lds, int lane, int p,
                                                           bool valid, int c0) {
  SpecLds<SMAX, UCFG> s;
  const int M = a.M, C = a.C;
  s.T = lds;
  if constexpr (UCFG) {
    s.D = nullptr;
    s.cfg = nullptr;
    s.F = s.T + (size_t)M * (SMAX + 1) + SMAX * JPW;
    const int S0 = a.cfg_stages[c0];
    for (int e = lane; e < M * (SMAX + 1); e += 64) {
      const int k = e % (SMAX + 1);
      const int m = e / (SMAX + 1);
      s.T[e] = k == SMAX ? a.d_single[m]
                         : (k < S0 ? a.stage_lat[((int64_t)m * C + c0) * a.smax_in + k] : 0.0);
    }
  } else {
    s.D = s.T + (size_t)M * C * SMAX;
    s.cfg = reinterpret_cast<uint16_t*>(s.D + M);
    s.F = reinterpret_cast<double*>(s.cfg + (size_t)a.G * JPW) + SMAX * JPW;
    // stage latencies (0 beyond S_c: never used)
    for (int e = lane; e < M * C * SMAX; e += 64) {
      const int k = e % SMAX;
      const int c = (e / SMAX) % C;
      const int m = e / (SMAX * C);
      s.T[e] = k < a.cfg_stages[c] ? a.stage_lat[((int64_t)m * C + c) * a.smax_in + k] : 0.0;
    }
    for (int m = lane; m < M; m += 64) s.D[m] = a.d_single[m];
    if (lane < JPW)
      for (int g = 0; g < a.G; ++g) {
        int c = valid ? a.group_cfg[(int64_t)p * a.G + g] : -1;
        if (c < 0 || c >= C) c = 0;  // a group hosting nothing is never chosen
        s.cfg[g * JPW + lane] = (uint16_t)c;
      }
  }
  // the sentinel row: stage 0 never wins, the other stages are never committed
  for (int e = lane; e < SMAX * JPW; e += 64) s.F[e - SMAX * JPW] = e < JPW ? __builtin_inf() : 0.0;
  __syncthreads();
  return s;
}

// The wavefront-uniform part of a request and this lane's hosting groups:
// arrival t, model m, hosting mask and the two lowest hosting groups (-1, the
// sentinel row, where there is none).
template <int MB>
struct Plan {
  using MaskT = typename LaneMasks<MB>::MaskT;
  double t;
  int m;
  MaskT mask;
  int g0, g1;
  // whether some lane of the wavefront hosts the model on more than two
  // groups (a ballot: wavefront-uniform)
  __device__ __forceinline__ bool extra() const {
    const MaskT r1 = mask & (mask - 1);
    return __builtin_amdgcn_ballot_w64((r1 & (r1 - 1)) != 0) != 0;
  }
};

template <int MB>
__device__ __forceinline__ Plan<MB> make_plan(const SpecArgs& a, const LaneMasks<MB>& msk, double t, int m) {
  Plan<MB> pl;
  pl.t = t;
  pl.m = m;
  const bool known = (unsigned)m < (unsigned)a.M;
  const auto x = msk.get(m);  // register moves only: cheaper than a branch around them
  pl.mask = known ? x : 0;
  const auto r1 = pl.mask & (pl.mask - 1);
  pl.g0 = lowest_or_m1(pl.mask);
  pl.g1 = lowest_or_m1(r1);
  return pl;
}

// LDS reads of one request, issued together: the rows of the two lowest
// hosting groups, the stage-0 entries of up to six more hosts when some lane
// of the wavefront has them, and the model's table row.  X: 0 never reads the
// extra hosts, 1 always, 2 when ex (wavefront-uniform) is set.
template <int SMAX, bool UCFG>
struct Reads {
  static constexpr int kX = 6;
  double A[SMAX], B[SMAX], X[kX];
  int hx[kX];
  bool extra;
  double L[UCFG ? SMAX : 1];
  double d;
};

template <int SMAX, bool UCFG, int MB, int JPW, int X>
__device__ __forceinline__ Reads<SMAX, UCFG> issue_reads(const SpecLds<SMAX, UCFG>& s, const Plan<MB>& pl,
                                                         int lane, bool ex) {
  constexpr int kX = Reads<SMAX, UCFG>::kX;
  Reads<SMAX, UCFG> rd;
#pragma unroll
  for (int k = 0; k < SMAX; ++k) {
    rd.A[k] = s.F[(pl.g0 * SMAX + k) * JPW + lane];
    rd.B[k] = s.F[(pl.g1 * SMAX + k) * JPW + lane];
  }
  rd.extra = X == 1 || (X == 2 && ex);
  if (rd.extra) {
    auto rest = pl.mask & (pl.mask - 1);
    rest &= rest - 1;
#pragma unroll
    for (int q = 0; q < kX; ++q) {
      rd.hx[q] = lowest_or_m1(rest);
      rest &= rest - 1;
    }
#pragma unroll
    for (int q = 0; q < kX; ++q) rd.X[q] = s.F[(rd.hx[q] * SMAX) * JPW + lane];
  }
  const int mi = (unsigned)pl.m < 64u ? pl.m : 0;
  if constexpr (UCFG) {
    const double* row = s.T + mi * (SMAX + 1);
#pragma unroll
    for (int k = 0; k < SMAX; ++k) rd.L[k] = row[k];
    rd.d = row[SMAX];
  } else {
    rd.d = s.D[mi];
  }
  return rd;
}

// Dispatch (least stage-0 free time among the hosting groups, lowest index on
// ties), stage chain, admission (finish <= t + scale * d_single[m]) and
// commit of one request on the lane's state.  Returns whether the request is
// served (never on an inactive lane); out is its finish time (-1 dropped, -2
// no hosting group).  Requests that are not served write the spare row G.
// X as for issue_reads (rd.extra: the extra hosts were read).
template <int SMAX, bool UCFG, int MB, int JPW, int X>
__device__ __forceinline__ bool finish_step(const SpecLds<SMAX, UCFG>& s, const Plan<MB>& pl,
                                            const Reads<SMAX, UCFG>& rd, int lane, double scale, int C, int G,
                                            bool active, double& out) {
  constexpr int kX = Reads<SMAX, UCFG>::kX;
  // g1 > g0, and further hosts come in increasing order: strict comparisons
  // keep the lowest index among equal free times (a missing host is the
  // sentinel row, +inf: with no host at all, g is -1 and nothing commits)
  const bool use_b = rd.B[0] < rd.A[0];
  int g = use_b ? pl.g1 : pl.g0;
  double Fv[SMAX];
#pragma unroll
  for (int k = 0; k < SMAX; ++k) Fv[k] = use_b ? rd.B[k] : rd.A[k];
  if (X == 1 || (X == 2 && rd.extra)) {
    double best = Fv[0];
#pragma unroll
    for (int q = 0; q < kX; ++q) {
      if (rd.X[q] < best) {
        best = rd.X[q];
        g = rd.hx[q];
      }
    }
    // hosts after the eighth
    typename LaneMasks<MB>::MaskT rest = pl.mask;
    if (__popcll((uint64_t)pl.mask) > 8) {
#pragma unroll
      for (int q = 0; q < 8; ++q) rest &= rest - 1;
      while (rest) {
        const int h = ctz_any(rest);
        rest &= rest - 1;
        const double v = s.F[(h * SMAX) * JPW + lane];
        if (v < best) {
          best = v;
          g = h;
        }
      }
    }
    if (g != pl.g0 && g != pl.g1) {
#pragma unroll
      for (int k = 0; k < SMAX; ++k) Fv[k] = s.F[(g * SMAX + k) * JPW + lane];
    }
  }
  double Lv[SMAX];
  if constexpr (UCFG) {
#pragma unroll
    for (int k = 0; k < SMAX; ++k) Lv[k] = rd.L[k];
  } else {
    const int c = s.cfg[(g < 0 ? 0 : g) * JPW + lane];
    const int mi = (unsigned)pl.m < 64u ? pl.m : 0;
    const double* Lrow = s.T + ((size_t)mi * C + c) * SMAX;
#pragma unroll
    for (int k = 0; k < SMAX; ++k) Lv[k] = Lrow[k];
  }
  // projection through the stage chain.  A stage past the group's depth has
  // zero latency: its free time is always the last real stage's (so at most
  // the new finish time), and the finish time passes it unchanged.
  double f[SMAX];
  double prev = pl.t;
#pragma unroll
  for (int k = 0; k < SMAX; ++k) {
    f[k] = vmax(prev, Fv[k]) + Lv[k];
    prev = f[k];
  }
  const double slo = scale * rd.d;
  const double deadline = pl.t + slo;
  const bool hosted = pl.mask != 0;
  const bool served = active && hosted && !(prev > deadline);
  out = served ? prev : (hosted ? -1.0 : -2.0);
  const int row = served ? g : G;
#pragma unroll
  for (int k = 0; k < SMAX; ++k) s.F[(row * SMAX + k) * JPW + lane] = f[k];
  return served;
}

struct SpecLane {
  int job, p, frow;
  bool valid;
  double scale;
};

template <int JPW>
__device__ __forceinline__ SpecLane spec_lane(const SpecArgs& a, int jb, int lane) {
  SpecLane l;
  l.job = jb * JPW + lane;
  l.valid = lane < JPW && l.job < a.J;
  l.p = l.valid ? l.job / a.K : 0;
  l.scale = l.valid ? a.slo_scale[l.job % a.K] : 0.0;
  l.frow = -1;
  if (l.valid)
    for (int f = 0; f < a.n_finish; ++f)
      if (a.finish_jobs[f] == l.job) l.frow = f;
  return l;
}

// Arrivals of [from, to) in chunks of 64 (lane r holds request base + r),
// the next chunk loaded while the current one is simulated.
struct TraceChunks {
  double tv, tn;
  int mv, mn;
  int64_t to;
  __device__ __forceinline__ void first(const SpecArgs& a, int64_t from, int64_t to_, int lane) {
    to = to_;
    const int64_t i = from + lane;
    tn = i < to ? a.t[i] : 0.0;
    mn = i < to ? a.model[i] : 0;
  }
  __device__ __forceinline__ void advance(const SpecArgs& a, int64_t next_base, int lane) {
    tv = tn;
    mv = mn;
    const int64_t i = next_base + lane;
    tn = i < to ? a.t[i] : 0.0;
    mn = i < to ? a.model[i] : 0;
  }
};

// Simulate requests [from, to) of one lane (only while the lane is active)
// with the next request's preparation overlapping the current one's LDS
// reads.  EXTRA false: no lane hosts a model on more than two groups.  ROWS
// false: no lane writes finish rows (the code for them is left out).  Per
// chunk of 64 requests: chunk_begin(base) returns 0 to stop the loop (once no
// lane of the wavefront is active), 1 to run the chunk, 2 to run it with
// finish rows; result(i, r, out, served, rows) sees every simulated request
// (on an inactive lane with served false and out meaningless; rows: the chunk
// writes finish rows), after a placeholder call per chunk (i = base - 1,
// served and rows false), chunk_end(base, cnt) closes the chunk.
template <int SMAX, int MB, bool UCFG, int JPW, bool EXTRA, bool ROWS, class Begin, class Result, class End>
__device__ __forceinline__ void spec_range(const SpecArgs& a, const SpecLds<SMAX, UCFG>& s,
                                           const LaneMasks<MB>& msk, const SpecLane& ln, int lane, int64_t from, int64_t to, const bool& active, Begin chunk_begin,
                                           Result result, End chunk_end) {
  if (from >= to) return;
  const int li = lane & (JPW - 1);  // lanes past JPW hold no job: they read a valid lane's slot
  TraceChunks tc;
  tc.first(a, from, to, lane);
  tc.advance(a, from + 64, lane);
  Plan<MB> cur = make_plan<MB>(a, msk, readlane_f64(tc.tv, 0), __builtin_amdgcn_readlane(tc.mv, 0));
  for (int64_t cb = from; cb < to; cb += 64) {
    const int code = chunk_begin(cb);
    if (code == 0) return;
    const int cnt = (int)(to - cb < 64 ? to - cb : 64);
    const bool last_chunk = cb + 64 >= to;
    // lane r: the request after request r (lane 63: the next chunk's first;
    // past the range a placeholder)
    const int from_lane = ((lane + 1) & 63) << 2;
    int t1_lo = __builtin_amdgcn_ds_bpermute(from_lane, __double2loint(tc.tv));
    int t1_hi = __builtin_amdgcn_ds_bpermute(from_lane, __double2hiint(tc.tv));
    int m1 = __builtin_amdgcn_ds_bpermute(from_lane, tc.mv);
    const int n_lo = __builtin_amdgcn_readlane(__double2loint(tc.tn), 0);
    const int n_hi = __builtin_amdgcn_readlane(__double2hiint(tc.tn), 0);
    const int n_m = __builtin_amdgcn_readlane(tc.mn, 0);
    if (lane == 63) {
      t1_lo = n_lo;
      t1_hi = n_hi;
      m1 = n_m;
    }
    const bool rows = ROWS && code == 2;
    // each request's bookkeeping (result) runs one request late, while the
    // next request's reads are in flight; the first call of a chunk is a
    // placeholder (not served: its accept bit is shifted out of the word at
    // the chunk's end, and it writes no row)
    double out_p = 0.0;
    bool served_p = false;
    for (int r = 0; r < cnt; ++r) {
      // the extra-host flag of this request (a ballot) is taken here, at the
      // top, so that its branch is a scalar one
      const bool ex = EXTRA && cur.extra();
      const Reads<SMAX, UCFG> rd = issue_reads<SMAX, UCFG, MB, JPW, EXTRA ? 2 : 0>(s, cur, li, ex);
      result(cb + r - 1, r - 1, out_p, served_p, rows && r > 0);
      // the next request, prepared while this one's reads are in flight
      const double t_nx =
          __hiloint2double(__builtin_amdgcn_readlane(t1_hi, r), __builtin_amdgcn_readlane(t1_lo, r));
      const Plan<MB> nxt = make_plan<MB>(a, msk, t_nx, __builtin_amdgcn_readlane(m1, r));
      served_p = finish_step<SMAX, UCFG, MB, JPW, EXTRA ? 2 : 0>(s, cur, rd, li, ln.scale, a.C, a.G, active, out_p);
      cur = nxt;
    }
    result(cb + cnt - 1, cnt - 1, out_p, served_p, rows);
    chunk_end(cb, cnt);
    if (!last_chunk) tc.advance(a, cb + 128, lane);
  }
}


// Pass 0 of one wavefront (the per-request output rows are written by
// spec_rows once the rounds have made every saved state exact).
template <int SMAX, int MB, bool UCFG, int JPW, bool EXTRA>
__device__ __forceinline__ void spec_pass0_body(const SpecArgs& a, double* lds, int lane, int k,
                                                const SpecLane& ln, int c0) {
  LaneMasks<MB> msk;
  (void)msk.load(a.host_mask + (int64_t)ln.p * a.M, a.M, a.G, ln.valid);
  const auto s = spec_tables<SMAX, UCFG, JPW>(a, lds, lane, ln.p, ln.valid, c0);
  const int GS = a.G * SMAX;
  if (lane < JPW)
    for (int q = 0; q < GS; ++q) s.F[q * JPW + lane] = 0.0;
  if (k == 0 && ln.valid) a.claimed[ln.job] = 0;

  const int64_t b = seg_bound(a.n, a.nseg, k), e = seg_bound(a.n, a.nseg, k + 1);
  const int64_t J = a.J;
  const bool on = true;
  // warm-up: the requests just before the segment, from the empty state, give
  // its start state (usually already the exact one: the rounds then find
  // nothing to redo); one pass over [w0, e) records from b on
  const int64_t wu = (a.warmup + 63) & ~(int64_t)63;
  const int64_t w0 = k == 0 ? b : (b > wu ? b - wu : 0);
  const size_t seg_base = ((size_t)k * GS) * J + ln.job;
  int64_t served = 0;
  uint64_t fsum = 0, word = 0;
  const size_t ck0 = (size_t)k * a.ckps;
  if (w0 == b && ln.valid)
    for (int q = 0; q < GS; ++q) a.st_start[seg_base + (size_t)q * J] = 0.0;
  spec_range<SMAX, MB, UCFG, JPW, EXTRA, false>(
      a, s, msk, ln, lane, w0, e, on,
      [&](int64_t cb) {
        if (cb == b) {
          // the warm-up counts nothing
          served = 0;
          fsum = 0;
        }
        if (cb == b && w0 < b && ln.valid)
          for (int q = 0; q < GS; ++q) a.st_start[seg_base + (size_t)q * J] = s.F[q * JPW + lane];
        if (cb > b && (cb - b) % a.ck == 0 && ln.valid) {
          const size_t j = ck0 + (size_t)((cb - b) / a.ck - 1);
          for (int q = 0; q < GS; ++q) a.ckpt[(j * GS + q) * J + ln.job] = s.F[q * JPW + lane];
          a.ck_served[j * J + ln.job] = served;
          a.ck_fsum[j * J + ln.job] = fsum;
        }
        return 1;
      },
      [&](int64_t i, int r, double out, bool sv, bool rows) {
        (void)i;
        (void)r;
        (void)rows;
        fsum += sv ? bits_of(out) : 0;
        word = push_bit(word, sv);
      },
      [&](int64_t cb, int cnt) {
        word = chunk_word(word, cnt);
        if (cb >= b && ln.valid) a.bitmap[(cb >> 6) * J + ln.job] = word;
        served += __popcll(word);
        word = 0;
      });

  // an empty segment's start state is its warm-up end, and it counts nothing
  if (b == e && w0 < b && ln.valid)
    for (int q = 0; q < GS; ++q) a.st_start[seg_base + (size_t)q * J] = s.F[q * JPW + lane];
  if (b == e) {
    served = 0;
    fsum = 0;
  }
  if (!ln.valid) return;
  for (int q = 0; q < GS; ++q) a.st_end[seg_base + (size_t)q * J] = a.xch[0][seg_base + (size_t)q * J] = s.F[q * JPW + lane];
  a.seg_served[(size_t)k * J + ln.job] = served;
  a.seg_fsum[(size_t)k * J + ln.job] = fsum;
}

// Pass 0: every (job, segment) from a warmed-up estimate of its start state;
// the state is also saved every ck requests (checkpoints for the rounds).
// Every kernel of the speculative pipeline that simulates requests comes in
// four variants, all launched: UCFG (all groups of all placements share one
// configuration) and EXTRA (some lane of the wavefront hosts a model on more
// than two groups) select the code; a workgroup whose data do not match its
// variant returns at once, before any side effect.
template <int SMAX, int MB, bool UCFG, int JPW, bool EXTRA>
__global__ __launch_bounds__(64) void spec_pass0(const SpecArgs a) {
  if ((a.cfg_info[0] != 0) != UCFG) return;
  const int c0 = UCFG ? a.cfg_info[1] : 0;
  extern __shared__ double lds[];
  const int lane = threadIdx.x;
  const int jb = blockIdx.x % a.njb;
  const int k = blockIdx.x / a.njb;
  const SpecLane ln = spec_lane<JPW>(a, jb, lane);
  {
    LaneMasks<MB> m0;
    const bool many = m0.load(a.host_mask + (int64_t)ln.p * a.M, a.M, a.G, ln.valid);
    if ((__builtin_amdgcn_ballot_w64(many) != 0) != EXTRA) return;
  }
  spec_pass0_body<SMAX, MB, UCFG, JPW, EXTRA>(a, lds, lane, k, ln, c0);
}

// Per job: served counts and finish-time sums over the segments, and the
// ordered hash over the accept words (the final step of the pipeline).
__device__ __forceinline__ void final_body(const SpecArgs& a, int64_t job) {
  if (job >= a.J) return;
  const int64_t J = a.J;
  int64_t served = 0;
  uint64_t fsum = 0;
  for (int k = 0; k < a.nseg; ++k) {
    served += a.seg_served[(size_t)k * J + job];
    fsum += a.seg_fsum[(size_t)k * J + job];
  }
  // the hash is sequential over words: the next 16 words are loaded while
  // the current 16 are folded in
  constexpr int kB = 16;
  uint64_t h = 0;
  const uint64_t* col = a.bitmap + job;
  const int64_t nb = a.nw / kB;
  uint64_t cur[kB], nxt[kB];
  if (nb > 0) {
#pragma unroll
    for (int q = 0; q < kB; ++q) cur[q] = col[(int64_t)q * J];
  }
  for (int64_t bi = 0; bi < nb; ++bi) {
    const int64_t nbase = (bi + 1 < nb ? bi + 1 : bi) * kB;
#pragma unroll
    for (int q = 0; q < kB; ++q) nxt[q] = col[(nbase + q) * J];
#pragma unroll
    for (int q = 0; q < kB; ++q) h = (h ^ cur[q]) * kSpecHashMul;
#pragma unroll
    for (int q = 0; q < kB; ++q) cur[q] = nxt[q];
  }
  for (int64_t w = nb * kB; w < a.nw; ++w) h = (h ^ col[w * J]) * kSpecHashMul;
  a.out_served[job] = served;
  if (a.out_attain) a.out_attain[job] = a.n > 0 ? (double)served / (double)a.n : 0.0;
  if (a.out_digest) {
    a.out_digest[2 * job] = h;
    a.out_digest[2 * job + 1] = fsum;
  }
}

// Per-request output rows of the jobs that have one.  Pass 0 and the rounds
// write none: once the rounds are done, every saved state is the exact state
// at its point of the trace (a segment's start, and every ck requests into
// it), so each piece of ck requests is simulated again from the state before
// it, all pieces at once, and only the rows are written.  Lanes are jobs with
// a row (JPW per wavefront); blocks are row blocks x segments x pieces, and a
// piece past its segment's end returns at once.
// The extra-host code (some lane hosts a model on more than two groups) is
// chosen per wavefront at run time, so that every row piece, and the final
// step in the dispatch's first nfb workgroups, run in one dispatch.
template <int SMAX, int MB, bool UCFG, int JPW, bool EXTRA>
__device__ __forceinline__ void rows_body(const SpecArgs& a, double* lds, int lane, const SpecLane& ln, int c0,
                                          int k, int pc, int64_t pb, int64_t pe) {
  LaneMasks<MB> msk;  // loaded again here: one copy per body keeps it in registers
  (void)msk.load(a.host_mask + (int64_t)ln.p * a.M, a.M, a.G, ln.valid);
  const auto s = spec_tables<SMAX, UCFG, JPW>(a, lds, lane, ln.p, ln.valid, c0);
  const int GS = a.G * SMAX;
  const int64_t J = a.J;
  if (lane < JPW)
    for (int q = 0; q < GS; ++q)
      s.F[q * JPW + lane] = !ln.valid ? 0.0
                            : pc == 0 ? a.st_start[((size_t)k * GS + q) * J + ln.job]
                                      : a.ckpt[(((size_t)k * a.ckps + pc - 1) * GS + q) * J + ln.job];
  const bool on = true;
  spec_range<SMAX, MB, UCFG, JPW, EXTRA, true>(
      a, s, msk, ln, lane, pb, pe, on, [](int64_t) { return 2; },
      [&](int64_t i, int r, double out, bool sv, bool rows) {
        (void)r;
        (void)sv;
        if (rows && ln.valid) a.out_finish[(int64_t)ln.frow * a.n + i] = out;
      },
      [](int64_t, int) {});
}

template <int SMAX, int MB, bool UCFG, int JPW>
__global__ __launch_bounds__(64) void spec_rows(const SpecArgs a, int nfb) {
  if (a.cfg_info[2] != 0) return;  // a re-run gave up: other kernels write the rows
  if ((a.cfg_info[0] != 0) != UCFG) return;
  if ((int)blockIdx.x < nfb) {
    final_body(a, (int64_t)blockIdx.x * 64 + threadIdx.x);
    return;
  }
  const int bx = (int)blockIdx.x - nfb;
  const int c0 = UCFG ? a.cfg_info[1] : 0;
  extern __shared__ double lds[];
  const int lane = threadIdx.x;
  const int nrb = (a.n_finish + JPW - 1) / JPW;
  const int np = a.ckps + 1;
  const int rb = bx % nrb;
  const int pc = (bx / nrb) % np;
  const int k = bx / (nrb * np);
  const int64_t b = seg_bound(a.n, a.nseg, k), e = seg_bound(a.n, a.nseg, k + 1);
  const int64_t pb = b + (int64_t)pc * a.ck;
  if (pb >= e) return;
  const int64_t pe = e - pb < a.ck ? e : pb + a.ck;
  SpecLane ln;
  const int f = rb * JPW + lane;
  ln.valid = lane < JPW && f < a.n_finish;
  ln.job = ln.valid ? a.finish_jobs[f] : 0;
  ln.p = ln.valid ? ln.job / a.K : 0;
  ln.scale = ln.valid ? a.slo_scale[ln.job % a.K] : 0.0;
  ln.frow = ln.valid ? f : -1;
  bool many;
  {
    LaneMasks<MB> msk;
    many = msk.load(a.host_mask + (int64_t)ln.p * a.M, a.M, a.G, ln.valid);
  }
  if (__builtin_amdgcn_ballot_w64(many) != 0)
    rows_body<SMAX, MB, UCFG, JPW, true>(a, lds, lane, ln, c0, k, pc, pb, pe);
  else
    rows_body<SMAX, MB, UCFG, JPW, false>(a, lds, lane, ln, c0, k, pc, pb, pe);
}

// Lists the segments k >= 1 whose start state is not, bit for bit, their
// predecessor's end state.  One thread per job and segment (blockIdx.y = k - 1).
__global__ __launch_bounds__(256) void spec_list(const SpecArgs a, int GS) {
  const int64_t job = (int64_t)blockIdx.x * 256 + threadIdx.x, J = a.J;
  if (job >= J) return;
  const int k = (int)blockIdx.y + 1;
  const size_t own = ((size_t)k * GS) * J + job, prv = own - (size_t)GS * J;
  bool differ = false;
  for (int x = 0; x < GS; ++x)
    differ |= bits_of(a.st_start[own + (size_t)x * J]) != bits_of(a.st_end[prv + (size_t)x * J]);
  if (differ) a.list[0][atomicAdd(a.count, 1)] = make_int2((int)job, k);
}

// Per job: totals over segments and the ordered digest over the accept words.
__global__ __launch_bounds__(64) void spec_final(const SpecArgs a) {
  if (a.cfg_info[2] != 0) return;  // a re-run gave up: other kernels write the results
  final_body(a, (int64_t)blockIdx.x * 64 + threadIdx.x);
}

}  // namespace
}  // namespace as_dev

namespace as_dev {
namespace {

// Whether every group that a placement uses (configuration >= 0) has one and
// the same configuration; cfg_info = {uniform, that configuration, 0 (no
// fix-up has given up)}; the fix-ups' lists and work start empty.  One workgroup of 1024 threads.
__global__ __launch_bounds__(1024) void spec_cfg_check(const int32_t* group_cfg, int64_t cells, int n_configs,
                                                       int32_t* cfg_info, int32_t* count, int32_t* taken,
                                                       unsigned long long* work) {
  __shared__ int lo[1024], hi[1024];
  int l = 0x7FFFFFFF, h = -1;
  for (int64_t i = threadIdx.x; i < cells; i += 1024) {
    const int c = group_cfg[i];
    if (c >= 0) {
      l = c < l ? c : l;
      h = c > h ? c : h;
    }
  }
  lo[threadIdx.x] = l;
  hi[threadIdx.x] = h;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      lo[threadIdx.x] = min(lo[threadIdx.x], lo[threadIdx.x + w]);
      hi[threadIdx.x] = max(hi[threadIdx.x], hi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const bool none = hi[0] < 0;
    // configurations >= n_configs are invalid input: such calls take the
    // per-lane tables, which clamp them
    cfg_info[0] = none || (lo[0] == hi[0] && lo[0] < n_configs) ? 1 : 0;
    cfg_info[1] = none ? 0 : lo[0];
    cfg_info[2] = 0;
    *work = 0;
    for (int q = 0; q < kSpecRounds + 2; ++q) count[q] = taken[q] = 0;
  }
}

template <int SMAX, int MB, int JPW>
hipError_t spec_launch_all(const SpecArgs& a, size_t lds_u, size_t lds_g, hipStream_t s) {
  const dim3 grid((unsigned)((int64_t)a.njb * a.nseg)), block(64);
  hipLaunchKernelGGL((spec_pass0<SMAX, MB, true, JPW, false>), grid, block, lds_u, s, a);
  hipLaunchKernelGGL((spec_pass0<SMAX, MB, true, JPW, true>), grid, block, lds_u, s, a);
  hipLaunchKernelGGL((spec_pass0<SMAX, MB, false, JPW, false>), grid, block, lds_g, s, a);
  hipLaunchKernelGGL((spec_pass0<SMAX, MB, false, JPW, true>), grid, block, lds_g, s, a);
  if (a.nseg > 1) {
    hipLaunchKernelGGL(spec_list, dim3((unsigned)((a.J + 255) / 256), (unsigned)(a.nseg - 1)), dim3(256), 0, s, a,
                       a.G * SMAX);
    // a job's segments are settled after nseg - 1 rounds, whatever the data
    for (int q = 1; q <= std::min(a.nseg - 1, kSpecRounds + 1); ++q) {
      const hipError_t e = as_host::launch_fix_any(SMAX, a, q, s);
      if (e != hipSuccess) return e;
    }
  }
  const int nfb = (int)((a.J + 63) / 64);
  if (a.n_finish > 0) {
    // the output rows, from the exact saved states, all pieces at once, and
    // in the same dispatch (its first nfb workgroups) the final step
    const dim3 rgrid((unsigned)(nfb + (int64_t)((a.n_finish + JPW - 1) / JPW) * a.nseg * (a.ckps + 1)));
    hipLaunchKernelGGL((spec_rows<SMAX, MB, true, JPW>), rgrid, block, lds_u, s, a, nfb);
    hipLaunchKernelGGL((spec_rows<SMAX, MB, false, JPW>), rgrid, block, lds_g, s, a, nfb);
  } else {
    hipLaunchKernelGGL(spec_final, dim3((unsigned)nfb), block, 0, s, a);
  }
  return hipGetLastError();
}

// Workgroups (one wavefront each) of the pass-0 kernel that one compute unit
// holds at this LDS size.
template <int SMAX, int MB, int JPW>
int spec_occupancy(size_t lds) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, spec_pass0<SMAX, MB, true, JPW, false>, 64, lds) != hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}

template <int SMAX>
int spec_occupancy_mb(int G, size_t lds) {
  return G <= 32 ? spec_occupancy<SMAX, 32, kSpecJobsPerWave>(lds) : spec_occupancy<SMAX, 64, kSpecJobsPerWave>(lds);
}

template <int SMAX>
hipError_t spec_launch_mb(int G, const SpecArgs& a, size_t l1, size_t l2, hipStream_t s) {
  return G <= 32 ? spec_launch_all<SMAX, 32, kSpecJobsPerWave>(a, l1, l2, s)
                 : spec_launch_all<SMAX, 64, kSpecJobsPerWave>(a, l1, l2, s);
}

}  // namespace
}  // namespace as_dev

namespace as_host {

// One round (spec_fix): up to two wavefronts per SIMD take the entries in turn.
hipError_t launch_fix_any(int smax, const as_dev::SpecArgs& a, int q, hipStream_t s) {
  const int W = std::max(4, pow2ceil(a.G));
  const int64_t blocks = std::min<int64_t>((int64_t)a.J * (a.nseg - 1), 8 * (int64_t)compute_units());
  const size_t lds = as_dev::lean_lds_bytes(W, a.M, pow2ceil(a.C), smax, false, 1);
  switch (W) {
    case 4: return launch_fix<4>(smax, a, q, blocks, lds, s);
    case 8: return launch_fix<8>(smax, a, q, blocks, lds, s);
    case 16: return launch_fix<16>(smax, a, q, blocks, lds, s);
    case 32: return launch_fix<32>(smax, a, q, blocks, lds, s);
    default: return launch_fix<64>(smax, a, q, blocks, lds, s);
  }
}

}  // namespace as_host

namespace as_host {

int compute_units() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) v = 256;
    cache[dev] = v;
  }
  return cache[dev];
}

namespace {



// Warm-up requests before a segment.  A shorter warm-up leaves more start
// states wrong, a longer one is simulated for nothing (1000 placements, 900,000
// requests, 64 segments, one seed: 4096 -> 12.2 ms, 8192 -> 11.3, 16384 -> 12.5,
// and on another, whose runs meet later, 99, 31 and 29).
constexpr int64_t kSpecWarmup = 8192;
// Requests per segment at least: beyond this the warm-up is nearly all of pass
// 0 (1000 placements, 200,000 requests: segments of 12,500 8.0 ms, 6250 7.2,
// 3125 6.5).
constexpr int64_t kSpecMinSegment = 2048;
// Requests between saved states: the closer, the sooner a re-run sees that it
// has met the old results (2048 against 8192: 11.3 and 13.4 ms on the workload
// above); doubled up to kSpecCheckpointMax until they fit kSpecCheckpointBytes.
constexpr int64_t kSpecCheckpoint = 2048, kSpecCheckpointMax = 8192;
constexpr int64_t kSpecCheckpointBytes = 512ll << 20;
// When the fix-ups give up and leave the call to the group-per-lane kernels,
// because under traffic that keeps groups saturated runs from different states
// never meet.  What they have cost by then is lost, and those kernels' time is
// what giving up costs, so the line lies at shares of that time (a re-run's
// request takes kSpecFixNs of a SIMD):
//   * kSpecTotal of it in all, and kSpecFirst in the first round.  Calls that
//     were worth finishing took 0.05 to 0.15 in the first round and up to 0.3 in
//     all, the others 0.22 to 8 in the first round;
//   * at once where more than kSpecPairs of all segments start wrong (worth
//     finishing: up to 0.45);
//   * after the first round, where more than kSpecAgain of the segments that it
//     took are listed again, so that the rounds leave most of the trace to the
//     job-by-job step (300 jobs, 200,000 requests: 0.71 and 0.73 took 13 and 15
//     ms, 0.80 took 31, where the group-per-lane kernels take 18); kSpecAgainSome
//     where they were at most kSpecSome of all segments, and never where they
//     were at most kSpecFew, since the few jobs then left cost no more than
//     giving up (20 to 1200 jobs of 132,000 to 914,000 requests, finished / given
//     up in ms: share 0.02 to 0.08 at 0.79 to 0.995 listed again 18.5 / 60, 38 /
//     105, 40 / 71, 20 / 26 and level on three others; 0.19 at 0.87 and 0.93 45 /
//     58 and 24 / 36; 0.12 to 0.23 at 0.93 to 0.995 30 / 25, 41 / 28, 52 / 34, 62
//     / 45; 0.27 to 0.4 at 0.84 to 0.92 65 / 53, 46 / 41, 47 / 40).
// Measured, giving up and finished: 1000 placements of 16 four-stage groups,
// 900,000 requests, seven seeds and loads 91 to 108 and 22 to 78 ms; 4000 of
// them 106 and 37; 300,000 requests 36 and 17; and where groups stay saturated
// 88 and 108 to 545.
constexpr double kSpecTotal = 1.0 / 3.0, kSpecFirst = 0.18, kSpecFixNs = 90.0;
constexpr double kSpecPairs = 0.5, kSpecAgain = 0.75;
constexpr double kSpecFew = 0.1, kSpecSome = 0.25, kSpecAgainSome = 0.93;

}  // namespace

// Stream-ordered workspace allocation from a memory pool private to this
// library, one per device, whose release threshold is at its maximum: the
// workspace freed by one call is reused by the next instead of going back to
// the driver, and the process's default pool keeps its own settings.  Where a
// private pool cannot be created, the default pool serves as it is.
hipError_t pool_alloc(void** p, size_t bytes, hipStream_t s) {
  static std::mutex mu;
  static hipMemPool_t pools[64];
  static int state[64] = {0};  // 0 not tried, 1 private pool, 2 default pool
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipMallocAsync(p, bytes, s);
  int st = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    if (state[dev] == 0) {
      hipMemPoolProps props;
      std::memset(&props, 0, sizeof props);
      props.allocType = hipMemAllocationTypePinned;
      props.handleTypes = hipMemHandleTypeNone;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      state[dev] = 2;
      if (hipMemPoolCreate(&pools[dev], &props) == hipSuccess) {
        uint64_t thr = UINT64_MAX;
        (void)hipMemPoolSetAttribute(pools[dev], hipMemPoolAttrReleaseThreshold, &thr);
        state[dev] = 1;
      } else {
        (void)hipGetLastError();
      }
    }
    st = state[dev];
  }
  return st == 1 ? hipMallocFromPoolAsync(p, bytes, pools[dev], s) : hipMallocAsync(p, bytes, s);
}

// Segments per job for the speculative path: enough (job block, segment)
// wavefronts to fill the device at the occupancy the LDS allows, none shorter
// than min_seg.  ALPASERVE_SPEC_SEGMENTS forces the count (tests).
int spec_segments(int64_t n, int64_t J, int jpw, int per_cu, int64_t min_seg, int max_seg) {
  if (const char* e = getenv("ALPASERVE_SPEC_SEGMENTS")) {
    const int v = atoi(e);
    if (v >= 1) return std::min(v, as_dev::kSpecMaxSeg);
  }
  const int64_t slots = (int64_t)compute_units() * std::max(per_cu, 1);
  const int64_t njb = (J + jpw - 1) / jpw;
  int64_t k = slots / std::max<int64_t>(njb, 1);
  k = std::min<int64_t>(k, n / min_seg);
  return (int)std::max<int64_t>(1, std::min<int64_t>(k, max_seg));
}

// Nanoseconds that the group-per-lane kernels take for a call: a request of one
// wavefront takes 50 + 5.5 per doubling of its lanes + 4.5 per stage alone on
// its SIMD (79 at 4 lanes and 4 stages, 90 at 16 and 4) and three quarters of
// that per wavefront beyond.
double lean_ns(const KArgs& k, int smax) {
  const int W = pow2ceil(k.G);
  const double waves = std::ceil((double)k.J / (64 / W));
  return (double)k.n * (50.0 + 5.5 * std::log2((double)W) + 4.5 * smax) *
         std::max(1.0, 0.75 * waves / (4.0 * compute_units()));
}

// Whether the speculative kernels beat the group-per-lane kernels on this
// call, by a model in nanoseconds of one wavefront: a request of pass 0, with 64
// jobs, 150 + 35 per stage (287 at 4 stages), over a segment and its warm-up; the
// fix-ups are taken as 2 ms.  The speculative kernels must promise 0.4 of the
// other time, because traffic under which runs do not meet costs both.  Measured
// on 16 four-stage groups, where runs meet / do not / the group-per-lane kernels
// alone: promise 0.08 (1000 placements, 900,000 requests) 11 to 79 / 88 to 105 /
// 83 to 93 ms; 0.34 (8000, 500,000) 31 / 86 to 97 / 70; 0.39 (8000, 300,000) 18 /
// 53 to 59 / 42; 0.43 (4000, 214,000) 9 to 20 / 25 to 29 / 20; 0.55 (1000, 99,000)
// 7 to 9 / 12 to 13 / 9; 0.64 (777 late selections of 32 two-stage groups, 76,801
// requests) - / 11 / 7.  A single segment never pays.
bool spec_pays(const KArgs& k, int smax, int nseg, int jpw, int per_cu) {
  if (nseg < 2) return false;
  const double slots = (double)compute_units() * std::max(per_cu, 1);
  const double waves_spec = std::ceil((double)k.J / jpw) * nseg;
  const double seg = (double)k.n / nseg + (double)std::min<int64_t>(kSpecWarmup, k.n);
  const double t_spec = seg * (150.0 + 35.0 * smax) * std::ceil(waves_spec / slots) + 2e6;
  return t_spec < 0.4 * lean_ns(k, smax);
}

size_t ws_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Calls that as_simulate_placements_noalloc refuses because of their
// workspace: those that segments of at least 131,072 requests would speed up
// (about 1150 cycles per request over a segment and its warm-up, and a fifth
// more, against 300 cycles, or 195 per wavefront of a SIMD) and whose
// workspace at that cut, with saved states every 8192 requests, exceeds the
// scratch.  The rule is the interface's; every other call is taken, on the
// group-per-lane kernels where the speculative workspace does not fit.
bool noalloc_refuses(const KArgs& k, int smax, int jpw, size_t scratch) {
  // wavefronts a compute unit held of the kernels that this rule was made for
  const size_t lds = (size_t)k.M * (smax + 1) * 8 + (size_t)(k.G + 2) * smax * jpw * 8;
  const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(8, 160 * 1024 / lds));
  const int nseg = spec_segments(k.n, k.J, jpw, per_cu, 131072, 64);
  if (nseg < 2) return false;
  const double simds = 4.0 * compute_units();
  const double waves_shared = std::ceil((double)k.J / (64 / pow2ceil(k.G)));
  const double t_shared = (double)k.n * std::max(300.0, 195.0 * waves_shared / simds);
  const double slots = (double)compute_units() * std::max(per_cu, 1);
  const double waves_spec = std::ceil((double)k.J / jpw) * nseg;
  const double seg = (double)k.n / nseg + (double)std::min<int64_t>(8192, k.n);
  if (seg * 1150.0 * 1.2 * std::ceil(waves_spec / slots) >= t_shared) return false;
  const size_t J = (size_t)k.J, GS = (size_t)k.G * smax, ckps = (size_t)((k.n / nseg + 64) / 8192 + 1);
  const size_t state = nseg * GS * J * 8;
  const size_t total = ws_up((size_t)((k.n + 63) / 64) * J * 8) + ws_up(state) + ws_up(2 * state) +
                       2 * ws_up(nseg * J * 8) + ws_up(nseg * ckps * GS * J * 8) + 2 * ws_up(nseg * ckps * J * 8) +
                       ws_up(256 + (size_t)nseg * 4);
  return total > scratch;
}

// Shared-trace simulation on the segment-speculative kernels.  Returns
// AS_E_LIMITS without launching when the state of one wavefront does not fit
// in the LDS, when the trace does not split into segments that pay (unless
// ALPASERVE_PATH=spec forces the kernels), or when the workspace would be too
// large.  With can_give_up the workspace outlives the call: the caller's
// gated fallback kernels read the give-up flag in it, then release it.
namespace {

// How a call is cut: segments, requests between saved states, saved states per
// segment, and the bytes of each workspace array.
struct SpecPlan {
  size_t lds_u = 0, lds_g = 0;
  int per_cu = 1, nseg = 1, ckps = 0;
  int64_t ck = 0;
  size_t bitmap = 0, state = 0, seg = 0, ckpt = 0, cks = 0, claim = 0, list = 0, small = 256, total = 0;
};

void spec_sizes(const KArgs& k, int smax, int nseg, SpecPlan& p) {
  const size_t J = (size_t)k.J, GS = (size_t)k.G * smax;
  p.nseg = nseg;
  p.ckps = (int)((k.n / nseg + 64) / p.ck + 1);
  p.bitmap = (size_t)((k.n + 63) / 64) * J * 8;
  p.state = nseg * GS * J * 8;
  p.seg = nseg * J * 8;
  p.ckpt = (size_t)nseg * p.ckps * GS * J * 8;
  p.cks = (size_t)nseg * p.ckps * J * 8;
  p.claim = J * 4;
  p.list = J * nseg * 8;
  p.total = ws_up(p.bitmap) + 4 * ws_up(p.state) + 2 * ws_up(p.seg) + ws_up(p.ckpt) + 2 * ws_up(p.cks) +
            ws_up(p.claim) + 2 * ws_up(p.list) + ws_up(p.small);
}

// Whether the speculative kernels take the call (sizes, LDS, segments that pay
// or are forced), and how they cut it.  scratch: bytes of a caller's workspace,
// 0 where it is allocated.  A trace is cut into as many segments as fill the
// device; where their workspace exceeds the scratch, into as many as fit, which
// must still pay: 1000 placements of 16 four-stage groups, 900,000 requests, fit
// 256 MiB with 32 segments instead of 64.
bool spec_plan(const KArgs& k, int smax, size_t scratch, SpecPlan& p) {
  using namespace as_dev;
  if (k.n <= 0 || k.J <= 0) return false;
  const size_t lim = shared_lds_limit();
  const int jpw = kSpecJobsPerWave;
  p.lds_u = spec_lds_bytes(k.M, k.C, k.G, smax, true, jpw);
  p.lds_g = spec_lds_bytes(k.M, k.C, k.G, smax, false, jpw);
  if (p.lds_g > lim || p.lds_u > lim) {
    p.lds_g = 0;  // no call of this size is theirs
    return false;
  }
  switch (smax) {
    case 1: p.per_cu = spec_occupancy_mb<1>(k.G, p.lds_u); break;
    case 2: p.per_cu = spec_occupancy_mb<2>(k.G, p.lds_u); break;
    case 4: p.per_cu = spec_occupancy_mb<4>(k.G, p.lds_u); break;
    default: p.per_cu = spec_occupancy_mb<8>(k.G, p.lds_u); break;
  }
  int nseg = spec_segments(k.n, k.J, jpw, p.per_cu, std::max(kSpecMinSegment, k.min_segment), kSpecMaxSeg);
  while (nseg > 1 && (int64_t)((k.J + jpw - 1) / jpw) * nseg > 0x7FFFFFFFLL) --nseg;
  p.ck = scratch ? kSpecCheckpointMax : kSpecCheckpoint;
  while (p.ck < kSpecCheckpointMax && k.n / p.ck * (int64_t)k.G * smax * k.J * 8 > kSpecCheckpointBytes) p.ck *= 2;
  if (const char* c = getenv("ALPASERVE_SPEC_CKPT")) p.ck = std::max<int64_t>(64, atoll(c) & ~(int64_t)63);
  spec_sizes(k, smax, nseg, p);
  while (scratch && p.total > scratch && p.nseg > 1 && !getenv("ALPASERVE_SPEC_SEGMENTS"))
    spec_sizes(k, smax, p.nseg - 1, p);
  return spec_forced() || spec_pays(k, smax, p.nseg, jpw, p.per_cu);
}

}  // namespace

bool spec_takes(const KArgs& k, int smax) {
  SpecPlan p;
  return spec_plan(k, smax, 0, p);
}

int run_spec(KArgs& k, int smax, hipStream_t stream, bool can_give_up, void* caller_ws,
             size_t caller_ws_bytes, void** workspace, const int32_t** gave_up) {
  using namespace as_dev;
  *workspace = nullptr;
  *gave_up = nullptr;
  const int jpw = kSpecJobsPerWave;
  SpecPlan pl;
  const bool takes = spec_plan(k, smax, caller_ws ? caller_ws_bytes : 0, pl);
  if (caller_ws && !spec_forced() && pl.lds_g > 0 && noalloc_refuses(k, smax, jpw, caller_ws_bytes)) {
    fail(AS_E_LIMITS,
         "this call, cut into segments of 131072 requests, needs more speculative-kernel workspace than the "
         "%zu-byte no-allocation scratch; as_simulate_placements takes it",
         caller_ws_bytes);
    return kSpecScratchTooSmall;
  }
  if (!takes) return AS_E_LIMITS;

  SpecArgs a;
  std::memset(&a, 0, sizeof a);
  a.t = k.t;
  a.model = k.model;
  a.n = k.n;
  a.d_single = k.d_single;
  a.stage_lat = k.stage_lat;
  a.group_cfg = k.group_cfg;
  a.host_mask = k.host_mask;
  a.slo_scale = k.slo_scale;
  a.out_served = k.out_served;
  a.out_attain = k.out_attain;
  a.out_digest = k.out_digest;
  a.out_finish = k.out_finish;
  a.M = k.M;
  a.C = k.C;
  a.smax_in = k.smax_in;
  a.G = k.G;
  a.K = k.K;
  a.J = k.J;
  a.n_finish = k.n_finish;
  std::memcpy(a.cfg_stages, k.cfg_stages, sizeof a.cfg_stages);
  std::memcpy(a.finish_jobs, k.finish_jobs, sizeof a.finish_jobs);
  a.njb = (int32_t)((k.J + jpw - 1) / jpw);
  a.nseg = pl.nseg;
  a.warmup = kSpecWarmup;
  if (const char* w = getenv("ALPASERVE_SPEC_WARMUP")) a.warmup = std::max<int64_t>(0, atoll(w));
  a.ck = pl.ck;
  a.ckps = (int32_t)pl.ckps;
  a.cap = INT64_MAX;
  a.budget = a.budget1 = a.pairs = a.few = a.some = INT64_MAX;  // never
  a.again = a.again_some = 1.0;
  if (can_give_up) {
    const double all = lean_ns(k, smax) * 4 * compute_units() / kSpecFixNs;
    a.budget = (int64_t)(kSpecTotal * all);
    a.budget1 = (int64_t)(kSpecFirst * all);
    const double starts = (double)k.J * (a.nseg - 1);
    a.pairs = (int64_t)(kSpecPairs * starts);
    a.few = (int64_t)(kSpecFew * starts);
    a.some = (int64_t)(kSpecSome * starts);
    a.again = kSpecAgain;
    a.again_some = kSpecAgainSome;
  }
  // ALPASERVE_SPEC_CAP (requests of one re-run) alone decides where it is set (tests)
  if (const char* c = getenv("ALPASERVE_SPEC_CAP"); c && can_give_up) {
    a.cap = std::max<int64_t>(64, atoll(c));
    a.budget = a.budget1 = a.pairs = a.few = a.some = INT64_MAX;
  }
  if ((int64_t)a.njb * a.nseg > 0x7FFFFFFFLL) return AS_E_LIMITS;
  a.nw = (k.n + 63) / 64;

  const size_t total = pl.total;
  char* ws = nullptr;
  hipError_t e = hipSuccess;
  if (caller_ws) {
    if (spec_forced() && total > caller_ws_bytes) {
      fail(AS_E_LIMITS,
           "this call needs %zu bytes of speculative-kernel workspace, more than the %zu-byte "
           "no-allocation scratch; as_simulate_placements takes it",
           total, caller_ws_bytes);
      return kSpecScratchTooSmall;
    }
    if (total > caller_ws_bytes) return AS_E_LIMITS;  // the kernels that need none take it
    ws = static_cast<char*>(caller_ws);
  } else {
    // a workspace beyond a quarter of the device's memory leaves the call to
    // the kernels that need none
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || total > total_b / 4) return AS_E_LIMITS;
    // ALPASERVE_SPEC_MAX_WORKSPACE (bytes) makes a larger workspace fail as a
    // failed allocation does (tests of the fallback to the other kernels)
    if (const char* cap = getenv("ALPASERVE_SPEC_MAX_WORKSPACE"))
      if ((long long)total > atoll(cap))
        return fail(AS_E_NOMEM, "workspace of %zu bytes above ALPASERVE_SPEC_MAX_WORKSPACE", total);
    e = pool_alloc(reinterpret_cast<void**>(&ws), total, stream);
    if (e != hipSuccess || !ws)
      return fail(AS_E_NOMEM, "workspace of %zu bytes: %s", total, hipGetErrorString(e));
  }
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = ws + off;
    off += ws_up(bytes);
    return p;
  };
  a.bitmap = reinterpret_cast<uint64_t*>(take(pl.bitmap));
  a.st_start = reinterpret_cast<double*>(take(pl.state));
  a.st_end = reinterpret_cast<double*>(take(pl.state));
  a.seg_served = reinterpret_cast<int64_t*>(take(pl.seg));
  a.seg_fsum = reinterpret_cast<uint64_t*>(take(pl.seg));
  a.ckpt = reinterpret_cast<double*>(take(pl.ckpt));
  a.ck_served = reinterpret_cast<int64_t*>(take(pl.cks));
  a.ck_fsum = reinterpret_cast<uint64_t*>(take(pl.cks));
  int32_t* small = reinterpret_cast<int32_t*>(take(pl.small));
  a.cfg_info = small;
  a.work = reinterpret_cast<unsigned long long*>(small + 4);
  a.count = small + 8;
  a.taken = a.count + as_dev::kSpecRounds + 2;
  a.claimed = reinterpret_cast<int32_t*>(take(pl.claim));
  for (int x = 0; x < 2; ++x) {
    a.xch[x] = reinterpret_cast<double*>(take(pl.state));
    a.list[x] = reinterpret_cast<int2*>(take(pl.list));
  }

  hipLaunchKernelGGL(spec_cfg_check, dim3(1), dim3(1024), 0, stream, k.group_cfg, (int64_t)k.P * k.G, k.C,
                     a.cfg_info, a.count, a.taken, a.work);
  switch (smax) {
    case 1: e = spec_launch_mb<1>(k.G, a, pl.lds_u, pl.lds_g, stream); break;
    case 2: e = spec_launch_mb<2>(k.G, a, pl.lds_u, pl.lds_g, stream); break;
    case 4: e = spec_launch_mb<4>(k.G, a, pl.lds_u, pl.lds_g, stream); break;
    default: e = spec_launch_mb<8>(k.G, a, pl.lds_u, pl.lds_g, stream); break;
  }
  if (e != hipSuccess || !can_give_up) {
    const hipError_t ef = caller_ws ? hipSuccess : hipFreeAsync(ws, stream);
    if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    if (ef != hipSuccess) return fail(AS_E_HIP, "workspace release failed: %s", hipGetErrorString(ef));
    return ok();
  }
  *workspace = caller_ws ? nullptr : ws;
  *gave_up = a.cfg_info + 2;
  return ok();
}

}  // namespace as_host
