// Dynamic batching (Sec. 6.5) on the batched simulator: an arriving request
// runs at once on an available group hosting its model, otherwise it waits in
// a per-model queue; a group that becomes idle runs the largest batch of one
// hosted model's queued requests that still meets the SLO; a batch's latency
// grows linearly with its size.  The exact rules are those of
// alpaserve_sim.h's as_simulate_batched.
//
// A queue needs no storage of its own.  A request joins its model's queue
// only when no hosting group is available at its arrival, and a group that
// is available then has already drained every queue of the models it hosts
// (the idle events up to the arrival are handled first, and a group with
// queued work stays busy or takes that work).  So an arrival served or
// dropped at once finds its model's queue empty, and a non-empty queue holds
// every arrival of its model since its head.  Requests leave a queue only at
// its head.  A queue is therefore a run [head, tail) of its model's arrivals
// in trace order: the launch first lists each model's arrivals (time, trace
// index, digest term) once for all jobs, and a job keeps per model only two
// positions in that list and its head's time and index.
//
// Layout: one job per wavefront (one wavefront per workgroup).  Lane g holds
// group g's stage free times; lane m holds model m's queue (positions, head
// time and index, SLO); the trace is read 64 requests at a time into
// registers.  Every decision is wave-uniform: the next idle group is a
// butterfly min over the lanes with queued work, the model with the oldest
// queued head a minimum over the model lanes, and the batch size one pass in
// which lane l runs the chain of a batch of l + 1 requests.  In LDS are the
// stage-latency table and, per model, a ring of its newest queued requests,
// small enough that every job of a launch is resident at once.  The
// arithmetic is the definition's (no FMA, v_max_f64, the batch factor rounded
// once), so served counts, digests and finish times are bit-identical to a
// sequential evaluation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "alpaserve_sim.h"
#include "sim_internal.hpp"
#include "sim_kernel.hpp"

namespace as_dev {
namespace {

// Per-model arrival lists of a trace: the requests of model m in trace order
// occupy positions [off[m], off[m + 1]) of lt (arrival time), li (trace
// index) and lmix (the digest term of the index); ord[i] is request i's rank
// among its model's requests (0 for requests of no model).
struct ListArgs {
  const double* t;
  const int32_t* model;
  int64_t n;
  int32_t M;
  uint32_t* blk;  // [nblk][M] requests of each model per block, then the exclusive prefix over blocks
  int64_t nblk;
  uint32_t* off;  // [M + 1]
  uint32_t* ord;  // [n]
  double* lt;     // [n]
  uint32_t* li;   // [n]
  uint64_t* lmix; // [n]
  uint32_t* flags;  // the batch kernel's flags word (cleared here)
};

struct BatchArgs {
  const double* t;
  const int32_t* model;
  int64_t n;
  const double* d_single;
  const double* stage_lat;
  const int32_t* group_cfg;
  const uint64_t* host_mask;
  const double* slo_scale;
  int64_t* out_served;
  uint64_t* out_digest;
  double* out_finish;
  uint32_t* flags;  // bit 0: a queue would exceed its capacity; bit 1: a queue broke the run invariant
  const uint32_t* off;
  const uint32_t* ord;
  const double* lt;
  const uint32_t* li;
  const uint64_t* lmix;
  double beta;
  int32_t M, C, smax_in, G, K, J, max_batch, qcap, ring, n_finish;  // ring: entries per model (0, 8, 16 or 32)
  int32_t cfg_stages[AS_MAX_CONFIGS];
  int32_t finish_jobs[AS_MAX_FINISH];
};

// SplitMix64 finaliser (the batched digest's per-request term).
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double rl_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ uint64_t rl_u64(uint64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

constexpr int kListBlock = 4096;  // trace requests per wavefront of the list kernels

// Walks one block's requests 64 at a time; for every chunk, body(i, ok, x,
// rank_base, mask) is called once per distinct model x of the chunk, where
// mask holds the chunk's lanes with model x and rank_base the number of
// earlier requests of x in the block (held in lane x of cnt).
template <class Body>
__device__ __forceinline__ void list_walk(const ListArgs& a, int64_t blk, uint32_t& cnt, Body body) {
  const int lane = threadIdx.x;
  const uint64_t below = (1ull << lane) - 1;
  const int64_t b = blk * kListBlock, e = std::min<int64_t>(a.n, b + kListBlock);
  for (int64_t c = b; c < e; c += 64) {
    const int64_t i = c + lane;
    const int x = i < e ? a.model[i] : -1;
    const bool ok = (unsigned)x < (unsigned)a.M;
    uint64_t rem = __builtin_amdgcn_ballot_w64(ok);
    uint32_t rank = 0;
    while (rem) {
      const int xm = __builtin_amdgcn_readlane(x, __builtin_ctzll(rem));
      const uint64_t mask = __builtin_amdgcn_ballot_w64(ok && x == xm);
      const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)cnt, xm);
      if (ok && x == xm) rank = base + (uint32_t)__builtin_popcountll(mask & below);
      if (lane == xm) cnt += (uint32_t)__builtin_popcountll(mask);
      rem &= ~mask;
    }
    body(i, i < e, ok, x, rank);
  }
}

// Requests of each model per block.
__global__ __launch_bounds__(64) void list_count(const ListArgs a) {
  uint32_t cnt = 0;
  list_walk(a, blockIdx.x, cnt, [](int64_t, bool, bool, int, uint32_t) {});
  if ((int)threadIdx.x < a.M) a.blk[(int64_t)blockIdx.x * a.M + threadIdx.x] = cnt;
}

// Exclusive prefixes: per model over the blocks, then over the models.
__global__ __launch_bounds__(64) void list_scan(const ListArgs a) {
  const int lane = threadIdx.x;
  uint32_t run = 0;
  if (lane < a.M) {
    for (int64_t b = 0; b < a.nblk; b += 8) {  // 8 loads in flight at a time
      uint32_t v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = b + k < a.nblk ? a.blk[(b + k) * a.M + lane] : 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (b + k < a.nblk) a.blk[(b + k) * a.M + lane] = run;
        run += v[k];
      }
    }
  }
  uint32_t acc = 0, mine = 0;
  for (int m = 0; m < a.M; ++m) {
    if (lane == m) mine = acc;
    acc += (uint32_t)__builtin_amdgcn_readlane((int)run, m);
  }
  if (lane < a.M) a.off[lane] = mine;
  if (lane == 0) {
    a.off[a.M] = acc;
    *a.flags = 0u;
  }
}

// Ranks and list entries.
__global__ __launch_bounds__(64) void list_fill(const ListArgs a) {
  const int lane = threadIdx.x;
  uint32_t cnt = lane < a.M ? a.blk[(int64_t)blockIdx.x * a.M + lane] : 0;
  const uint32_t offl = lane < a.M ? a.off[lane] : 0;
  list_walk(a, blockIdx.x, cnt, [&](int64_t i, bool in, bool ok, int x, uint32_t rank) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute((ok ? x : 0) << 2, (int)offl);
    if (!in) return;
    a.ord[i] = ok ? rank : 0u;
    if (ok) {
      const uint32_t pos = o + rank;
      a.lt[pos] = a.t[i];
      a.li[pos] = (uint32_t)i;
      a.lmix[pos] = mix64((uint64_t)i);
    }
  });
}

// LDS of one job: the stage-latency table [M][Cp][SMAX], then per model a ring
// of its R last queued requests (arrival times, then trace indices).
__host__ __device__ constexpr size_t batch_lds_bytes(int M, int Cp, int SMAX, int R) {
  return (size_t)M * Cp * SMAX * 8 + (size_t)M * R * 12;
}

// Smallest key over the job's W lanes, in each of them.
template <int W>
__device__ __forceinline__ double batch_min(double v) {
  v = seg_min<16>(v);
  if constexpr (W >= 32) {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = vmin(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
  }
  if constexpr (W >= 64) {
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = vmin(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
  }
  return v;
}

using LdsF64 = __attribute__((address_space(3))) double;
using LdsU32 = __attribute__((address_space(3))) uint32_t;

// Smallest of 64 lanes' values, uniform: one DPP minimum per row of 16 lanes,
// then the four rows in scalar registers.
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  v = std::min(v, dpp_u32<kXor1>(v));
  v = std::min(v, dpp_u32<kXor2>(v));
  v = std::min(v, dpp_u32<kHalfMirror>(v));
  v = std::min(v, dpp_u32<kMirror>(v));
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return std::min(std::min(r0, r1), std::min(r2, r3));
}

// W: lanes reduced per job, the group count rounded up to a power of two (at
// least 16, so the reductions inside a 16-lane row are DPP only).
//
// What bounds it is one wavefront's chain of dependent instructions and
// branches per request, not throughput: 2048 jobs are two wavefronts a SIMD.
// So a request's hosts, deadline and digest term are gathered 64 requests at a
// time; masks stay in scalar registers and reductions run only when a ballot
// is not empty; the oldest queued head is one DPP minimum; commits are selects;
// and the queues' newest entries are in LDS, because a new head read from the
// lists (L2) was waited for by the next event.  Measured: 256 placements of 16
// four-stage groups x 8 scales, 76,800 requests: 84.7 ms a call before, 67.0
// with this.
template <int W, int SMAX>
__global__ __launch_bounds__(64) void batch_kernel(const BatchArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  int cp = 1;
  while (cp < a.C) cp <<= 1;
  double* sL = reinterpret_cast<double*>(smem);  // [M][cp][SMAX]
  const int nL = a.M * cp * SMAX;
  // the rings; with none (R = 0) slot 0 of the table stands in for reads that are not used
  const uint32_t R = (uint32_t)a.ring, rmask = R ? R - 1 : 0;
  // (LDS pointers by type: a generic one would merge with the list reads into flat loads)
  LdsF64* rt = (LdsF64*)(sL + (R ? nL : 0));
  LdsU32* ri = (LdsU32*)(rt + (size_t)a.M * R);
  const int lane = threadIdx.x;
  const int64_t job = blockIdx.x;
  const int p = (int)(job / a.K);
  const double sigma = a.slo_scale[job % a.K];

  int cfg = lane < a.G ? a.group_cfg[(int64_t)p * a.G + lane] : -1;
  if (cfg >= a.C || cfg < 0) cfg = -1;
  const uint64_t exists = __builtin_amdgcn_ballot_w64(cfg >= 0);
  uint64_t hostbits = 0;  // bit m: this lane's group hosts model m
  if (cfg >= 0) {
    const uint64_t* hm = a.host_mask + (int64_t)p * a.M;
    for (int m = 0; m < a.M; ++m) hostbits |= ((hm[m] >> lane) & 1u) << m;
  }
  for (int idx = lane; idx < nL; idx += 64) {
    const int s = idx % SMAX;
    const int mc = idx / SMAX;
    const int c = mc % cp;
    const int m = mc / cp;
    sL[idx] = (c < a.C && s < a.cfg_stages[c]) ? a.stage_lat[((int64_t)m * a.C + c) * a.smax_in + s] : 0.0;
  }
  int frow = -1;
  for (int f = 0; f < a.n_finish; ++f)
    if (a.finish_jobs[f] == job) frow = f;
  double* frowp = frow >= 0 ? a.out_finish + (int64_t)frow * a.n : nullptr;
  __syncthreads();

  // lane m: the groups that host model m, its SLO and its queue, the run
  // [qh, qt) of its list starting at loff, with the head's time and index
  const bool mlane = lane < a.M;
  const uint64_t hostm = mlane ? a.host_mask[(int64_t)p * a.M + lane] & exists : 0ull;
  const double slo = mlane ? sigma * a.d_single[lane] : 0.0;
  const uint32_t loff = mlane ? a.off[lane] : 0u;
  uint32_t qh = 0, qt = 0, qidx = 0;
  double qht = 0.0;
  uint64_t nonempty = 0;  // bit m: model m has queued requests (wave-uniform)

  const double* lbase = sL + (size_t)(cfg < 0 ? 0 : cfg) * SMAX;  // + m * cp * SMAX
  const double facl = 1.0 + a.beta * (double)lane;                // factor of a batch of lane + 1
  double F[SMAX];
#pragma unroll
  for (int s = 0; s < SMAX; ++s) F[s] = 0.0;
  uint64_t fin_sum = 0, finl = 0;  // finish bits of batches (uniform) and of single requests (per lane)
  uint64_t hl = 0;                 // per-lane digest terms
  // indices of batched requests, in lanes below pfill; their terms are
  // computed when no more fit
  uint32_t pidx = 0, pfill = 0;
  int64_t served = 0;
  uint32_t flags = 0;
  const double kInf = __builtin_inf();

  // model mc's queue [.., tl) has its head moved to list position hn.  Every
  // queued request was written to the ring when it joined, so the newest R
  // are there; older ones are read from the arrival lists.
  auto set_head = [&](int mc, uint32_t hn, uint32_t tl) {
    double nt;
    uint32_t ni;
    if (__builtin_expect(tl - hn <= R, 1)) {
      const uint32_t slot = (uint32_t)mc * R + (hn & rmask);
      nt = rt[slot];
      ni = ri[slot];
    } else {
      const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)loff, mc) + hn;
      nt = a.lt[pos];
      ni = a.li[pos];
    }
    const bool own = lane == mc;
    qh = own ? hn : qh;
    qht = own ? nt : qht;
    qidx = own ? ni : qidx;
    nonempty = hn == tl ? nonempty & ~(1ull << mc) : nonempty;
  };

  // the trace, 64 requests per register chunk, the next chunk in flight
  auto load_chunk = [&](int64_t base, double& tv, int& mv, uint32_t& ov) {
    const int64_t i = base + lane;
    tv = i < a.n ? a.t[i] : 0.0;
    mv = i < a.n ? a.model[i] : -1;
    ov = i < a.n ? a.ord[i] : 0u;
  };
  double tv, tvn = 0.0;
  int mv, mvn = -1;
  uint32_t ov, ovn = 0;
  load_chunk(0, tv, mv, ov);

  for (int64_t base = 0; base <= a.n; base += 64) {
    const int cnt = (int)((a.n - base) < 64 ? (a.n - base) : 64);
    if (base + 64 < a.n) load_chunk(base + 64, tvn, mvn, ovn);
    // lane e: request e's model, hosts (none for a model out of range),
    // deadline and digest term
    const bool mok = (unsigned)mv < (unsigned)a.M;
    const int mrow = mok ? mv : 0;
    const auto gather = [&](int v) { return __builtin_amdgcn_ds_bpermute(mrow << 2, v); };
    const uint32_t hlo = (uint32_t)gather((int)(uint32_t)hostm), hhi = (uint32_t)gather((int)(uint32_t)(hostm >> 32));
    const uint64_t hmv = mok ? ((uint64_t)hhi << 32) | hlo : 0ull;
    const double dlv = tv + __hiloint2double(gather(__double2hiint(slo)), gather(__double2loint(slo)));
    const uint64_t mixv = mix64((uint64_t)(base + lane));
    uint64_t okm = 0;  // bit e: request e was served at its arrival
    // cnt requests of this chunk, then (after the last one) the final drain
    const int steps = base + 64 > a.n ? cnt + 1 : cnt;
    for (int e = 0; e < steps; ++e) {
      const bool last = e == cnt;
      const double ti = last ? kInf : rl_f64(tv, e);
      const int m = __builtin_amdgcn_readlane(mrow, e);
      double Lm[SMAX];  // of the request's model on every lane's group
#pragma unroll
      for (int s = 0; s < SMAX; ++s) Lm[s] = lbase[(size_t)m * cp * SMAX + s];
      // idle events up to the arrival (all remaining ones after the last)
      for (;;) {
        const uint64_t evm = __builtin_amdgcn_ballot_w64((hostbits & nonempty) != 0) & __builtin_amdgcn_ballot_w64(F[0] <= ti);
        if (evm == 0) break;
        const double emin = batch_min<W>(__builtin_amdgcn_inverse_ballot_w64(evm) ? F[0] : kInf);
        const int g = __builtin_ctzll(__builtin_amdgcn_ballot_w64(F[0] == emin) & evm);
        const uint64_t ghost = rl_u64(hostbits, g);
        const int gcfg = __builtin_amdgcn_readlane(cfg, g);
        double Fg[SMAX];
#pragma unroll
        for (int s = 0; s < SMAX; ++s) Fg[s] = rl_f64(F[s], g);
        const double mn = Fg[0];
        for (;;) {
          const uint64_t cand = ghost & nonempty;
          if (cand == 0) break;  // nothing left for this group: it stays idle
          // the queued model whose head has the lowest trace index
          const uint32_t hidx = wave_min_u32(__builtin_amdgcn_inverse_ballot_w64(cand) ? qidx : 0xFFFFFFFFu);
          const int mc = __builtin_ctzll(__builtin_amdgcn_ballot_w64(qidx == hidx) & cand);
          const uint32_t h0 = (uint32_t)__builtin_amdgcn_readlane((int)qh, mc);
          const uint32_t tl = (uint32_t)__builtin_amdgcn_readlane((int)qt, mc);
          const double dl = rl_f64(qht + slo, mc);  // the head's deadline
          const uint32_t avail = tl - h0;
          const int bmax = (int)(avail < (uint32_t)a.max_batch ? avail : (uint32_t)a.max_batch);
          // the largest batch meeting the deadline: the sizes are tried 64 at
          // a time, lane l the size p0 + l + 1, and the first size that
          // misses ends the search (as trying them one by one would)
          const double* L = sL + ((size_t)mc * cp + gcfg) * SMAX;
          auto sizes = [&](int p0, double fac, double (&fs)[SMAX]) {  // how many of p0 + 1 .. p0 + 64 meet it
            double f = mn;
#pragma unroll
            for (int s = 0; s < SMAX; ++s) {
              fs[s] = vmax(f, Fg[s]) + L[s] * fac;
              f = fs[s];
            }
            const int lim = bmax - p0;
            const uint64_t stop = __builtin_amdgcn_ballot_w64(f > dl) | (lim < 64 ? ~0ull << lim : 0ull);
            return stop ? __builtin_ctzll(stop) : 64;
          };
          double fs[SMAX], fsel[SMAX];
          int b = sizes(0, facl, fs);
          if (b == 0) {
            // the head cannot meet its deadline: dropped (its output stays -1)
            set_head(mc, h0 + 1, tl);
            continue;
          }
#pragma unroll
          for (int s = 0; s < SMAX; ++s) fsel[s] = rl_f64(fs[s], b - 1);
          if (__builtin_expect(b == 64 && bmax > 64, 0)) {
            for (int p0 = 64; p0 < bmax; p0 += 64) {
              const int nok = sizes(p0, 1.0 + a.beta * (double)(p0 + lane), fs);
              if (nok == 0) break;
              b = p0 + nok;
#pragma unroll
              for (int s = 0; s < SMAX; ++s) fsel[s] = rl_f64(fs[s], nok - 1);
              if (nok < 64) break;
            }
          }
          const double fin = fsel[SMAX - 1];
#pragma unroll
          for (int s = 0; s < SMAX; ++s) F[s] = lane == g ? fsel[s] : F[s];
          // the batch's digest terms
          const uint32_t lb0 = (uint32_t)__builtin_amdgcn_readlane((int)loff, mc) + h0;
          if (__builtin_expect(avail <= R, 1)) {
            if (pfill + (uint32_t)b > 64) {
              hl += (uint32_t)lane < pfill ? mix64(pidx) : 0ull;
              pfill = 0;
            }
            const uint32_t k = (uint32_t)lane - pfill;
            const uint32_t v = ri[(uint32_t)mc * R + ((h0 + k) & rmask)];
            pidx = k < (uint32_t)b ? v : pidx;
            pfill += (uint32_t)b;
          } else {
            for (int k0 = 0; k0 < b; k0 += 64)
              if (k0 + lane < b) hl += a.lmix[lb0 + k0 + lane];
          }
          fin_sum += (uint64_t)b * (uint64_t)__double_as_longlong(fin);
          served += b;
          if (frowp) {
            for (int k0 = 0; k0 < b; k0 += 64)
              if (k0 + lane < b) frowp[a.li[lb0 + k0 + lane]] = fin;
          }
          set_head(mc, h0 + (uint32_t)b, tl);
          break;
        }
      }
      if (last) break;
      // the arrival
      const uint64_t hm = rl_u64(hmv, e);
      if (hm == 0) continue;  // no group hosts it: a miss
      const uint64_t avm = __builtin_amdgcn_ballot_w64(F[0] <= ti) & hm;
      if (avm != 0) {
        // the hosting group that has been idle longest, ties to the lowest
        const double amin = batch_min<W>(__builtin_amdgcn_inverse_ballot_w64(avm) ? F[0] : kInf);
        const uint64_t tie = __builtin_amdgcn_ballot_w64(F[0] == amin) & avm;
        // every lane's chain through its own group (the factor of one request is 1)
        double fs[SMAX];
        double f = ti;
#pragma unroll
        for (int s = 0; s < SMAX; ++s) {
          fs[s] = vmax(f, F[s]) + Lm[s];
          f = fs[s];
        }
        const uint64_t acc = __builtin_amdgcn_ballot_w64(!(f > rl_f64(dlv, e))) & (tie & (0 - tie));
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(acc);
#pragma unroll
        for (int s = 0; s < SMAX; ++s) F[s] = mine ? fs[s] : F[s];
        finl += mine ? (uint64_t)__double_as_longlong(f) : 0ull;
        okm |= (uint64_t)(acc != 0) << e;
        if (frowp) {
          if (mine) frowp[base + e] = f;
        }
      } else {
        // Queue heads of model m that can no longer be served are dropped
        // now rather than when a group reaches them: any batch that could
        // still serve a queued request starts at or after ti, so it finishes
        // no earlier than the chain from ti through a hosting group's stages
        // with single-request latencies, free times ignored (fp64 rounding
        // is monotone); a head whose deadline lies before the smallest such
        // bound is dropped by the definition too, and dropping it earlier
        // changes no other decision.  This keeps each queue to the requests
        // that are still servable.
        const uint32_t rank = (uint32_t)__builtin_amdgcn_readlane((int)ov, e);
        const uint32_t h0 = (uint32_t)__builtin_amdgcn_readlane((int)qh, m);
        const uint32_t tl = (uint32_t)__builtin_amdgcn_readlane((int)qt, m);
        uint32_t hd = h0;
        if (hd != tl) {
          double lbv = ti;
#pragma unroll
          for (int s = 0; s < SMAX; ++s) lbv = lbv + Lm[s];
          const double lb = rl_f64(batch_min<W>(__builtin_amdgcn_inverse_ballot_w64(hm) ? lbv : kInf), 0);
          if (rl_f64(qht + slo, m) < lb) {
            // 64 entries at a time, lane l the one at hd + l; the first that
            // is kept is the new head
            const double slom = rl_f64(slo, m);
            const uint32_t lm = (uint32_t)__builtin_amdgcn_readlane((int)loff, m);
            do {
              const uint32_t left = tl - hd;
              double nt;
              uint32_t ni;
              if (left <= R) {
                const uint32_t slot = (uint32_t)m * R + ((hd + (uint32_t)lane) & rmask);
                nt = rt[slot];
                ni = ri[slot];
              } else {
                const uint32_t pos = lm + hd + std::min((uint32_t)lane, left - 1);
                nt = a.lt[pos];
                ni = a.li[pos];
              }
              const uint64_t keep = __builtin_amdgcn_ballot_w64(!(nt + slom < lb)) & (left < 64 ? ~(~0ull << left) : ~0ull);
              if (keep) {
                const int k = __builtin_ctzll(keep);
                hd += (uint32_t)k;
                const double kt = rl_f64(nt, k);
                const uint32_t ki = (uint32_t)__builtin_amdgcn_readlane((int)ni, k);
                qh = lane == m ? hd : qh;
                qht = lane == m ? kt : qht;
                qidx = lane == m ? ki : qidx;
                break;
              }
              hd += std::min(left, 64u);
            } while (hd != tl);
          }
        }
        const bool own = lane == m;
        const bool first = own && hd == tl;  // an empty queue: request i becomes its head
        qh = first ? rank : qh;
        qht = first ? ti : qht;
        qidx = first ? (uint32_t)(base + e) : qidx;
        if (hd != tl) {
          if (rank != tl) flags |= 2u;  // not the run's next arrival (cannot happen by the rules)
          if (tl - hd >= (uint32_t)a.qcap) flags |= 1u;  // past the capacity: the results are incomplete
        }
        qt = own ? rank + 1 : qt;
        nonempty |= 1ull << m;
        if (R) {  // every lane writes the same words, so every lane may read them
          const uint32_t slot = (uint32_t)m * R + (rank & rmask);
          rt[slot] = ti;
          ri[slot] = (uint32_t)(base + e);
        }
      }
    }
    hl += (okm >> lane) & 1 ? mixv : 0ull;
    served += __builtin_popcountll(okm);
    tv = tvn;
    mv = mvn;
    ov = ovn;
  }
  hl += (uint32_t)lane < pfill ? mix64(pidx) : 0ull;
  const uint64_t hsum = seg_sum_u64<64>(hl);
  const uint64_t fsum = seg_sum_u64<64>(finl);
  if (lane == 0) {
    if (flags) atomicOr(a.flags, flags);
    a.out_served[job] = served;
    if (a.out_digest) {
      a.out_digest[2 * job] = hsum;
      a.out_digest[2 * job + 1] = fin_sum + fsum;
    }
  }
}

// Per-request output rows before a batched launch: -2 for requests whose model
// the job's placement does not host, -1 for the others (served ones are
// overwritten by the kernel).
__global__ void fill_batch_rows(const BatchArgs a) {
  const int64_t total = (int64_t)a.n_finish * a.n;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < total;
       x += (int64_t)gridDim.x * blockDim.x) {
    const int f = (int)(x / a.n);
    const int64_t i = x % a.n;
    const int p = a.finish_jobs[f] / a.K;
    const int32_t m = a.model[i];
    const bool hosted = (unsigned)m < (unsigned)a.M && a.host_mask[(int64_t)p * a.M + m] != 0;
    a.out_finish[x] = hosted ? -1.0 : -2.0;
  }
}

}  // namespace
}  // namespace as_dev

using namespace as_host;

extern "C" int as_simulate_batched(const as_trace_t* trace, const as_models_t* models,
                                   const as_placements_t* placements, const double* slo_scale,
                                   int32_t n_scales, int32_t max_batch, double beta, int32_t queue_cap,
                                   int64_t* out_served, uint64_t* out_digest, const int32_t* finish_jobs,
                                   int32_t n_finish, double* out_finish, void* stream) {
  KArgs ka;
  std::memset(&ka, 0, sizeof ka);
  if (!trace) return fail(AS_E_INVALID_ARG, "trace must not be NULL");
  if (trace->n < 0) return fail(AS_E_INVALID_ARG, "trace n=%lld < 0", (long long)trace->n);
  if (trace->n > 0 && (!trace->t || !trace->model))
    return fail(AS_E_INVALID_ARG, "trace arrays must not be NULL");
  if (trace->n > 0xFFFFFFFFLL) return fail(AS_E_LIMITS, "batched: trace of %lld requests > 2^32 - 1", (long long)trace->n);
  int W = 1, smax = 1;
  int rc = check_common(models, placements, ka, W, smax);
  if (rc != AS_OK) return rc;
  if (n_scales < 0) return fail(AS_E_INVALID_ARG, "n_scales=%d < 0", n_scales);
  if (max_batch < 1) return fail(AS_E_INVALID_ARG, "max_batch=%d < 1", max_batch);
  if (!(beta >= 0.0) || !(beta <= 1.7976931348623157e308))
    return fail(AS_E_INVALID_ARG, "beta must be finite and >= 0");
  if (queue_cap < 1 || (queue_cap & (queue_cap - 1)) != 0 || queue_cap > (1 << 20))
    return fail(AS_E_INVALID_ARG, "queue_cap=%d must be a power of two in 1..2^20", queue_cap);
  const int64_t J = (int64_t)placements->n_placements * n_scales;
  if (J > 0x7FFFFFFFLL) return fail(AS_E_LIMITS, "placements x scales = %lld jobs > 2^31-1", (long long)J);
  if (J > 0 && (!slo_scale || !out_served))
    return fail(AS_E_INVALID_ARG, "slo_scale and out_served must not be NULL");
  if (n_finish < 0 || n_finish > AS_MAX_FINISH)
    return fail(n_finish < 0 ? AS_E_INVALID_ARG : AS_E_LIMITS, "n_finish=%d outside 0..%d", n_finish, AS_MAX_FINISH);
  if (n_finish > 0 && (!finish_jobs || !out_finish))
    return fail(AS_E_INVALID_ARG, "finish_jobs and out_finish must not be NULL when n_finish > 0");
  as_dev::BatchArgs a;
  std::memset(&a, 0, sizeof a);
  for (int f = 0; f < n_finish; ++f) {
    if (finish_jobs[f] < 0 || finish_jobs[f] >= J)
      return fail(AS_E_INVALID_ARG, "finish_jobs[%d]=%d outside [0, %lld)", f, finish_jobs[f], (long long)J);
    for (int q = 0; q < f; ++q)
      if (finish_jobs[q] == finish_jobs[f]) return fail(AS_E_INVALID_ARG, "finish_jobs[%d] repeats job %d", f, finish_jobs[f]);
    a.finish_jobs[f] = finish_jobs[f];
  }
  const int cp = pow2ceil(ka.C);
  const size_t table = as_dev::batch_lds_bytes(ka.M, cp, smax, 0);
  if (table > shared_lds_limit())
    return fail(AS_E_LIMITS, "batched: the stage-latency table needs %zu bytes of LDS (> %zu)", table,
                shared_lds_limit());
  // Entries of each model's LDS ring: 32, 16 or 8, as many as leave all jobs
  // resident (up to the 32 wavefronts a compute unit holds), else none: a queue
  // longer than its ring reads the lists, an L2 access instead of an LDS one,
  // which costs less than a job that waits for another's place.  64 models, 8000
  // requests, no ring and 8 entries: 4096 jobs and a 16 KiB table 12.7 and 15.7
  // ms, 8192 jobs and a 2 KiB table 17.1 and 19.4; 1024 jobs, where both fit, 6.3
  // and 6.0.
  const int64_t cus = compute_units(), per_cu = std::min<int64_t>((J + cus - 1) / cus, 32);
  auto halve = [](int r) { return r > 8 ? r / 2 : 0; };
  int ring = 32;
  while (ring > 0 && as_dev::batch_lds_bytes(ka.M, cp, smax, ring) * per_cu > 160 * 1024) ring = halve(ring);
  while (ring > 0 && as_dev::batch_lds_bytes(ka.M, cp, smax, ring) > shared_lds_limit()) ring = halve(ring);
  const size_t lds = as_dev::batch_lds_bytes(ka.M, cp, smax, ring);
  if (J == 0) return ok();
  hipStream_t s = (hipStream_t)stream;
  a.t = trace->t;
  a.model = trace->model;
  a.n = trace->n;
  a.d_single = ka.d_single;
  a.stage_lat = ka.stage_lat;
  a.group_cfg = ka.group_cfg;
  a.host_mask = ka.host_mask;
  a.slo_scale = slo_scale;
  a.out_served = out_served;
  a.out_digest = out_digest;
  a.out_finish = out_finish;
  a.beta = beta;
  a.M = ka.M;
  a.C = ka.C;
  a.smax_in = ka.smax_in;
  a.G = ka.G;
  a.K = n_scales;
  a.J = (int32_t)J;
  a.max_batch = max_batch;
  a.qcap = queue_cap;
  a.ring = ring;
  a.n_finish = n_finish;
  for (int c = 0; c < AS_MAX_CONFIGS; ++c) a.cfg_stages[c] = ka.cfg_stages[c];
  // one workspace: the flags word, then the per-model arrival lists
  as_dev::ListArgs la;
  std::memset(&la, 0, sizeof la);
  la.t = trace->t;
  la.model = trace->model;
  la.n = trace->n;
  la.M = ka.M;
  la.nblk = (trace->n + as_dev::kListBlock - 1) / as_dev::kListBlock;
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t n = (size_t)trace->n;
  const size_t o_blk = 256, o_off = o_blk + up((size_t)la.nblk * ka.M * 4), o_ord = o_off + up((size_t)(ka.M + 1) * 4),
               o_lt = o_ord + up(n * 4), o_li = o_lt + up(n * 8), o_mix = o_li + up(n * 4), total = o_mix + up(n * 8);
  unsigned char* ws = nullptr;
  hipError_t e = pool_alloc(reinterpret_cast<void**>(&ws), total, s);
  if (e != hipSuccess) return fail(AS_E_NOMEM, "device allocation of %zu bytes: %s", total, hipGetErrorString(e));
  a.flags = reinterpret_cast<uint32_t*>(ws);
  la.flags = a.flags;
  la.blk = reinterpret_cast<uint32_t*>(ws + o_blk);
  la.off = reinterpret_cast<uint32_t*>(ws + o_off);
  la.ord = reinterpret_cast<uint32_t*>(ws + o_ord);
  la.lt = reinterpret_cast<double*>(ws + o_lt);
  la.li = reinterpret_cast<uint32_t*>(ws + o_li);
  la.lmix = reinterpret_cast<uint64_t*>(ws + o_mix);
  a.off = la.off;
  a.ord = la.ord;
  a.lt = la.lt;
  a.li = la.li;
  a.lmix = la.lmix;
  if (la.nblk > 0) hipLaunchKernelGGL(as_dev::list_count, dim3((unsigned)la.nblk), dim3(64), 0, s, la);
  hipLaunchKernelGGL(as_dev::list_scan, dim3(1), dim3(64), 0, s, la);  // also clears the flags
  if (la.nblk > 0) hipLaunchKernelGGL(as_dev::list_fill, dim3((unsigned)la.nblk), dim3(64), 0, s, la);
  e = hipGetLastError();
  if (e == hipSuccess && n_finish > 0 && a.n > 0) {
    const int64_t cells = (int64_t)n_finish * a.n;
    const int blocks = (int)std::min<int64_t>((cells + 255) / 256, 8192);
    hipLaunchKernelGGL(as_dev::fill_batch_rows, dim3(blocks), dim3(256), 0, s, a);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    const int W = std::max(16, pow2ceil(a.G));
    const dim3 grid((unsigned)J), block(64);
#define AS_BATCH_LAUNCH(WW)                                                                         \
  switch (smax) {                                                                                   \
    case 1: hipLaunchKernelGGL((as_dev::batch_kernel<WW, 1>), grid, block, lds, s, a); break;       \
    case 2: hipLaunchKernelGGL((as_dev::batch_kernel<WW, 2>), grid, block, lds, s, a); break;       \
    case 4: hipLaunchKernelGGL((as_dev::batch_kernel<WW, 4>), grid, block, lds, s, a); break;       \
    default: hipLaunchKernelGGL((as_dev::batch_kernel<WW, 8>), grid, block, lds, s, a); break;      \
  }
    if (W == 16) {
      AS_BATCH_LAUNCH(16)
    } else if (W == 32) {
      AS_BATCH_LAUNCH(32)
    } else {
      AS_BATCH_LAUNCH(64)
    }
#undef AS_BATCH_LAUNCH
    e = hipGetLastError();
  }
  uint32_t flag = 0;
  if (e == hipSuccess) e = hipMemcpyAsync(&flag, a.flags, sizeof flag, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  const hipError_t ef = hipFreeAsync(ws, s);
  if (e == hipSuccess) e = ef;
  if (e != hipSuccess) return fail(AS_E_HIP, "batched: %s", hipGetErrorString(e));
  if (flag & 2u)
    return fail(AS_E_INVALID_DATA, "batched: a queue was not a run of its model's arrivals; results are invalid");
  if (flag & 1u) return fail(AS_E_LIMITS, "batched: a model queue exceeded queue_cap=%d; results are incomplete", queue_cap);
  return ok();
}
