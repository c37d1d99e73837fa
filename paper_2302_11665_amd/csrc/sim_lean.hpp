// Group-per-lane serving-simulator kernels for gfx950: shared traces (several
// jobs per wavefront) and jobs with trace segments of their own (one job per
// wavefront).
//
// Layout: a job owns W lanes of a wavefront, lane r of the job holds group r's
// stage free times F[0..SMAX-1] in registers.  Each wavefront stages its own
// requests through LDS, 64 at a time; there is no workgroup barrier in the
// request loop.
//
// What bounds it: a request depends on the state that the one before it left,
// so a job's time is (requests) x (instructions of one request), and a lone
// wavefront of a SIMD issues one instruction of any kind every 4 to 5.5 cycles
// and loses about 28 on a branch that is not taken, 40 on one that is.  Hence:
//   * requests that no job of the wavefront can host are left out when a chunk
//     is staged (they change no state and are misses);
//   * a request is straight-line code: no branch on whether a dispatch minimum
//     is needed, on ties or on admission.  The minimum is a binary64 one over
//     the job's lanes (lanes that do not host are NaN, which v_min_f64 passes
//     over); near and exact ties are common, because bursty arrivals lie
//     closer together than any shorter key resolves, and the lowest of equal
//     lanes is found by masking the equality's ballot with the lanes below;
//   * dispatch, tie and admission narrow the exec mask (v_cmpx) and the commit
//     is plain moves under it, with no selects.
// Measured, nanoseconds per request of a lone wavefront, before (records,
// branches on ties and single hosts, selects) and now: 16 lanes per job and 4
// stages 154 and 91, 4 lanes and 4 stages 151 and 79, 64 lanes and 1 stage 156
// and 104, 64 lanes and 4 stages 181 and 118.  With two wavefronts on every
// SIMD the first takes 141 (was 185).  With eight the vector instructions count,
// which is why a wavefront of one job ends its minimum in a lane read and breaks
// ties on the scalar unit: 64 lanes and 1 stage, 8192 jobs of 3000 requests,
// take 1.44 ms with that, 1.72 with swaps and vector masks, 1.66 with the
// branches; 6000 jobs of 20,000 requests of their own 6.8, 8.2 and 6.7 ms.
//
// Exactness: v_max_f64, single v_add_f64, no FMA, in the definition's order,
// so finish times are bit-identical to a sequential IEEE evaluation.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alpaserve_sim.h"
#include "sim_kernel.hpp"
#include "sim_shared.hpp"

namespace as_dev {

constexpr int kLeanB = 8;  // requests per batch: their LDS reads are issued together

// A staged request: {t, deadline}, {hosting lanes (u64), L[0] or, where the
// lanes differ in configuration, the latency table's row offset}, L[1..].
// The stride keeps the 64 lanes' 16-byte writes free of bank conflicts.
__host__ __device__ constexpr int lean_stride(int SMAX) { return SMAX <= 2 ? 48 : SMAX == 4 ? 80 : 112; }
// LDS bytes of one wavefront: 64 staged requests, padded to whole batches.
__host__ __device__ constexpr size_t lean_wave_bytes(int SMAX) { return (size_t)(64 + kLeanB) * lean_stride(SMAX); }

template <int SMAX>
struct LeanLane {
  double F[SMAX];
  uint64_t fin;  // bit patterns of this group's accepted finish times, summed
  double busy;   // statistics: this group's busy time
  double sigma;  // MS: this job's SLO scale
};

// Dispatch and admission on the exec mask, then the commit under it: lanes
// whose key equals their job's minimum; of those the lowest of each job (blo,
// bhi: this lane's job's lanes below it); of those the ones that meet the
// deadline take the projected state.  Lane and DPP reads of
// vector registers written here, and of lanes after the exec mask's vector
// writes, are at least four instructions away.
#define AS_LEAN_TAIL                             \
  "v_cmpx_ngt_f64_e32 vcc, %[f], %[dl]\n\t"      \
  "v_mov_b64_e32 %[F0], %[f0]\n\t"
#define AS_LEAN_SUMS                             \
  "v_lshl_add_u64 %[fin], %[f], 0, %[fin]\n\t"   \
  "v_or_b32_e32 %[sr], %[bit], %[sr]\n\t"
#define AS_LEAN_END "s_mov_b64 exec, -1"
#define AS_LEAN_END1 "s_mov_b64 exec, -1\n\ts_nop 0"  // one stage: the fifth instruction
#define AS_LEAN_OUT AS_LEAN_TMP, [fin] "+v"(st.fin), [sr] "+v"(sr), [F0] "+v"(st.F[0])
#define AS_LEAN_IN AS_LEAN_SEL, [key] "v"(key), [f] "v"(f), [dl] "v"(dl), [f0] "v"(fs[0]), [bit] "i"(1 << BIT)
#define AS_LEAN_ASM(MOVS, OUTS, INS, END)                                                                     \
  if constexpr (STATS)                                                                                        \
    asm(AS_LEAN_HEAD AS_LEAN_TAIL MOVS AS_LEAN_SUMS "v_add_f64 %[busy], %[busy], %[slow]\n\t" END             \
        : AS_LEAN_OUT OUTS, [busy] "+v"(st.busy)                                                              \
        : AS_LEAN_IN INS, [slow] "v"(slow)                                                                    \
        : AS_LEAN_CLOBBERS);                                                                                  \
  else if constexpr (ROW)                                                                                     \
    asm volatile(AS_LEAN_HEAD AS_LEAN_TAIL MOVS AS_LEAN_SUMS "ds_write_b64 %[orow], %[f] offset:%[at]\n\t" END \
                 : AS_LEAN_OUT OUTS                                                                           \
                 : AS_LEAN_IN INS, [orow] "v"(orow), [at] "i"(8 * BIT)                                        \
                 : AS_LEAN_CLOBBERS, "memory");                                                               \
  else                                                                                                        \
    asm(AS_LEAN_HEAD AS_LEAN_TAIL MOVS AS_LEAN_SUMS END : AS_LEAN_OUT OUTS : AS_LEAN_IN INS : AS_LEAN_CLOBBERS)
#define AS_COMMA ,
#define AS_LEAN_STAGES                                                                                          \
  if constexpr (SMAX == 1) {                                                                                    \
    AS_LEAN_ASM("", , , AS_LEAN_END1);                                                                          \
  } else if constexpr (SMAX == 2) {                                                                             \
    AS_LEAN_ASM("v_mov_b64_e32 %[F1], %[f1]\n\t", AS_COMMA[F1] "+v"(st.F[1]), AS_COMMA[f1] "v"(fs[1]),          \
                AS_LEAN_END);                                                                                   \
  } else if constexpr (SMAX == 4) {                                                                             \
    AS_LEAN_ASM("v_mov_b64_e32 %[F1], %[f1]\n\tv_mov_b64_e32 %[F2], %[f2]\n\tv_mov_b64_e32 %[F3], %[f3]\n\t", \
                AS_COMMA[F1] "+v"(st.F[1]) AS_COMMA[F2] "+v"(st.F[2]) AS_COMMA[F3] "+v"(st.F[3]),               \
                AS_COMMA[f1] "v"(fs[1]) AS_COMMA[f2] "v"(fs[2]) AS_COMMA[f3] "v"(fs[3]), AS_LEAN_END);          \
  } else {                                                                                                      \
    AS_LEAN_ASM("v_mov_b64_e32 %[F1], %[f1]\n\tv_mov_b64_e32 %[F2], %[f2]\n\tv_mov_b64_e32 %[F3], %[f3]\n\t"  \
                "v_mov_b64_e32 %[F4], %[f4]\n\tv_mov_b64_e32 %[F5], %[f5]\n\tv_mov_b64_e32 %[F6], %[f6]\n\t"  \
                "v_mov_b64_e32 %[F7], %[f7]\n\t",                                                               \
                AS_COMMA[F1] "+v"(st.F[1]) AS_COMMA[F2] "+v"(st.F[2]) AS_COMMA[F3] "+v"(st.F[3])                \
                    AS_COMMA[F4] "+v"(st.F[4]) AS_COMMA[F5] "+v"(st.F[5]) AS_COMMA[F6] "+v"(st.F[6])            \
                        AS_COMMA[F7] "+v"(st.F[7]),                                                             \
                AS_COMMA[f1] "v"(fs[1]) AS_COMMA[f2] "v"(fs[2]) AS_COMMA[f3] "v"(fs[3]) AS_COMMA[f4] "v"(fs[4]) \
                    AS_COMMA[f5] "v"(fs[5]) AS_COMMA[f6] "v"(fs[6]) AS_COMMA[f7] "v"(fs[7]),                    \
                AS_LEAN_END);                                                                                   \
  }

#define AS_LEAN_HEAD                             \
  "v_cmpx_eq_f64_e32 vcc, %[mn], %[key]\n\t"     \
  "s_nop 1\n\t"                                  \
  "v_and_b32_e32 %[x], vcc_lo, %[blo]\n\t"       \
  "v_and_or_b32 %[x], vcc_hi, %[bhi], %[x]\n\t"  \
  "v_cmpx_eq_u32_e32 vcc, 0, %[x]\n\t"
#define AS_LEAN_TMP [x] "=&v"(x)
#define AS_LEAN_SEL [mn] "v"(mn), [blo] "v"(blo), [bhi] "v"(bhi)
#define AS_LEAN_CLOBBERS "vcc"
// orow: LDS address where ROW stores the accepting lane's finish time, 8 bytes
// per request of the batch.
template <int SMAX, int BIT, bool STATS, bool ROW>
__device__ __forceinline__ void lean_commit(LeanLane<SMAX>& st, double mn, double key, uint32_t blo, uint32_t bhi,
                                            const double (&fs)[SMAX], double dl, double slow, uint32_t& sr,
                                            uint32_t orow) {
  static_assert(!(STATS && ROW), "statistics launches carry no rows");
  uint32_t x;
  const double f = fs[SMAX - 1];
  AS_LEAN_STAGES
}
#undef AS_LEAN_HEAD
#undef AS_LEAN_TMP
#undef AS_LEAN_SEL
#undef AS_LEAN_CLOBBERS

// One job in the wavefront: the minimum is uniform and the lowest of the equal
// lanes a scalar bit search (none equal: no lane), which leaves the vector unit
// to the other wavefronts of the SIMD.
#define AS_LEAN_HEAD                             \
  "s_nop 1\n\t"                                  \
  "v_cmp_eq_f64_e32 vcc, %[mn], %[key]\n\t"      \
  "s_ff1_i32_b64 %[i], vcc\n\t"                  \
  "s_lshl_b64 %[m], 1, %[i]\n\t"                 \
  "s_and_b64 exec, vcc, %[m]\n\t"
#define AS_LEAN_TMP [i] "=&s"(i), [m] "=&s"(m)
#define AS_LEAN_SEL [mn] "s"(mn)
#define AS_LEAN_CLOBBERS "vcc", "scc"
template <int SMAX, int BIT, bool STATS, bool ROW>
__device__ __forceinline__ void lean_commit_one(LeanLane<SMAX>& st, double mn, double key, const double (&fs)[SMAX],
                                                double dl, double slow, uint32_t& sr, uint32_t orow) {
  uint32_t i;
  uint64_t m;
  const double f = fs[SMAX - 1];
  AS_LEAN_STAGES
}
#undef AS_LEAN_HEAD
#undef AS_LEAN_TMP
#undef AS_LEAN_SEL
#undef AS_LEAN_CLOBBERS
#undef AS_LEAN_STAGES
#undef AS_LEAN_ASM
#undef AS_COMMA
#undef AS_LEAN_TAIL
#undef AS_LEAN_SUMS
#undef AS_LEAN_END
#undef AS_LEAN_END1
#undef AS_LEAN_OUT
#undef AS_LEAN_IN

// Inputs of one staged request.
template <int SMAX>
struct LeanReq {
  double t, dl;
  uint64_t hm;     // as read: the same in every lane
  double L[SMAX];  // this lane's stage latencies
};

template <int SMAX, bool UNI>
__device__ __forceinline__ LeanReq<SMAX> lean_read(const unsigned char* r, const char* lrow) {
  LeanReq<SMAX> q;
  const double2 td = *(const double2*)r;
  q.t = td.x;
  q.dl = td.y;
  if constexpr (UNI) {
    const ulonglong2 h = *(const ulonglong2*)(r + 16);
    q.hm = h.x;
    q.L[0] = __longlong_as_double((long long)h.y);
    if constexpr (SMAX == 2) q.L[1] = *(const double*)(r + 32);
#pragma unroll
    for (int s = 1; s + 1 < SMAX; s += 2) {
      const double2 l2 = *(const double2*)(r + 24 + 8 * s);
      q.L[s] = l2.x;
      q.L[s + 1] = l2.y;
    }
    if constexpr (SMAX >= 4) q.L[SMAX - 1] = *(const double*)(r + 24 + 8 * (SMAX - 1));
  } else {
    const uint4 h = *(const uint4*)(r + 16);
    q.hm = ((uint64_t)h.y << 32) | h.x;
    const char* l = lrow + h.z;
    if constexpr (SMAX == 1) {
      q.L[0] = *(const double*)l;
    } else {
#pragma unroll
      for (int s = 0; s < SMAX; s += 2) {
        const double2 l2 = *(const double2*)(l + 8 * s);
        q.L[s] = l2.x;
        q.L[s + 1] = l2.y;
      }
    }
  }
  return q;
}

__device__ __forceinline__ uint64_t lean_uniform(uint64_t x) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

template <int SMAX>
__device__ __forceinline__ double lean_slow(const double (&L)[SMAX]) {
  double m = L[0];
#pragma unroll
  for (int s = 1; s < SMAX; ++s) m = vmax(m, L[s]);
  return m;
}

// Minimum over each aligned group of W lanes, in every lane of it (W = 64: a
// scalar); NaN lanes are passed over.
template <int W>
__device__ __forceinline__ double lean_min(double v) {
  if constexpr (W >= 2) v = vmin(v, dpp_f64<kXor1>(v));
  if constexpr (W >= 4) v = vmin(v, dpp_f64<kXor2>(v));
  if constexpr (W >= 8) v = vmin(v, dpp_f64<kHalfMirror>(v));
  if constexpr (W >= 16) v = vmin(v, dpp_f64<kMirror>(v));
  if constexpr (W == 32) {
    const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = vmin(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
  }
  if constexpr (W == 64) {
    // the rows' minima meet in the last row (what the broadcasts bring to rows
    // without a source does not reach it)
    v = vmin(v, dpp_f64<kBcast15>(v));
    v = vmin(v, dpp_f64<kBcast31>(v));
    v = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                         __builtin_amdgcn_readlane(__double2loint(v), 63));
  }
  return v;
}

// MS: the jobs of the wavefront differ in scale, and q.dl is the model's
// d_single (two more instructions a request).
template <int W, int SMAX, int BIT, bool STATS, bool ROW, bool MS>
__device__ __forceinline__ void lean_step(LeanLane<SMAX>& st, const LeanReq<SMAX>& q, uint32_t blo, uint32_t bhi,
                                          uint32_t& sr, uint32_t orow) {
  const bool host = __builtin_amdgcn_inverse_ballot_w64(lean_uniform(q.hm));
  const double key = __hiloint2double(host ? __double2hiint(st.F[0]) : 0x7ff80000, __double2loint(st.F[0]));
  const double mn = lean_min<W>(key);
  double fs[SMAX], f = q.t;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) f = fs[s] = vmax(f, st.F[s]) + q.L[s];
  const double slow = STATS ? lean_slow<SMAX>(q.L) : 0.0;
  const double dl = MS ? q.t + st.sigma * q.dl : q.dl;
  if constexpr (W == 64)
    lean_commit_one<SMAX, BIT, STATS, ROW>(st, mn, key, fs, dl, slow, sr, orow);
  else
    lean_commit<SMAX, BIT, STATS, ROW>(st, mn, key, blo, bhi, fs, dl, slow, sr, orow);
}

template <int W, int SMAX, bool STATS, bool ROW, bool MS, int K, int N, int AT = 0>
__device__ __forceinline__ void lean_steps(LeanLane<SMAX>& st, const LeanReq<SMAX> (&q)[N], uint32_t blo,
                                           uint32_t bhi, uint32_t& sr, uint32_t orow) {
  if constexpr (AT < N) {
    lean_step<W, SMAX, K + AT, STATS, ROW, MS>(st, q[AT], blo, bhi, sr, orow);
    lean_steps<W, SMAX, STATS, ROW, MS, K, N, AT + 1>(st, q, blo, bhi, sr, orow);
  }
}

// kLeanB staged requests.  Returns their accept bits (bit k: request k was
// accepted by this lane).  A wavefront that writes a row beside its results reads
// them by halves at 2 and 4 stages: all at once, its registers (134 and 170, not
// 124 and 160) would take a wavefront from every SIMD, also without rows (16,384
// jobs of 16 four-stage groups: 5.4 ms instead of 5.2).  So does one with the
// statistics of 33 to 64 groups of differing depths: with all eight requests in
// registers the compiler leaves the chain behind the minimum instead of between
// its steps (2 and 4 stages, 15,000 requests: 2.05 and 2.34 ms, 1.83 and 1.99 by
// halves; elsewhere halves are up to 4 % slower or the same).
template <int W, int SMAX, bool UNI, bool STATS, int ROW, bool MS>
__device__ __forceinline__ uint32_t lean_batch(LeanLane<SMAX>& st, const unsigned char* r, const char* lrow,
                                               uint32_t blo, uint32_t bhi, uint32_t orow) {
  constexpr bool kHalves = ROW == 1 || (STATS && W == 64 && !UNI);
  constexpr int N = kHalves && (SMAX == 2 || SMAX == 4) ? kLeanB / 2 : kLeanB;
  uint32_t sr = 0;
  {
    LeanReq<SMAX> q[N];
#pragma unroll
    for (int k = 0; k < N; ++k) q[k] = lean_read<SMAX, UNI>(r + k * lean_stride(SMAX), lrow);
    lean_steps<W, SMAX, STATS, ROW != 0, MS, 0>(st, q, blo, bhi, sr, orow);
  }
  if constexpr (N < kLeanB) {
    LeanReq<SMAX> q[N];
#pragma unroll
    for (int k = 0; k < N; ++k) q[k] = lean_read<SMAX, UNI>(r + (N + k) * lean_stride(SMAX), lrow);
    lean_steps<W, SMAX, STATS, ROW != 0, MS, N>(st, q, blo, bhi, sr, orow);
  }
  return sr;
}

// Order LDS writes of some lanes of the wavefront before reads of others.
__device__ __forceinline__ void lean_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What one wavefront simulates: jw <= 64 / W jobs of one trace (every member but
// cfg, hm and, with MS, sigma is the same in all lanes).
struct LeanIn {
  const double* t;
  const int32_t* model;
  int64_t n;
  int jw;
  double sigma;
  int cfg;      // this lane's group's configuration, -1: no group
  uint64_t hm;  // lane m: lanes whose group hosts model m
  double* row;  // ROW: per-request output of the job in slot row_slot (0 for 2)
  int64_t row_n;
  int row_slot;
  bool digest;  // the ordered hash is wanted
};

struct LeanOut {
  int64_t served;  // this lane's job's
  uint64_t hash;
  uint64_t fin_sum;
  double busy;  // this lane's group's
};

// What a wavefront keeps for all its chunks.
template <int W, int SMAX>
struct LeanWave {
  const char* lrow;  // this lane's configuration's latency row of model 0 (LDS)
  const char* urow;  // the first group's (UNI: every group's)
  int lshift;        // a model's rows are 1 << lshift bytes apart
  unsigned char* rec;  // lean_wave_bytes of LDS, then finish times by rank (ROW)
  uint64_t row_lanes;  // ROW: the lanes of the job whose row is written
  double slo;          // lane m: model m's SLO (MS: its d_single)
  uint64_t hm;         // lane m: lanes whose group hosts model m
  uint64_t hosted;     // models some job hosts
  uint32_t blo, bhi;   // this lane's job's lanes below it
};

// sL: stage-latency table [M][Cp][SMAX] in LDS; cfg: this lane's group's
// configuration, -1: no group.
template <int W, int SMAX, bool MS = false, class Args>
__device__ __forceinline__ LeanWave<W, SMAX> lean_wave(const Args& a, double sigma, int cfg, uint64_t hm,
                                                       const double* sL, int lshift, unsigned char* rec) {
  LeanWave<W, SMAX> w;
  const int lane = threadIdx.x & 63;
  const uint64_t valid = __builtin_amdgcn_ballot_w64(cfg >= 0);
  const int c = cfg < 0 ? 0 : cfg;
  w.lrow = reinterpret_cast<const char*>(sL + c * SMAX);
  w.urow = reinterpret_cast<const char*>(
      sL + (valid ? __builtin_amdgcn_readlane(c, __builtin_ctzll(valid)) : 0) * SMAX);
  w.lshift = lshift;
  w.rec = rec;
  w.slo = lane < a.M ? (MS ? a.d_single[lane] : sigma * a.d_single[lane]) : 0.0;
  w.hm = hm;
  w.hosted = __builtin_amdgcn_ballot_w64(hm != 0);
  const uint64_t below = ((1ull << lane) - 1) & ~((1ull << (lane / W * W)) - 1);
  w.blo = (uint32_t)below;
  w.bhi = (uint32_t)(below >> 32);
  return w;
}

// One configuration for every group of the wavefront?
__device__ __forceinline__ bool lean_uni(int cfg) {
  const uint64_t valid = __builtin_amdgcn_ballot_w64(cfg >= 0);
  const int cfg0 = valid ? __builtin_amdgcn_readlane(cfg, __builtin_ctzll(valid)) : 0;
  return __builtin_amdgcn_ballot_w64(cfg >= 0 && cfg != cfg0) == 0;
}

// One chunk: lane e holds request e (mine: it exists and some job hosts it;
// rank: hosted requests before it).  Returns the job's accept bits in all its
// lanes, the request of rank k at bit k.  ROW: the row's job's finish times (-1:
// rejected, -2: it does not host the model) by rank are left behind the staged
// requests, and the other jobs' lanes store theirs past them; 2: the row alone of
// a wavefront's only job, 1: beside all results.  Called by whole wavefronts in
// uniform control flow (the commit restores a full exec mask).
template <int W, int SMAX, bool UNI, bool STATS, int ROW, bool MS = false>
__device__ __forceinline__ uint64_t lean_chunk(LeanLane<SMAX>& st, const LeanWave<W, SMAX>& w, double tv, int mv,
                                               bool mine, int rank, int nh) {
  constexpr int R = lean_stride(SMAX);
  if (nh == 0) return 0;
  const int lane = threadIdx.x & 63;
  uint64_t word = 0;  // this lane's accept bits
  double* orow = reinterpret_cast<double*>(w.rec + (64 + kLeanB) * R);
  uint32_t olds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) double*)orow;
  if constexpr (ROW == 1) olds += __builtin_amdgcn_inverse_ballot_w64(w.row_lanes) ? 0 : (64 + kLeanB) * 8;
  // stage the hosted requests, then requests that no lane hosts up to a
  // whole batch
  const int from = (mv & 63) << 2;
  const double ms = __hiloint2double(__builtin_amdgcn_ds_bpermute(from, __double2hiint(w.slo)),
                                     __builtin_amdgcn_ds_bpermute(from, __double2loint(w.slo)));
  const uint32_t hl = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)w.hm);
  const uint32_t hh = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)(w.hm >> 32));
  lean_fence();
  if (mine) {
    unsigned char* r = w.rec + rank * R;
    *(double2*)r = make_double2(tv, MS ? ms : tv + ms);  // the deadline t + SLO, each rounded once
    const uint32_t off = (uint32_t)mv << w.lshift;
    if constexpr (UNI) {
      const double* l = reinterpret_cast<const double*>(w.urow + off);
      ulonglong2 h;
      h.x = ((uint64_t)hh << 32) | hl;
      h.y = (uint64_t)__double_as_longlong(l[0]);
      *(ulonglong2*)(r + 16) = h;
#pragma unroll
      for (int s = 1; s < SMAX; ++s) *(double*)(r + 24 + 8 * s) = l[s];
    } else {
      *(uint4*)(r + 16) = make_uint4(hl, hh, off, 0u);
    }
    if constexpr (ROW == 1) orow[rank] = (((uint64_t)hh << 32 | hl) & w.row_lanes) != 0 ? -1.0 : -2.0;
  }
  if (lane < kLeanB) {
    unsigned char* r = w.rec + (nh + lane) * R;
    *(double2*)r = make_double2(0.0, 0.0);
    *(uint4*)(r + 16) = make_uint4(0u, 0u, 0u, 0u);
  }
  if constexpr (ROW == 2) orow[lane] = -1.0;
  lean_fence();
  const int nb = (nh + kLeanB - 1) / kLeanB;
  for (int b = 0; b < nb; ++b) {
    const uint32_t bits = lean_batch<W, SMAX, UNI, STATS, ROW, MS>(st, w.rec + b * kLeanB * R, w.lrow, w.blo, w.bhi,
                                                               olds + b * kLeanB * 8);
    word |= (uint64_t)bits << (b * kLeanB);
  }
  return seg_or<W>(word);
}

// Whether the request in this lane is one to simulate, how many there are
// (nh) and how many come before it (rank).
template <int W, int SMAX>
__device__ __forceinline__ bool lean_mine(const LeanWave<W, SMAX>& w, bool in, int mv, int& rank, int& nh) {
  const bool mine = in && (unsigned)mv < 64u && ((w.hosted >> (mv & 63)) & 1u);
  const uint64_t todo = __builtin_amdgcn_ballot_w64(mine);
  nh = (int)__builtin_popcountll(todo);
  rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(todo >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)todo, 0u));
  return mine;
}

// cnt: STATS, this wavefront's [jw][M] served counters in LDS, zeroed.
template <int W, int SMAX, bool UNI, bool STATS, int ROW, bool MS>
__device__ __forceinline__ LeanOut lean_run(const KArgs& a, const LeanIn& in, const double* sL, int lshift,
                                            unsigned char* rec, uint32_t* cnt) {
  const int lane = threadIdx.x & 63;
  LeanWave<W, SMAX> w = lean_wave<W, SMAX, MS>(a, in.sigma, in.cfg, in.hm, sL, lshift, rec);
  if constexpr (ROW == 1) w.row_lanes = (W == 64 ? ~0ull : ((1ull << (W & 63)) - 1)) << (in.row_slot * (W & 63));
  LeanLane<SMAX> st;
#pragma unroll
  for (int s = 0; s < SMAX; ++s) st.F[s] = 0.0;
  st.fin = 0;
  st.busy = 0.0;
  st.sigma = in.sigma;
  uint64_t hash = 0;
  int64_t served = 0;
  const int64_t n = in.n, top = n > 0 ? n - 1 : 0;
  if (n <= 0) return LeanOut{0, 0, 0, 0.0};

  double tn = in.t[lane < n ? lane : top];
  int mn = in.model[lane < n ? lane : top];
  for (int64_t base = 0; base < n; base += 64) {
    const double tv = tn;
    const int mv = mn;
    const int64_t ahead = base + 64 + lane;
    tn = in.t[ahead < n ? ahead : top];
    mn = in.model[ahead < n ? ahead : top];
    int rank, nh;
    const bool mine = lean_mine<W, SMAX>(w, base + lane < n, mv, rank, nh);
    uint64_t word = lean_chunk<W, SMAX, UNI, STATS, ROW, MS>(st, w, tv, mv, mine, rank, nh);
    served += __builtin_popcountll(word);
    if (STATS || (in.digest && nh < 64)) {
      // back to trace order: lane e is request e, whose bit is at its rank
      uint64_t full = word;
#pragma unroll 1
      for (int j = 0; j < in.jw; ++j) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, j * W);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(word >> 32), j * W);
        const bool bit = mine && (((((uint64_t)hi << 32) | lo) >> rank) & 1u);
        const uint64_t wj = __builtin_amdgcn_ballot_w64(bit);
        full = lane / W == j ? wj : full;
        if constexpr (STATS) {
          if (bit) atomicAdd(cnt + j * a.M + (mv & 63), 1u);
        }
      }
      word = full;
    }
    if (in.digest) hash = (hash ^ word) * kHashMul;
    if constexpr (ROW != 0) {
      lean_fence();
      const double* orow = reinterpret_cast<const double*>(rec + (64 + kLeanB) * lean_stride(SMAX));
      if (lane < (int)(in.row_n - base < 64 ? in.row_n - base : 64)) (in.row + base)[lane] = mine ? orow[rank] : -2.0;
    }
  }
  return LeanOut{served, hash, seg_sum_u64<W>(st.fin), st.busy};
}

// LDS bytes of a workgroup of `waves` wavefronts: the stage-latency table,
// each wavefront's staged requests, and for statistics its counters, else its
// row (twice: once for what the other jobs' lanes store).
__host__ __device__ constexpr size_t lean_wave_lds(int W, int M, int SMAX, bool stats) {
  return lean_wave_bytes(SMAX) + (stats ? ((size_t)(64 / W) * M * 4 + 15) / 16 * 16 : (size_t)2 * (64 + kLeanB) * 8);
}
__host__ __device__ constexpr size_t lean_lds_bytes(int W, int M, int Cp, int SMAX, bool stats, int waves) {
  return ((size_t)M * Cp * SMAX * 8 + 15) / 16 * 16 + (size_t)waves * lean_wave_lds(W, M, SMAX, stats);
}

// The stage-latency table padded with zero-latency stages (sim_kernel.hpp);
// returns log2 of a model's row stride in bytes and the table's bytes.
template <int SMAX, class Args>
__device__ __forceinline__ int lean_table(const Args& a, double* sL, size_t& bytes) {
  int cp = 1, lshift = 0;
  while (cp < a.C) cp <<= 1;
  while ((1 << lshift) < cp * SMAX * 8) ++lshift;
  const int nL = a.M * cp * SMAX;
  for (int idx = threadIdx.x; idx < nL; idx += blockDim.x) {
    const int s = idx % SMAX, mc = idx / SMAX, c = mc % cp, m = mc / cp;
    sL[idx] = (c < a.C && s < a.cfg_stages[c]) ? a.stage_lat[((int64_t)m * a.C + c) * a.smax_in + s] : 0.0;
  }
  bytes = ((size_t)nL * 8 + 15) / 16 * 16;
  __syncthreads();
  return lshift;
}

template <int W, int SMAX, bool STATS, int ROW, bool MS = false>
__device__ __forceinline__ LeanOut lean_go(const KArgs& a, const LeanIn& in, const double* sL, int lshift,
                                           unsigned char* rec, uint32_t* cnt) {
  if (lean_uni(in.cfg))
    return lean_run<W, SMAX, true, STATS, ROW, MS>(a, in, sL, lshift, rec, cnt);
  return lean_run<W, SMAX, false, STATS, ROW, MS>(a, in, sL, lshift, rec, cnt);
}

// The first of the launch's row jobs (f < n) for which own(job) holds, -1: none.
// Called by whole wavefronts.
template <class Own>
__device__ __forceinline__ int lean_row(const KArgs& a, int n, Own own) {
  const int lane = threadIdx.x & 63;
  for (int b = 0; b < n; b += 64) {
    const uint64_t hit = __builtin_amdgcn_ballot_w64(b + lane < n && own(a.finish_jobs[b + lane < n ? b + lane : 0]));
    if (hit) return b + __builtin_ctzll(hit);
  }
  return -1;
}

// Workgroup blk of the jobs v of one shared trace.  Wavefront w runs jw
// placements at one scale or, with MS, jw jobs in a row whatever their scale,
// and writes the per-request row of the first of them that has one; after the
// last of them, wavefront by wavefront, the other jobs with a row once more for
// the row alone (rows_apart, where SIMDs are left for them: all jobs with a row).
// A row makes its wavefront 4 to 9 % longer, and a wavefront more on a SIMD that
// has others makes the launch a third to a half longer: 2048 jobs of 64 one-stage
// groups, 20,000 requests, take 2.81 ms, with 4 rows 2.92 this way and 4.01 with
// wavefronts of their own; 512 jobs 2.23, 2.31 and 2.24.
template <int W, int SMAX, bool STATS, bool ROWS, bool MS = false>
__device__ __forceinline__ void lean_body(const KArgs& a, const JobSet& v, int64_t blk) {
  static_assert(!(STATS && MS), "statistics launches run one scale a wavefront");
  extern __shared__ __align__(16) unsigned char smem[];
  double* sL = reinterpret_cast<double*>(smem);
  size_t tab = 0;
  const int lshift = lean_table<SMAX>(a, sL, tab);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char* rec = smem + tab + (size_t)wave * lean_wave_lds(W, a.M, SMAX, STATS);
  uint32_t* cnt = reinterpret_cast<uint32_t*>(rec + lean_wave_bytes(SMAX));
  const int64_t w = blk * (int64_t)(blockDim.x >> 6) + wave;
  const int64_t P = v.J / a.K, per = (P + v.jw - 1) / v.jw;
  const int64_t nw = MS ? (v.J + v.jw - 1) / v.jw : per * a.K;
  const bool again = ROWS && w >= nw;
  if (again ? w - nw >= a.n_finish : w >= nw) return;

  LeanIn in;
  in.t = a.t;
  in.model = a.model;
  in.n = a.n;
  in.row = nullptr;
  in.row_n = a.n;
  in.row_slot = 0;
  // the jobs of the wavefront: slot s has job job0 + s * step; of_wave: whether
  // a job is one of wavefront x's
  const uint32_t K = (uint32_t)a.K, jw = (uint32_t)v.jw;
  auto wave_of = [&](uint32_t j) -> int64_t { return MS ? j / jw : (int64_t)(j % K) * per + j / K / jw; };
  int64_t job0, step = MS ? 1 : a.K;
  if (again) {
    const int f = (int)(w - nw);
    job0 = a.finish_jobs[f];
    const int64_t x = wave_of((uint32_t)job0);
    if (!a.rows_apart && lean_row(a, f, [&](int j) { return wave_of((uint32_t)j) == x; }) < 0) return;  // x writes it
    in.jw = 1;
    in.row = a.out_finish + f * a.n;
  } else {
    const int64_t k = w / per, p0 = (w % per) * v.jw;
    job0 = MS ? w * v.jw : p0 * a.K + k;
    const int64_t left = MS ? v.J - job0 : P - p0;
    in.jw = (int)(left < v.jw ? left : v.jw);
    if constexpr (ROWS) {
      const int f = a.n > 0 && !a.rows_apart
                        ? lean_row(a, a.n_finish, [&](int j) { return wave_of((uint32_t)j) == w; })
                        : -1;
      if (f >= 0) {
        in.row = a.out_finish + f * a.n;
        in.row_slot = (int)((a.finish_jobs[f] - job0) / step);
      }
    }
  }
  in.digest = !again && v.out_digest != nullptr;
  const int slot = lane / W, g = lane % W;
  const bool mine = slot < in.jw && g < v.G;
  const int64_t job = job0 + slot * step;
  // (a placement's number: J < 2^31)
  const int64_t p = MS ? (int64_t)((uint32_t)(slot < in.jw ? job : job0) / (uint32_t)a.K) : job0 / a.K + slot;
  in.sigma = a.slo_scale[MS ? (slot < in.jw ? job : job0) - p * a.K : job0 % a.K];
  in.cfg = mine ? v.group_cfg[p * v.G + g] : -1;
  if (in.cfg >= a.C || in.cfg < 0) in.cfg = -1;
  const uint64_t valid = __builtin_amdgcn_ballot_w64(in.cfg >= 0);
  in.hm = 0;
  const uint64_t groups = W == 64 ? ~0ull : (1ull << W) - 1;
  int64_t pj = job0 / a.K, kj = job0 % a.K;
#pragma unroll 4
  for (int j = 0; j < in.jw; ++j) {
    const uint64_t x = lane < a.M ? v.host_mask[pj * a.M + lane] & groups : 0;
    in.hm |= x << (W == 64 ? 0 : j * W);
    if (!MS || ++kj == a.K) {
      ++pj;
      kj = 0;
    }
  }
  in.hm &= valid;
  if constexpr (STATS) {
    for (int i = lane; i < in.jw * a.M; i += 64) cnt[i] = 0;
    lean_fence();
  }
  LeanOut o;
  bool done = false;
  if constexpr (ROWS) {
    if (again) {
      (void)lean_go<W, SMAX, false, 2>(a, in, sL, lshift, rec, cnt);
      return;
    }
    if (in.row) {
      o = lean_go<W, SMAX, false, 1, MS>(a, in, sL, lshift, rec, cnt);
      done = true;
    }
  }
  if (!done) o = lean_go<W, SMAX, STATS, 0, MS>(a, in, sL, lshift, rec, cnt);
  if (slot < in.jw && g == 0) {
    v.out_served[job] = o.served;
    if (v.out_attain) v.out_attain[job] = a.n > 0 ? (double)o.served / (double)a.n : 0.0;
    if (v.out_digest) {
      v.out_digest[2 * job] = o.hash;
      v.out_digest[2 * job + 1] = o.fin_sum;
    }
  }
  if constexpr (STATS) {
    if (mine && v.out_group_busy) v.out_group_busy[job * v.G + g] = o.busy;
    lean_fence();
    if (v.out_model_served)
      for (int i = lane; i < in.jw * a.M; i += 64)
        v.out_model_served[(job0 + i / a.M * step) * a.M + i % a.M] = (int64_t)cnt[i];
  }
}

template <int W, int SMAX, bool STATS, bool MS>
__global__ __launch_bounds__(kThreads) void shared_kernel(const KArgs a, int jw) {
  if (a.gate && *a.gate == 0) return;
  lean_body<W, SMAX, STATS, !STATS, MS>(a, job_set(a, jw), blockIdx.x);
}

// Jobs with trace segments of their own, one per wavefront at a time: slot ->
// job through a.order where it is set; with a.next_slot (0 at launch) the
// wavefronts take slots in turn until none is left, otherwise wavefront w of
// the launch runs slot w.  With rows_apart the first slots are the jobs with a
// row, for the row alone; otherwise a job's wavefront writes its row too.
template <int W, int SMAX>
__global__ __launch_bounds__(kThreads) void seg_kernel(const KArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  double* sL = reinterpret_cast<double*>(smem);
  size_t tab = 0;
  const int lshift = lean_table<SMAX>(a, sL, tab);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned char* rec = smem + tab + (size_t)wave * lean_wave_lds(W, a.M, SMAX, false);
  auto take_slot = [&]() -> int64_t {
    int v = 0;
    if (lane == 0) v = atomicAdd(a.next_slot, 1);
    return (int64_t)__builtin_amdgcn_readfirstlane(v);
  };
  int64_t slot = a.next_slot ? take_slot() : (int64_t)blockIdx.x * (blockDim.x >> 6) + wave;
  const int64_t apart = a.rows_apart ? a.n_finish : 0;
  while (slot < apart + a.J) {
    const bool again = slot < apart;
    const int64_t s = slot - apart;
    const int64_t job = again ? (int64_t)a.finish_jobs[slot]
                              : a.order ? (int64_t)__builtin_amdgcn_readfirstlane(a.order[s]) : s;
    int p = 0;
    double sigma = 0.0;
    int64_t begin = 0, len = 0;
    seg_job(a, job, p, sigma, begin, len);
    p = __builtin_amdgcn_readfirstlane(p);
    begin = (int64_t)lean_uniform((uint64_t)begin);
    len = (int64_t)lean_uniform((uint64_t)len);
    LeanIn in;
    in.t = a.t + begin;
    in.model = a.model + begin;
    in.n = len;
    in.jw = 1;
    in.sigma = sigma;
    in.row_n = len < a.finish_stride ? len : a.finish_stride;
    in.row_slot = 0;
    const int f = again ? (int)slot
                        : apart || in.row_n <= 0 ? -1 : lean_row(a, a.n_finish, [&](int j) { return j == job; });
    in.row = f >= 0 ? a.out_finish + f * a.finish_stride : nullptr;
    in.digest = !again && a.out_digest != nullptr;
    if (again && in.n > in.row_n) in.n = in.row_n;  // the row needs no more requests
    in.cfg = lane < a.G ? a.group_cfg[(int64_t)p * a.G + lane] : -1;
    if (in.cfg >= a.C || in.cfg < 0) in.cfg = -1;
    in.hm = (lane < a.M ? a.host_mask[(int64_t)p * a.M + lane] : 0) & __builtin_amdgcn_ballot_w64(in.cfg >= 0);
    if (again) {
      (void)lean_go<W, SMAX, false, 2>(a, in, sL, lshift, rec, nullptr);
    } else {
      LeanOut o;
      if (in.row)
        o = lean_go<W, SMAX, false, 1>(a, in, sL, lshift, rec, nullptr);
      else
        o = lean_go<W, SMAX, false, 0>(a, in, sL, lshift, rec, nullptr);
      if (lane == 0) {
        a.out_served[job] = o.served;
        if (a.out_attain) a.out_attain[job] = len > 0 ? (double)o.served / (double)len : 0.0;
        if (a.out_digest) {
          a.out_digest[2 * job] = o.hash;
          a.out_digest[2 * job + 1] = o.fin_sum;
        }
      }
    }
    if (!a.next_slot) break;
    slot = take_slot();
  }
}

}  // namespace as_dev
