// C-ABI of the batched serving simulator: argument checks, kernel selection,
// launches on the caller's stream, error reporting.  See alpaserve_sim.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "alpaserve_sim.h"
#include "sim_kernel.hpp"
#include "sim_shared.hpp"
#include "sim_launch.hpp"
#include "sim_lean.hpp"
#include "sim_internal.hpp"

namespace as_host {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int ok() {
  g_err.clear();
  return AS_OK;
}

int pow2ceil(int x) {
  int p = 1;
  while (p < x) p <<= 1;
  return p;
}

using as_dev::KArgs;

// LDS bytes of one workgroup for lanes-per-job W and padded stage count SMAX.
size_t lds_bytes(int W, int SMAX, bool seg, int M, int C) {
  const int slots = (64 / W) * as_dev::kWaves;
  int ch = as_dev::kChunk;
  if (seg) {
    ch = 4096 / slots;
    if (ch > 128) ch = 128;
    if (ch < 32) ch = 32;
    ch *= slots;
  }
  return (size_t)M * pow2ceil(C) * SMAX * 8 + (size_t)M * 8 + (size_t)ch * 12;
}

constexpr size_t kMaxLds = 64 * 1024;

// LDS a workgroup of the shared-trace kernel may use: the device's per-block
// limit (160 KiB on gfx950), cached per device.
size_t shared_lds_limit() {
  static size_t cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return kMaxLds;
  if (cache[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
      v = (int)kMaxLds;
    cache[dev] = (size_t)(v > 160 * 1024 ? 160 * 1024 : v);
  }
  return cache[dev];
}


hipError_t launch_lds_any(int W, int gpl, int smax, bool seg, const KArgs& a, size_t lds, hipStream_t s) {
  switch (W) {
    case 1: return as_host::launch_lds<1>(gpl, smax, seg, a, lds, s);
    case 2: return as_host::launch_lds<2>(gpl, smax, seg, a, lds, s);
    case 4: return as_host::launch_lds<4>(gpl, smax, seg, a, lds, s);
    case 8: return as_host::launch_lds<8>(gpl, smax, seg, a, lds, s);
    case 16: return as_host::launch_lds<16>(gpl, smax, seg, a, lds, s);
    case 32: return as_host::launch_lds<32>(gpl, smax, seg, a, lds, s);
    default: return as_host::launch_lds<64>(gpl, smax, seg, a, lds, s);
  }
}

hipError_t launch_lean_any(LeanKind kind, int W, int smax, const KArgs& a, int jw, int64_t blocks, int waves,
                           size_t lds, hipStream_t s) {
  switch (W) {
    case 1: return as_host::launch_lean<1>(kind, smax, a, jw, blocks, waves, lds, s);
    case 2: return as_host::launch_lean<2>(kind, smax, a, jw, blocks, waves, lds, s);
    case 4: return as_host::launch_lean<4>(kind, smax, a, jw, blocks, waves, lds, s);
    case 8: return as_host::launch_lean<8>(kind, smax, a, jw, blocks, waves, lds, s);
    case 16: return as_host::launch_lean<16>(kind, smax, a, jw, blocks, waves, lds, s);
    case 32: return as_host::launch_lean<32>(kind, smax, a, jw, blocks, waves, lds, s);
    default: return as_host::launch_lean<64>(kind, smax, a, jw, blocks, waves, lds, s);
  }
}

// SIMDs of the current device (4 per compute unit), cached per device.
int simd_count() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1024;
  if (cache[dev] == 0) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return 1024;
    cache[dev] = prop.multiProcessorCount * 4;
  }
  return cache[dev];
}

// Jobs per wavefront of a shared trace (at most 64 / W): as few as leave one
// wavefront per SIMD, since jobs that share a wavefront stage the requests of
// all of them and a second wavefront on a SIMD slows the first.
int lean_jobs_per_wave(int W, int64_t J) {
  const int64_t need = (J + simd_count() - 1) / simd_count();
  return (int)std::max<int64_t>(1, std::min<int64_t>(64 / W, need));
}

// Wavefronts per workgroup: as many as put every workgroup on a compute unit
// of its own, up to the four that its SIMDs run side by side (two workgroups
// of two wavefronts can share two SIMDs and leave two idle: 777 wavefronts of
// 32 lanes and 2 stages took 10.8 ms so, 7.4 ms in workgroups of four),
// fewer where their LDS does not fit.
int lean_waves_per_block(int64_t waves, int W, const KArgs& a, int smax, bool stats) {
  const int64_t cus = compute_units();
  int w = waves > 2 * cus ? 4 : waves > cus ? 2 : 1;
  while (w > 1 && as_dev::lean_lds_bytes(W, a.M, pow2ceil(a.C), smax, stats, w) > shared_lds_limit()) w /= 2;
  return w;
}

// Wavefronts of J jobs (K scales per placement) at jw jobs of one scale per
// wavefront.
int64_t lean_wave_count(int64_t J, int64_t K, int jw) { return K * ((J / K + jw - 1) / jw); }

// Whether wavefronts take jobs of several scales, which costs a request two
// instructions: where wavefronts of one scale, at most one job for every
// placement, are a tenth more and do not all have a SIMD of their own.  Measured
// at 4000 requests, apart and mixed: 1 placement x 16,384 scales on 4 four-stage
// groups 3.16 and 0.35 ms, on 32 one-stage groups 3.42 and 1.89; 3 x 4096 on 16
// four-stage groups 1.04 and 0.84.
bool lean_mixes_scales(int W, int64_t J, int64_t K, int jw) {
  const int64_t apart = lean_wave_count(J, K, jw), mixed = (J + jw - 1) / jw;
  return W < 64 && apart > simd_count() && mixed * 11 < apart * 10;
}

// Which calls the group-per-lane kernels take, by their stage-latency tables:
// the sizes these calls have always been taken up to (the table, 32 to 128 bytes
// a model for four wavefronts and a staged chunk of 2048, or of four times 256,
// requests in a workgroup's LDS).  Larger ones are refused, as they always have
// been: the general kernel takes tables of 64 KB at most, all of them among
// these.  The kernels themselves need less.
bool lean_takes(const KArgs& a, int smax, int chunk = 2048) {
  const size_t records = (size_t)as_dev::kWaves * a.M * ((size_t)1 << as_dev::rec_shift(smax));
  return records + (size_t)a.M * pow2ceil(a.C) * smax * 8 + (size_t)chunk * 20 <= shared_lds_limit();
}

// Jobs with trace segments of their own: whether each gets a wavefront (the
// group-per-lane kernel) or the general kernel packs 64 / W of them into one.
// A wavefront to itself has the shorter chain, by two to nine times while the
// SIMDs are not full; packed, a request of all of them costs one wavefront
// about what two to four requests cost there.  The line lies at the jobs per
// SIMD where both take the same time on segments of equal length (which the
// host does not know; with lengths spread over a factor of ten the packed
// wavefronts wait for their longest and lose up to three times there).
// Measured, packed / one per wavefront, at jobs per SIMD: 1 lane 1.5 at 16 and
// 0.6 at 64; 2 lanes 0.9 to 1.2 at 16, 0.5 to 0.7 at 32; 4 lanes 1.7 at 2, 0.9
// at 4, 0.4 at 16; 8 lanes 1.2 at 2 and 0.8 at 3; 16 lanes 1.0 and 0.7 to 0.8;
// 32 lanes 1.1 to 1.3 and 0.7 to 1.1, 0.6 at 4.
bool seg_one_per_wave(int W, int64_t J) {
  const int64_t per_simd = W >= 64 ? INT64_MAX / 65536 : W >= 8 ? 2 : W == 4 ? 4 : W == 2 ? 16 : 24;
  return J <= per_simd * simd_count();
}

// Lanes per job W and groups per lane GPL (W * GPL >= G, powers of two).
// Cost model: a wavefront issues in order, so the time of a launch is about
// (wavefronts per SIMD, at least 1) x (instructions per request of one
// wavefront); a lane that carries more groups needs more instructions per
// request but fewer wavefronts.  Relative instruction counts per request for
// GPL = 1, 2, 4 are measured values.  Shapes whose LDS tables do not fit are
// skipped (a wider W means fewer job slots per workgroup).  ALPASERVE_GPL=1|2|4
// forces GPL.  Returns false when no shape fits.
bool choose_shape(int G, int64_t J, bool seg, int M, int C, int smax, int& W, int& GPL,
                  bool allow_force = true) {
  const int Gp = pow2ceil(G);
  const double instr[3] = {1.0, 1.45, 2.3};
  const int n_simd = simd_count();
  int force = 0;
  if (const char* e = getenv("ALPASERVE_GPL"); e && allow_force) force = atoi(e);
  double best = 1e300;
  bool found = false;
  for (int i = 0; i < 3; ++i) {
    const int gpl = 1 << i;
    if (gpl > Gp || (force && force != gpl)) continue;
    for (int w = Gp / gpl; w <= 64 && w * gpl <= 64; w *= 2) {
      if (lds_bytes(w, smax, seg, M, C) > kMaxLds) continue;
      const int64_t waves = (J + (64 / w) - 1) / (64 / w);
      const double occ = (double)waves / n_simd;
      const double cost = (occ > 1.0 ? occ : 1.0) * instr[i];
      if (cost < best) {
        best = cost;
        W = w;
        GPL = gpl;
        found = true;
      }
      break;  // the narrowest W that fits is the cheapest for this GPL
    }
  }
  // a forced GPL that does not apply to this problem yields to the cost model
  if (!found && force) return choose_shape(G, J, seg, M, C, smax, W, GPL, false);
  return found;
}

// Which kernel family runs a shared-trace call: by default the
// segment-speculative kernels when the trace splits into segments, else the
// shared-trace kernel; ALPASERVE_PATH=lds selects the LDS-staged kernel,
// =spec the segment-speculative one, =shared the shared-trace one (tests
// cover each).
bool use_shared_path() {
  const char* e = getenv("ALPASERVE_PATH");
  return !(e && std::strcmp(e, "lds") == 0);
}

// The segment-speculative kernels take a call unless another family is
// forced; they decline (AS_E_LIMITS) calls they cannot cut into segments.
bool want_spec(const KArgs& a, int smax) {
  (void)a;
  (void)smax;
  const char* e = getenv("ALPASERVE_PATH");
  return !(e && *e) || std::strcmp(e, "spec") == 0;
}

bool spec_forced() {
  const char* e = getenv("ALPASERVE_PATH");
  return e && std::strcmp(e, "spec") == 0;
}

// Checks shared by both simulate entry points; fills the model/placement part
// of KArgs and the kernel shape.
int check_common(const as_models_t* models, const as_placements_t* plc, KArgs& a, int& W,
                 int& smax) {
  if (!models || !plc) return fail(AS_E_INVALID_ARG, "models and placements must not be NULL");
  const as_models_t& md = *models;
  const as_placements_t& pl = *plc;
  if (md.n_models < 1 || md.n_models > AS_MAX_MODELS)
    return fail(md.n_models < 1 ? AS_E_INVALID_ARG : AS_E_LIMITS, "n_models=%d outside 1..%d",
                md.n_models, AS_MAX_MODELS);
  if (md.n_configs < 1 || md.n_configs > AS_MAX_CONFIGS)
    return fail(md.n_configs < 1 ? AS_E_INVALID_ARG : AS_E_LIMITS, "n_configs=%d outside 1..%d",
                md.n_configs, AS_MAX_CONFIGS);
  if (md.max_stages < 1) return fail(AS_E_INVALID_ARG, "max_stages=%d < 1", md.max_stages);
  if (!md.d_single || !md.stage_lat || !md.cfg_stages)
    return fail(AS_E_INVALID_ARG, "d_single, cfg_stages and stage_lat must not be NULL");
  int smax_used = 1;
  for (int c = 0; c < md.n_configs; ++c) {
    const int S = md.cfg_stages[c];
    if (S < 1 || S > md.max_stages)
      return fail(AS_E_INVALID_ARG, "cfg_stages[%d]=%d outside 1..max_stages=%d", c, S, md.max_stages);
    if (S > AS_MAX_STAGES)
      return fail(AS_E_LIMITS, "cfg_stages[%d]=%d > %d", c, S, AS_MAX_STAGES);
    if (S > smax_used) smax_used = S;
  }
  if (pl.n_placements < 0) return fail(AS_E_INVALID_ARG, "n_placements=%d < 0", pl.n_placements);
  if (pl.max_groups < 1 || pl.max_groups > AS_MAX_GROUPS)
    return fail(pl.max_groups < 1 ? AS_E_INVALID_ARG : AS_E_LIMITS, "max_groups=%d outside 1..%d",
                pl.max_groups, AS_MAX_GROUPS);
  if (pl.n_placements > 0 && (!pl.group_cfg || !pl.host_mask))
    return fail(AS_E_INVALID_ARG, "group_cfg and host_mask must not be NULL");
  a.d_single = md.d_single;
  a.stage_lat = md.stage_lat;
  a.group_cfg = pl.group_cfg;
  a.host_mask = pl.host_mask;
  a.M = md.n_models;
  a.C = md.n_configs;
  a.smax_in = md.max_stages;
  a.G = pl.max_groups;
  a.P = pl.n_placements;
  for (int c = 0; c < AS_MAX_CONFIGS; ++c) a.cfg_stages[c] = c < md.n_configs ? md.cfg_stages[c] : 1;
  W = pl.max_groups;  // group count; the shape is chosen per call
  smax = pow2ceil(smax_used);
  return AS_OK;
}

int check_finish(const int32_t* finish_jobs, int32_t n_finish, double* out_finish, int64_t J,
                 KArgs& a) {
  if (n_finish < 0) return fail(AS_E_INVALID_ARG, "n_finish=%d < 0", n_finish);
  if (n_finish > AS_MAX_FINISH) return fail(AS_E_LIMITS, "n_finish=%d > %d", n_finish, AS_MAX_FINISH);
  if (n_finish > 0 && (!finish_jobs || !out_finish))
    return fail(AS_E_INVALID_ARG, "finish_jobs and out_finish must not be NULL when n_finish > 0");
  for (int f = 0; f < n_finish; ++f) {
    if (finish_jobs[f] < 0 || finish_jobs[f] >= J)
      return fail(AS_E_INVALID_ARG, "finish_jobs[%d]=%d outside [0, %lld)", f, finish_jobs[f],
                  (long long)J);
    for (int q = 0; q < f; ++q)
      if (finish_jobs[q] == finish_jobs[f])
        return fail(AS_E_INVALID_ARG, "finish_jobs[%d] repeats job %d", f, finish_jobs[f]);
    a.finish_jobs[f] = finish_jobs[f];
  }
  a.n_finish = n_finish;
  a.out_finish = out_finish;
  return AS_OK;
}


// ---------------------------------------------------------------- validation
enum : uint32_t {
  V_T_ORDER = 1u << 0,   // t not finite, negative or decreasing
  V_MODEL = 1u << 1,     // model id out of range
  V_CFG = 1u << 2,       // group configuration outside [-1, C)
  V_MASK = 1u << 3,      // hosting bit on a missing group
  V_LAT = 1u << 4,       // stage latency not finite or negative
  V_DSINGLE = 1u << 5,   // d_single not finite or not positive
  V_SCALE = 1u << 6,     // SLO scale negative or NaN
};
const char* kValidateMsg[] = {
    "trace times must be finite, >= 0 and nondecreasing",
    "model ids must lie in [0, n_models)",
    "group_cfg entries must lie in [-1, n_configs)",
    "host_mask may only set bits of groups with group_cfg >= 0",
    "stage latencies (s < S_c) must be finite and >= 0",
    "d_single must be finite and > 0",
    "slo_scale must be >= 0 and not NaN",
};

__global__ void validate_kernel(const double* t, const int32_t* model, int64_t n, int M, int C,
                                const int32_t* group_cfg, const uint64_t* host_mask, int64_t P, int G,
                                const double* stage_lat, int smax_in, const double* d_single,
                                const double* scales, int K, KArgs cfgs, uint32_t* flags) {
  uint32_t bad = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t tid0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = tid0; i < n; i += stride) {
    const double ti = t[i];
    if (!(ti >= 0.0) || !(ti <= 1.7976931348623157e308)) bad |= V_T_ORDER;
    if (i > 0 && !(t[i - 1] <= ti)) bad |= V_T_ORDER;
    const int32_t m = model[i];
    if (m < 0 || m >= M) bad |= V_MODEL;
  }
  for (int64_t j = tid0; j < P * G; j += stride) {
    const int32_t c = group_cfg[j];
    if (c < -1 || c >= C) bad |= V_CFG;
  }
  for (int64_t j = tid0; j < P * M; j += stride) {
    const int64_t p = j / M;
    const uint64_t mask = host_mask[j];
    for (int g = 0; g < 64; ++g)
      if ((mask >> g) & 1u)
        if (g >= G || group_cfg[p * G + g] < 0) bad |= V_MASK;
  }
  for (int64_t j = tid0; j < (int64_t)M * C * smax_in; j += stride) {
    const int s = (int)(j % smax_in);
    const int c = (int)((j / smax_in) % C);
    const double v = stage_lat[j];
    if (s < cfgs.cfg_stages[c] && (!(v >= 0.0) || !(v <= 1.7976931348623157e308))) bad |= V_LAT;
  }
  for (int64_t j = tid0; j < M; j += stride) {
    const double d = d_single[j];
    if (!(d > 0.0) || !(d <= 1.7976931348623157e308)) bad |= V_DSINGLE;
  }
  for (int64_t j = tid0; j < K; j += stride)
    if (!(scales[j] >= 0.0)) bad |= V_SCALE;
  if (bad) atomicOr(flags, bad);
}

// Statistics launch of the group-per-lane kernels.  They take the tables that
// fit a workgroup's LDS beside the models' SLOs, 1024 staged requests and the
// counters of four jobs, as these calls always have; the kernels need less,
// with at most four jobs per wavefront where the counters of more do not fit.
int run_shared_stats(KArgs& a, int smax, hipStream_t stream) {
  const int cp = pow2ceil(a.C);
  if ((size_t)a.M * cp * smax * 8 + (size_t)a.M * (8 + as_dev::kWaves * 4) + 1024 * 12 > shared_lds_limit())
    return fail(AS_E_LIMITS, "stage-latency table (%d models x %d configs x %d stages) does not fit in LDS",
                a.M, a.C, smax);
  int W = pow2ceil(a.G);
  while (W < 16 && as_dev::lean_lds_bytes(W, a.M, cp, smax, true, 1) > shared_lds_limit()) W *= 2;
  const int jw = lean_jobs_per_wave(W, a.J);
  const int64_t nw = lean_wave_count(a.J, a.K, jw);
  const int waves = lean_waves_per_block(nw, W, a, smax, true);
  const size_t lds = as_dev::lean_lds_bytes(W, a.M, cp, smax, true, waves);
  const hipError_t e =
      launch_lean_any(LeanKind::kStats, W, smax, a, jw, (nw + waves - 1) / waves, waves, lds, stream);
  if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return ok();
}

// Multi-shape dispatches pay where the jobs are few: a step whose shapes run
// on separate streams costs a trace pass of latency per shape that shares a
// hardware queue.  Where the blocks fill the device many times over, launches
// of their own shapes run faster (the multi-shape kernel holds the registers
// and LDS of its largest shape), and they overlap anyway.
constexpr int64_t kMultiMaxBlocks = 2048;

int run_shared_multi(const KArgs& a, void* dev_args, const ShapeJobs* sh, int n, bool stats, hipStream_t stream) {
  if (!use_shared_path() || a.K != 1 || a.n_finish != 0 || n < 1 || n > as_dev::kMaxShapeSegs || !dev_args)
    return AS_E_LIMITS;
  size_t lds = 0;
  as_dev::MultiSegs ms;
  std::memset(&ms, 0, sizeof ms);
  int64_t blocks = 0, all = 0;
  for (int i = 0; i < n; ++i) all += sh[i].v.J;
  const int waves = 4;
  for (int i = 0; i < n; ++i) {
    const int W = sh[i].W, sm = sh[i].smax;
    if (W < 1 || W > 64 || (W & (W - 1)) != 0 || sh[i].v.G > W || (sm != 1 && sm != 2 && sm != 4 && sm != 8))
      return AS_E_LIMITS;
    if (sh[i].v.J <= 0) continue;
    if (!lean_takes(a, sm)) return AS_E_LIMITS;
    if (!stats) {
      KArgs ak = a;
      ak.J = sh[i].v.J;
      ak.G = sh[i].v.G;
      if (want_spec(ak, sm) && spec_takes(ak, sm)) return AS_E_LIMITS;
    }
    lds = std::max(lds, as_dev::lean_lds_bytes(W, a.M, pow2ceil(a.C), sm, stats, waves));
    as_dev::ShapeSeg& g = ms.s[ms.n++];
    int wl = 0, sl = 0;
    while ((1 << wl) < W) ++wl;
    while ((1 << sl) < sm) ++sl;
    g.wl = wl;
    g.sl = sl;
    g.block0 = blocks;
    g.v = sh[i].v;
    g.v.jw = lean_jobs_per_wave(W, all);
    blocks += (lean_wave_count(g.v.J, 1, g.v.jw) + waves - 1) / waves;
  }
  if (lds > shared_lds_limit() || blocks > kMultiMaxBlocks) return AS_E_LIMITS;
  if (ms.n == 0) return ok();
  hipError_t e = hipMemcpyAsync(dev_args, &a, sizeof(KArgs), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = launch_shared_multi(stats, static_cast<const KArgs*>(dev_args), ms, blocks, waves, lds, stream);
  if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return ok();
}

// The shared-trace kernel (one group per lane, W = G rounded up to a power of
// two) unless its tables exceed the LDS of a workgroup; then the general
// kernel, whose tables are smaller.  With only_check, whether one of them
// takes the call (AS_OK) or not (AS_E_LIMITS), without launching.
int run_trace_kernels(KArgs& a, int W, int smax, hipStream_t stream, bool only_check) {
  const int64_t J = a.J;
  const int Ws = pow2ceil(a.G), jw = lean_jobs_per_wave(Ws, J);
  const bool mixes = lean_mixes_scales(Ws, J, a.K, jw);
  // the jobs, and those with a per-request row once more (most return at once
  // unless the rows are apart)
  const int64_t nw = (mixes ? (J + jw - 1) / jw : lean_wave_count(J, a.K, jw)) + (a.n > 0 ? a.n_finish : 0);
  a.rows_apart = nw <= simd_count();
  const int waves = lean_waves_per_block(nw, Ws, a, smax, false);
  const size_t lds_shared = as_dev::lean_lds_bytes(Ws, a.M, pow2ceil(a.C), smax, false, waves);
  if (use_shared_path() && lean_takes(a, smax) && lds_shared <= shared_lds_limit()) {
    if (only_check) return AS_OK;
    const hipError_t e = launch_lean_any(mixes ? LeanKind::kScales : LeanKind::kShared, Ws, smax, a, jw,
                                         (nw + waves - 1) / waves, waves, lds_shared, stream);
    if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    return ok();
  }
  int GPL = 1;
  if (!choose_shape(a.G, J, false, a.M, a.C, smax, W, GPL))
    return only_check ? AS_E_LIMITS
                      : fail(AS_E_LIMITS, "stage-latency tables (%d models x %d configs x %d stages) do not fit in LDS",
                             a.M, a.C, smax);
  if (only_check) return AS_OK;
  const size_t lds = lds_bytes(W, smax, false, a.M, a.C);
  hipError_t e = launch_lds_any(W, GPL, smax, false, a, lds, stream);
  if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return ok();
}

// Launch the batched simulation of a shared trace (a fully filled except the
// kernel shape).  W is the group count on entry.  The segment-speculative
// kernels go first where they take the call; when one of their re-runs gives
// up (traffic under which runs from different states do not meet), the
// kernels above, launched behind them and gated on that flag, produce the
// results instead.  All of it stays stream-ordered: no host synchronisation.
// A workspace allocation that fails leaves the call to those kernels where
// they can take it (they need no workspace).  With scratch, the speculative
// workspace comes from it (nothing is allocated), and a call that needs more
// than scratch_bytes returns AS_E_LIMITS.
int run_shared_trace(KArgs& a, int W, int smax, hipStream_t stream, void* scratch, size_t scratch_bytes) {
  if (want_spec(a, smax)) {
    const bool fallback = run_trace_kernels(a, W, smax, stream, true) == AS_OK;
    void* ws = nullptr;
    const int32_t* gave_up = nullptr;
    int rc = run_spec(a, smax, stream, fallback, scratch, scratch_bytes, &ws, &gave_up);
    if (rc == kSpecScratchTooSmall) return AS_E_LIMITS;
    if (rc == AS_E_NOMEM && fallback) rc = AS_E_LIMITS;
    if (rc != AS_E_LIMITS) {
      if (rc != AS_OK || !fallback) return rc;
      a.gate = gave_up;
      const int rc2 = run_trace_kernels(a, W, smax, stream, false);
      a.gate = nullptr;
      const hipError_t ef = ws ? hipFreeAsync(ws, stream) : hipSuccess;
      if (rc2 != AS_OK) return rc2;
      if (ef != hipSuccess) return fail(AS_E_HIP, "workspace release failed: %s", hipGetErrorString(ef));
      return ok();
    }
  }
  return run_trace_kernels(a, W, smax, stream, false);
}

}  // namespace as_host

using namespace as_host;

extern "C" {

const char* as_last_error(void) { return g_err.c_str(); }

const char* as_version(void) { return "alpaserve_sim 0.1 gfx950"; }

}  // extern "C"

namespace as_host {
namespace {

// Workspace of as_simulate_placements_noalloc: one array per device, held
// until the process ends, shared by every call on that device.
static __device__ __align__(256) unsigned char scratch[AS_NOALLOC_SCRATCH_BYTES];

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept; null with a message set when
// the lookup fails.  In host code the array's name is only a stand-in for
// the symbol, never a device address.
void* scratch_ptr() {
  static std::mutex mu;
  static void* ptrs[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    fail(AS_E_HIP, "no current HIP device");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!ptrs[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      fail(AS_E_HIP, "scratch address on device %d: %s", dev, hipGetErrorString(e));
      return nullptr;
    }
    ptrs[dev] = p;
  }
  return ptrs[dev];
}

// Body of as_simulate_placements; with no_alloc, the speculative kernels'
// workspace comes from `scratch` and nothing is allocated.
int simulate_placements(const as_trace_t* trace, const as_models_t* models,
                        const as_placements_t* placements, const double* slo_scale, int32_t n_scales,
                        int64_t* out_served, double* out_attain, uint64_t* out_digest,
                        const int32_t* finish_jobs, int32_t n_finish, double* out_finish, void* stream,
                        bool no_alloc) {
  KArgs a;
  std::memset(&a, 0, sizeof a);
  if (!trace) return fail(AS_E_INVALID_ARG, "trace must not be NULL");
  if (trace->n < 0) return fail(AS_E_INVALID_ARG, "trace n=%lld < 0", (long long)trace->n);
  if (trace->n > 0 && (!trace->t || !trace->model))
    return fail(AS_E_INVALID_ARG, "trace arrays must not be NULL");
  int W = 1, smax = 1;
  int rc = check_common(models, placements, a, W, smax);
  if (rc != AS_OK) return rc;
  if (n_scales < 0) return fail(AS_E_INVALID_ARG, "n_scales=%d < 0", n_scales);
  const int64_t J = (int64_t)placements->n_placements * n_scales;
  if (J > 0x7FFFFFFFLL) return fail(AS_E_LIMITS, "placements x scales = %lld jobs > 2^31-1", (long long)J);
  if (J > 0 && (!slo_scale || !out_served))
    return fail(AS_E_INVALID_ARG, "slo_scale and out_served must not be NULL");
  rc = check_finish(finish_jobs, n_finish, out_finish, J, a);
  if (rc != AS_OK) return rc;
  if (J == 0) return ok();
  a.t = trace->t;
  a.model = trace->model;
  a.n = trace->n;
  a.slo_scale = slo_scale;
  a.K = n_scales;
  a.J = (int32_t)J;
  a.out_served = out_served;
  a.out_attain = out_attain;
  a.out_digest = out_digest;
  a.finish_stride = trace->n;
  if (!no_alloc) return run_shared_trace(a, W, smax, (hipStream_t)stream);
  void* ws = scratch_ptr();
  if (!ws) return AS_E_HIP;
  return run_shared_trace(a, W, smax, (hipStream_t)stream, ws, AS_NOALLOC_SCRATCH_BYTES);
}

}  // namespace
}  // namespace as_host

extern "C" {

int as_simulate_placements(const as_trace_t* trace, const as_models_t* models,
                           const as_placements_t* placements, const double* slo_scale,
                           int32_t n_scales, int64_t* out_served, double* out_attain,
                           uint64_t* out_digest, const int32_t* finish_jobs, int32_t n_finish,
                           double* out_finish, void* stream) {
  return simulate_placements(trace, models, placements, slo_scale, n_scales, out_served, out_attain,
                             out_digest, finish_jobs, n_finish, out_finish, stream, false);
}

int as_simulate_placements_noalloc(const as_trace_t* trace, const as_models_t* models,
                                   const as_placements_t* placements, const double* slo_scale,
                                   int32_t n_scales, int64_t* out_served, double* out_attain,
                                   uint64_t* out_digest, const int32_t* finish_jobs, int32_t n_finish,
                                   double* out_finish, void* stream) {
  return simulate_placements(trace, models, placements, slo_scale, n_scales, out_served, out_attain,
                             out_digest, finish_jobs, n_finish, out_finish, stream, true);
}

namespace as_dev {
namespace {

constexpr int kOrderMaxJobs = 4096;  // jobs the one-workgroup sort below takes

// Launch order of the one-job-per-wavefront kernel: the jobs sorted by
// segment length (longest first, lower index first on ties).  queue 0: one
// job per wavefront, the longest and the shortest alternating -- order[2i]
// the i-th longest, order[2i + 1] the i-th shortest -- so that the longest
// chains share their SIMDs with short ones.  queue 1: fewer wavefronts than
// jobs take the jobs in turn, longest first, from the slot counter
// order[J], which is set to 0 here.  J <= 4096.  A workgroup finds the places of
// 64 jobs, each of its 16 wavefronts counting the longer ones among a sixteenth
// of all (2000 jobs: 10 us; a bitonic sort in one workgroup took 50).
__global__ __launch_bounds__(1024) void seg_order(const KArgs a, int32_t* __restrict__ order, int queue) {
  __shared__ uint64_t key[kOrderMaxJobs];
  __shared__ int32_t place[64];
  const int J = (int)a.J, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < J; i += 1024) {
    int p = 0;
    double sigma = 0.0;
    int64_t begin = 0, len = 0;
    seg_job(a, i, p, sigma, begin, len);
    key[i] = ((uint64_t)len << 12) | (uint32_t)(kOrderMaxJobs - 1 - i);  // all different
  }
  if (threadIdx.x < 64) place[threadIdx.x] = 0;
  __syncthreads();
  const int i = (int)blockIdx.x * 64 + lane;
  const uint64_t mine = key[i < J ? i : J - 1];
  const int per = (J + 15) / 16, end = min(J, (wave + 1) * per);
  int before = 0;
#pragma unroll 8
  for (int q = wave * per; q < end; ++q) before += key[q] > mine ? 1 : 0;
  atomicAdd(place + lane, before);
  __syncthreads();
  if (threadIdx.x < 64 && i < J) {
    const int r = place[lane];
    order[queue ? r : 2 * r < J ? 2 * r : 2 * (J - 1 - r) + 1] = i;
  }
  if (queue && blockIdx.x == 0 && threadIdx.x == 0) order[J] = 0;
}

// Wavefronts per SIMD that take the sweep's jobs in turn.  Two: the longest
// job shares its SIMD with one other wavefront, which works through shorter
// jobs meanwhile (ALPASERVE_SEG_WAVES sets 1-4, for measurements).
int seg_waves_per_simd() {
  const char* e = getenv("ALPASERVE_SEG_WAVES");
  const int v = e ? atoi(e) : 2;
  return v < 1 ? 1 : (v > 4 ? 4 : v);
}

// Workgroups that take the jobs in turn: seg_waves_per_simd() per compute
// unit (ALPASERVE_SEG_BLOCKS sets the count, 1-4096, for the tests: a few
// workgroups then each work through many jobs).
int64_t seg_queue_blocks(int wps) {
  const char* e = getenv("ALPASERVE_SEG_BLOCKS");
  const int v = e ? atoi(e) : 0;
  if (v >= 1 && v <= 4096) return v;
  return (int64_t)wps * as_host::compute_units();
}

}  // namespace
}  // namespace as_dev

int as_simulate_jobs(const double* t, const int32_t* model, const int64_t* seg_offsets,
                     int32_t n_segments, const as_models_t* models,
                     const as_placements_t* placements, const as_job_t* jobs, int32_t n_jobs,
                     int64_t* out_served, double* out_attain, uint64_t* out_digest,
                     const int32_t* finish_jobs, int32_t n_finish, double* out_finish,
                     int64_t finish_stride, void* stream) {
  KArgs a;
  std::memset(&a, 0, sizeof a);
  if (n_segments < 0 || n_jobs < 0) return fail(AS_E_INVALID_ARG, "negative n_segments or n_jobs");
  int W = 1, smax = 1;
  int rc = check_common(models, placements, a, W, smax);
  if (rc != AS_OK) return rc;
  if (n_jobs > 0 && n_segments < 1)
    return fail(AS_E_INVALID_ARG, "n_segments must be >= 1 when there are jobs");
  if (n_jobs > 0 && (!t || !model || !seg_offsets || !jobs || !out_served))
    return fail(AS_E_INVALID_ARG, "t, model, seg_offsets, jobs and out_served must not be NULL");
  if (finish_stride < 0) return fail(AS_E_INVALID_ARG, "finish_stride < 0");
  rc = check_finish(finish_jobs, n_finish, out_finish, n_jobs, a);
  if (rc != AS_OK) return rc;
  if (n_jobs == 0) return ok();
  a.t = t;
  a.model = model;
  a.seg_off = seg_offsets;
  a.n_segments = n_segments;
  a.jobs = jobs;
  a.J = n_jobs;
  a.out_served = out_served;
  a.out_attain = out_attain;
  a.out_digest = out_digest;
  a.finish_stride = finish_stride;
  hipStream_t s = (hipStream_t)stream;
  const int Ws = pow2ceil(a.G);
  const size_t lds_seg = as_dev::lean_lds_bytes(Ws, a.M, pow2ceil(a.C), smax, false, as_dev::kWaves);
  int GPL = 1;
  const bool general = choose_shape(a.G, n_jobs, true, a.M, a.C, smax, W, GPL);
  if (use_shared_path() && (general || (Ws == 64 && lean_takes(a, smax, 1024))) && lds_seg <= shared_lds_limit() &&
      seg_one_per_wave(Ws, n_jobs)) {
    hipError_t e = hipSuccess;
    // Jobs longest first.  With more jobs than seg_waves_per_simd()
    // wavefronts per SIMD, that many wavefronts take them in turn (each
    // compute unit holds that many workgroups of one wavefront per SIMD: the
    // LDS request leaves room for no more); otherwise one job per wavefront,
    // long and short chains interleaved.  Skipped where every job has a SIMD of
    // its own and, never an error, where the jobs are too many for the sort or
    // its array cannot be allocated.
    const int wps = as_dev::seg_waves_per_simd();
    const int64_t queue_blocks = as_dev::seg_queue_blocks(wps);
    const int64_t n_rows = finish_stride > 0 ? a.n_finish : 0;
    a.rows_apart = n_rows > 0 && n_jobs + n_rows <= simd_count();
    const int64_t nw = n_jobs + (a.rows_apart ? n_rows : 0);
    int waves = lean_waves_per_block(nw, Ws, a, smax, false);
    int64_t blocks = (nw + waves - 1) / waves;
    size_t lds = lds_seg;
    int32_t* order = nullptr;
    const bool queue = blocks > queue_blocks;
    if (n_jobs <= as_dev::kOrderMaxJobs && (queue || n_jobs > simd_count()) &&
        pool_alloc(reinterpret_cast<void**>(&order), ((size_t)n_jobs + 1) * 4, s) != hipSuccess) {
      (void)hipGetLastError();
      order = nullptr;
    }
    if (order) {
      hipLaunchKernelGGL(as_dev::seg_order, dim3((unsigned)((n_jobs + 63) / 64)), dim3(1024), 0, s, a, order,
                         queue ? 1 : 0);
      if ((e = hipGetLastError()) != hipSuccess) {
        (void)hipFreeAsync(order, s);
        return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
      }
      a.order = order;
      if (queue) {
        a.next_slot = order + n_jobs;
        waves = as_dev::kWaves;
        blocks = queue_blocks;
        const size_t per_cu = 160 * 1024;  // LDS of a compute unit
        const size_t cap = per_cu / (size_t)(wps + 1) + 1024;
        if (cap > lds && cap <= shared_lds_limit()) lds = cap;
      }
    }
    e = launch_lean_any(LeanKind::kSeg, Ws, smax, a, 1, blocks, waves, lds, s);
    const hipError_t ef = order ? hipFreeAsync(order, s) : hipSuccess;
    if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
    if (ef != hipSuccess) return fail(AS_E_HIP, "order release failed: %s", hipGetErrorString(ef));
    return ok();
  }
  if (!general)
    return fail(AS_E_LIMITS, "stage-latency tables (%d models x %d configs x %d stages) do not fit in LDS",
                a.M, a.C, smax);
  const size_t lds = lds_bytes(W, smax, true, a.M, a.C);
  hipError_t e = launch_lds_any(W, GPL, smax, true, a, lds, s);
  if (e != hipSuccess) return fail(AS_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return ok();
}

int as_validate(const as_trace_t* trace, const as_models_t* models,
                const as_placements_t* placements, const double* slo_scale, int32_t n_scales,
                void* stream) {
  KArgs a;
  std::memset(&a, 0, sizeof a);
  if (!trace) return fail(AS_E_INVALID_ARG, "trace must not be NULL");
  if (trace->n < 0) return fail(AS_E_INVALID_ARG, "trace n=%lld < 0", (long long)trace->n);
  if (trace->n > 0 && (!trace->t || !trace->model))
    return fail(AS_E_INVALID_ARG, "trace arrays must not be NULL");
  int W = 1, smax = 1;
  int rc = check_common(models, placements, a, W, smax);
  if (rc != AS_OK) return rc;
  if (n_scales < 0) return fail(AS_E_INVALID_ARG, "n_scales=%d < 0", n_scales);
  if (n_scales > 0 && !slo_scale) return fail(AS_E_INVALID_ARG, "slo_scale must not be NULL");
  hipStream_t s = (hipStream_t)stream;
  uint32_t* d_flags = nullptr;
  hipError_t e = hipMallocAsync((void**)&d_flags, sizeof(uint32_t), s);
  if (e != hipSuccess) return fail(AS_E_NOMEM, "hipMallocAsync: %s", hipGetErrorString(e));
  uint32_t flags = 0;
  e = hipMemsetAsync(d_flags, 0, sizeof(uint32_t), s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(validate_kernel, dim3(1024), dim3(256), 0, s, trace->t, trace->model,
                       trace->n, a.M, a.C, a.group_cfg, a.host_mask,
                       (int64_t)placements->n_placements, a.G, a.stage_lat, a.smax_in, a.d_single,
                       slo_scale, n_scales, a, d_flags);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&flags, d_flags, sizeof flags, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  hipError_t ef = hipFreeAsync(d_flags, s);
  if (e == hipSuccess) e = ef;
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(AS_E_HIP, "as_validate: %s", hipGetErrorString(e));
  for (int b = 0; b < 7; ++b)
    if (flags & (1u << b)) return fail(AS_E_INVALID_DATA, "%s", kValidateMsg[b]);
  return ok();
}

}  // extern "C"
