// Kernel launchers, one translation unit per lanes-per-job width W (the
// build compiles sim_launch.hip once per W with -DAS_W=W and links them).
#pragma once

#include <hip/hip_runtime.h>

#include "sim_kernel.hpp"
#include "sim_shared.hpp"

namespace as_dev {
struct SpecArgs;
}

namespace as_host {

using as_dev::KArgs;

// General LDS-staged kernel: GPL groups per lane, SEG = per-job segments.
template <int W>
hipError_t launch_lds(int gpl, int smax, bool seg, const KArgs& a, size_t lds, hipStream_t s);

// Group-per-lane kernels (sim_lean.hpp), one group per lane: the jobs of a
// shared trace (one scale, or several scales, a wavefront), the same with the
// heuristic's statistics (one scale), or segmented jobs (a.order, a.next_slot).
// jw: jobs per wavefront of a shared trace; blocks workgroups of `waves`
// wavefronts.
enum class LeanKind { kShared, kScales, kStats, kSeg };
template <int W>
hipError_t launch_lean(LeanKind kind, int smax, const KArgs& a, int jw, int64_t blocks, int waves, size_t lds,
                       hipStream_t s);

// Several shapes of the shared-trace kernel (one SLO scale, no per-request
// rows) in one dispatch over `blocks` workgroups (sim_multi.hip); a_dev: the
// common arguments in device memory, unchanged until the launch has run.
hipError_t launch_shared_multi(bool stats, const KArgs* a_dev, const as_dev::MultiSegs& ms, int64_t blocks,
                               int waves, size_t lds, hipStream_t s);

// Round q of the speculative kernels' fix-ups (sim_spec.hpp), one job per
// wavefront, W = 4 .. 64 lanes hold the groups.
template <int W>
hipError_t launch_fix(int smax, const as_dev::SpecArgs& a, int q, int64_t blocks, size_t lds, hipStream_t s);
extern template hipError_t launch_fix<4>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
extern template hipError_t launch_fix<8>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
extern template hipError_t launch_fix<16>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
extern template hipError_t launch_fix<32>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
extern template hipError_t launch_fix<64>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
// The same for any group count; the grid and the LDS are chosen here.
hipError_t launch_fix_any(int smax, const as_dev::SpecArgs& a, int q, hipStream_t s);

#define AS_DECLARE_W(W)                                                                       \
  extern template hipError_t launch_lds<W>(int, int, bool, const KArgs&, size_t, hipStream_t); \
  extern template hipError_t launch_lean<W>(LeanKind, int, const KArgs&, int, int64_t, int, size_t, hipStream_t);
AS_DECLARE_W(1)
AS_DECLARE_W(2)
AS_DECLARE_W(4)
AS_DECLARE_W(8)
AS_DECLARE_W(16)
AS_DECLARE_W(32)
AS_DECLARE_W(64)
#undef AS_DECLARE_W

}  // namespace as_host
