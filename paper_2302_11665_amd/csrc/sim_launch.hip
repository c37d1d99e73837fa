// Kernel launchers for one lanes-per-job width W = AS_W (see sim_launch.hpp).
#include <hip/hip_runtime.h>

#include "sim_kernel.hpp"
#include "sim_launch.hpp"
#include "sim_lean.hpp"
#include "sim_spec.hpp"

#ifndef AS_W
#error "compile with -DAS_W=<lanes per job>"
#endif

namespace as_host {
namespace {

template <int W, int GPL, int SMAX, bool SEG>
hipError_t lds_t(const KArgs& a, size_t lds, hipStream_t s) {
  if constexpr (W * GPL > 64) {
    return hipErrorInvalidValue;
  } else {
    constexpr int slots = (64 / W) * as_dev::kWaves;
    const int grid = (a.J + slots - 1) / slots;
    hipLaunchKernelGGL((as_dev::sim_kernel<W, GPL, SMAX, SEG>), dim3(grid), dim3(as_dev::kThreads), lds,
                       s, a);
    return hipGetLastError();
  }
}

template <int W, int GPL, bool SEG>
hipError_t lds_s(int smax, const KArgs& a, size_t lds, hipStream_t s) {
  switch (smax) {
    case 1: return lds_t<W, GPL, 1, SEG>(a, lds, s);
    case 2: return lds_t<W, GPL, 2, SEG>(a, lds, s);
    case 4: return lds_t<W, GPL, 4, SEG>(a, lds, s);
    default: return lds_t<W, GPL, 8, SEG>(a, lds, s);
  }
}

template <int SMAX>
void lean_t(LeanKind kind, const KArgs& a, int jw, int64_t blocks, int waves, size_t lds, hipStream_t s) {
  const dim3 grid((unsigned)blocks), block(64 * (unsigned)waves);
  switch (kind) {
    case LeanKind::kShared:
      hipLaunchKernelGGL((as_dev::shared_kernel<AS_W, SMAX, false, false>), grid, block, lds, s, a, jw);
      break;
    case LeanKind::kScales:  // (64 lanes hold one job)
      hipLaunchKernelGGL((as_dev::shared_kernel<AS_W, SMAX, false, AS_W < 64>), grid, block, lds, s, a, jw);
      break;
    case LeanKind::kStats:
      hipLaunchKernelGGL((as_dev::shared_kernel<AS_W, SMAX, true, false>), grid, block, lds, s, a, jw);
      break;
    default: hipLaunchKernelGGL((as_dev::seg_kernel<AS_W, SMAX>), grid, block, lds, s, a); break;
  }
}

}  // namespace

template <int W>
hipError_t launch_lds(int gpl, int smax, bool seg, const KArgs& a, size_t lds, hipStream_t s) {
  switch (gpl) {
    case 1: return seg ? lds_s<W, 1, true>(smax, a, lds, s) : lds_s<W, 1, false>(smax, a, lds, s);
    case 2: return seg ? lds_s<W, 2, true>(smax, a, lds, s) : lds_s<W, 2, false>(smax, a, lds, s);
    default: return seg ? lds_s<W, 4, true>(smax, a, lds, s) : lds_s<W, 4, false>(smax, a, lds, s);
  }
}

template <int W>
hipError_t launch_lean(LeanKind kind, int smax, const KArgs& a, int jw, int64_t blocks, int waves, size_t lds,
                       hipStream_t s) {
  switch (smax) {
    case 1: lean_t<1>(kind, a, jw, blocks, waves, lds, s); break;
    case 2: lean_t<2>(kind, a, jw, blocks, waves, lds, s); break;
    case 4: lean_t<4>(kind, a, jw, blocks, waves, lds, s); break;
    default: lean_t<8>(kind, a, jw, blocks, waves, lds, s); break;
  }
  return hipGetLastError();
}

#if AS_W >= 4
template <int W>
hipError_t launch_fix(int smax, const as_dev::SpecArgs& a, int q, int64_t blocks, size_t lds, hipStream_t s) {
  const dim3 grid((unsigned)blocks), block(64);
  switch (smax) {
    case 1: hipLaunchKernelGGL((as_dev::spec_fix<W, 1>), grid, block, lds, s, a, q); break;
    case 2: hipLaunchKernelGGL((as_dev::spec_fix<W, 2>), grid, block, lds, s, a, q); break;
    case 4: hipLaunchKernelGGL((as_dev::spec_fix<W, 4>), grid, block, lds, s, a, q); break;
    default: hipLaunchKernelGGL((as_dev::spec_fix<W, 8>), grid, block, lds, s, a, q); break;
  }
  return hipGetLastError();
}
template hipError_t launch_fix<AS_W>(int, const as_dev::SpecArgs&, int, int64_t, size_t, hipStream_t);
#endif

template hipError_t launch_lds<AS_W>(int, int, bool, const KArgs&, size_t, hipStream_t);
template hipError_t launch_lean<AS_W>(LeanKind, int, const KArgs&, int, int64_t, int, size_t, hipStream_t);

}  // namespace as_host
