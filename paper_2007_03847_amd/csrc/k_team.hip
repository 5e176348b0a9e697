// k_team.hip -- the team integrator (k_team.hpp) as fmc_run launches it: a
// workgroup per tile of 16 trajectories, FP64 and FP32.
#include "k_team.hpp"
#include "k_variants.hpp"

namespace fmc {

// Registers: a CU's SIMDs take the waves of a workgroup rounded up to a multiple of
// four, so two teams of five to seven waves share a CU only at four waves per
// SIMD.  FP32 fits that with a few spills (37 machines, 2e4 samples: 19.4 -> 16.0 us
// per step, 256 tiles 3.85 -> 4.1); FP64 does not.
template <typename R, int NB>
__global__ void __launch_bounds__(64 * NB)
    __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 2 : NB > 4 ? 4 : 3))) k_rk4_team(IntegArgs<R> a, int NG) {
  __shared__ TeamLds<R, NB, 1> S;
  const int64_t tl = blockIdx.x;
  GroupStats st{reinterpret_cast<double2*>(a.partial) + tl * (a.S + 1) * a.V, 0};
  team_run<R, NB, 1>(a, NG, tl, S, st);
}

template <typename R>
hipError_t launch_team(const VariantInfo& v, const IntegArgs<R>& a, int64_t n_groups, hipStream_t st) {
  if (a.sde || v.PM != kTeamPM || a.n > v.NG || a.P > kTeamPM || a.P > 4 * v.WPB)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)n_groups), block((unsigned)(64 * v.WPB));
  switch (v.WPB) {
#define FMC_X(NGX, NBX)                                                                     \
  case NBX:                                                                                 \
    hipLaunchKernelGGL((k_rk4_team<R, NBX>), grid, block, 0, st, a, v.NG);                  \
    break;
    FMC_TEAM_VARIANTS(FMC_X)
#undef FMC_X
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
template hipError_t launch_team<double>(const VariantInfo&, const IntegArgs<double>&, int64_t, hipStream_t);
template hipError_t launch_team<float>(const VariantInfo&, const IntegArgs<float>&, int64_t, hipStream_t);

}  // namespace fmc
