// k_team_batch.hip -- classes 3-9 of the persistent batched integrator: the
// FP32 team integrator (k_team.hpp) over work items of consecutive tiles, one
// persistent kernel per team size (a kernel's register and LDS footprint is that
// of its team).
//
// These replaced kernels with one wave per 16 trajectories that streamed Y from
// L2 at every stage (147 KB per wave and step at 48 machines, which bounded them).
// Per step of 2e4 samples: 50 machines 77 -> 23 us, 40 machines 41 -> 15, 24
// machines 24 -> 7.4, 16 machines 10.5 -> 3.6.  Sixteen uneven scenarios of 4 to 47
// machines: 414 -> 227 ms per call.
//
// Registers: scenario and item go to scalar registers (load_uniform) and the
// set-up's addresses are recomputed per tile (team_run), which takes the team of
// six from 256 registers and 211 spilled to 168 and 11, three waves per SIMD.  A
// SIMD takes the waves of a workgroup rounded up to four, so teams of five and six
// run in pairs (12 waves: 48 machines, 512 tiles 7.7 -> 6.4 us per step), teams of
// seven and eight at four waves per SIMD.
#include "k_team.hpp"

namespace fmc {

template <int NB, int TW>
__global__ void __launch_bounds__(64 * NB * TW)
    __attribute__((amdgpu_waves_per_eu(TW == 1 && NB > 4 ? 4 : 3))) k_rk4_persistent_team(BatchArgs b) {
  __shared__ TeamLds<float, NB, TW> S;
  __shared__ int s_item;
  for (;;) {
    __syncthreads();  // everyone has read the previous s_item
    if (threadIdx.x == 0) s_item = atomicAdd(b.head, 1);
    __syncthreads();
    const int q = __builtin_amdgcn_readfirstlane(s_item);
    if (q >= b.n_items) break;  // uniform over the workgroup
    const BatchItem it = load_uniform(b.items + b.order[q]);
    const IntegArgs<float> a = load_uniform(b.scen + it.scen);
    // the rows hold the chunk's steps s_begin..s_end
    double2* rows = it.rows - a.s_begin * a.V;
    for (int64_t t = it.tile0; t < it.tile1; ++t)
      team_run<float, NB, TW>(a, 8 * NB, t, S, GroupStats{rows, (t - it.tile0) * kTeamT * TW});
  }
}

template <int NB, int TW>
static int blocks_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_rk4_persistent_team<NB, TW>, 64 * NB * TW, 0) !=
      hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}

#define FMC_TEAMS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

int persistent_team_blocks_per_cu(int nb) {
#define FMC_X(NB) \
  if (nb == NB) return blocks_per_cu<NB, batch_teams(NB)>();
  FMC_TEAMS(FMC_X)
#undef FMC_X
  return 1;
}

hipError_t launch_persistent_team(int nb, const BatchArgs& b, int grid, hipStream_t st) {
#define FMC_X(NB)                                                                             \
  if (nb == NB) {                                                                             \
    constexpr int TW = batch_teams(NB);                                                       \
    hipLaunchKernelGGL((k_rk4_persistent_team<NB, TW>), dim3((unsigned)grid), dim3(64 * NB * TW), \
                       0, st, b);                                                             \
    return hipGetLastError();                                                                 \
  }
  FMC_TEAMS(FMC_X)
#undef FMC_X
  return hipErrorInvalidValue;
}

}  // namespace fmc
