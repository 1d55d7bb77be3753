// walk_g6.hip -- walk kernel variants: 16 columns per lane, Gray levels 0-5 in VGPRs or levels 0-2 and 5 in VGPRs with 3-4 in LDS.
#include "walk.h"

namespace qk {

hipError_t launch_walk_g6(bool lds, const WalkLaunch &w)
{
    return lds ? launch_walk_g<16, 6, kRowsWave>(w) : launch_walk_g<16, 6>(w);
}

int occupancy_walk_g6(bool lds, int tier)
{
    return lds ? occupancy_g<16, 6, kRowsWave>(tier) : occupancy_g<16, 6>(tier);
}

hipError_t launch_walk_pair(const WalkLaunch &a, const WalkLaunch &b)
{
    if (a.tier != 2 || b.tier != 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL((walk_pair_kernel<16, 6, kRowsWave>), dim3(a.waves), dim3(kWave),
                       (walk_lds_bytes<16, 6, kRowsWave>(4)), a.stream, a.insts, a.n_inst, a.claims,
                       a.counter, b.insts, b.n_inst, b.claims, b.counter, a.k);
    return hipGetLastError();
}

}  // namespace qk
