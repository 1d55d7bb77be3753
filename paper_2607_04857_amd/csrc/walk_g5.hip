// walk_g5.hip -- walk kernel variants: 16 columns per lane, Gray levels 0-4 in VGPRs or levels 0-2 in VGPRs with 3-4 in LDS.
#include "walk.h"

namespace qk {

hipError_t launch_walk_g5(bool lds, const WalkLaunch &w)
{
    return lds ? launch_walk_g<16, 5, kRowsWave>(w) : launch_walk_g<16, 5>(w);
}

int occupancy_walk_g5(bool lds, int tier)
{
    return lds ? occupancy_g<16, 5, kRowsWave>(tier) : occupancy_g<16, 5>(tier);
}

}  // namespace qk
