// walk_g4.hip -- walk kernel of a lone instance: 16 columns per lane, Gray levels 0-3 (top-k: 0-2) in VGPRs, the next ones in LDS, one copy per block of four waves.
#include "walk.h"

namespace qk {

hipError_t launch_walk_g4(const WalkLaunch &w) { return launch_walk_g<16, kBlockLow, kRowsBlock>(w); }

int occupancy_walk_g4_topk(int tier)
{
    return tier == 3 ? occupancy_tier<16, kBlockLowTopk, 3, kRowsBlock>()
                     : occupancy_tier<16, kBlockLowTopk, 5, kRowsBlock>();
}

}  // namespace qk
