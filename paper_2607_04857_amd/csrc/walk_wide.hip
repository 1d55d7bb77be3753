// walk_wide.hip -- walk kernel of a lone instance on wide words: 16 columns per lane, three to a 64-bit word.
#include "walk.h"

namespace qk {

hipError_t launch_walk_wide(const WalkLaunch &w)
{
    if (w.n_inst != 1) return hipErrorInvalidValue;
    if (w.tier == 2) return launch_walk_tier<16, kWideLow, 2, kRowsWide>(w, TopkWalk{});
    if (w.tier != 3 || !w.tk || w.tk->k < 2) return hipErrorInvalidValue;
    return launch_walk_tier<16, kWideLow, 3, kRowsWide>(w, *w.tk);
}

}  // namespace qk
