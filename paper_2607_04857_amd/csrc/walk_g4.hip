// walk_g4.hip -- walk kernel of a lone instance: 16 columns per lane, Gray levels 0-3 in VGPRs, the next ones in LDS, one copy per block of four waves.
#include "walk.h"

namespace qk {

hipError_t launch_walk_g4(const WalkLaunch &w) { return launch_walk_g<16, 4, kRowsBlock>(w); }

}  // namespace qk
