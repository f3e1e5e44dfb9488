// Explicit instantiations of the split members, one unit per number of multiplying waves (WPK_PART: 1, 2 or 4).
#include "wpk_split.h"

#ifndef WPK_PART
#error "compile with -DWPK_PART=<1, 2 or 4>"
#endif

namespace wpk {
template hipError_t launch_split<WPK_PART>(const IgemmArgs &, hipStream_t);
}  // namespace wpk
