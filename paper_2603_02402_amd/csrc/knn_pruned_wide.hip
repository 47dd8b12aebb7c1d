// The pruned screen with lists of 32 keys per contraction half.

#include <hip/hip_runtime.h>

#include "screen_split_grid.hpp"

namespace rsc {

template int scr::pruned_launch<32>(const PrunedArgs &, const char *, hipStream_t);

}  // namespace rsc
