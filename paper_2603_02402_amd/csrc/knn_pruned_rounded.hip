// The pruned screen of the BF16 form: rows rounded to BF16, one FP16 part each,
// lists of 32 keys per contraction half.

#include <hip/hip_runtime.h>

#include "screen_split_grid.hpp"

namespace rsc {

int scr::rounded_launch(const PrunedArgs &a, const char *name, hipStream_t s) {
    switch (rounded_geom(a.s.d).tc) {
#define X(TC) \
    case TC: return pruned_launch_geom<0, TC, 32, true>(a, name, s);
        RSC_ROUNDED_CHUNKS(X)
#undef X
    }
    set_error("internal: no rounded screen for this dimension");
    return RSC_ERR_UNSUPPORTED;
}

}  // namespace rsc
