// Instantiations of the small-tile kernel for bf16 W_lm.
#include "lm_head_slab.h"

namespace aj {

hipError_t lm_head_slab_bf16(const SlabTile &t, const LmHeadArgs &a, hipStream_t s)
{
    return a.M <= 0 ? hipSuccess : dispatch_slab<false>(t, a, s);
}

}  // namespace aj
