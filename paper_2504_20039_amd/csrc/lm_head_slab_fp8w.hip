// Instantiations of the small-tile kernel for OCP FP8 E4M3 W_lm (bf16 hidden_t).
#include "lm_head_slab.h"

namespace aj {

hipError_t lm_head_slab_fp8w(const SlabTile &t, const LmHeadArgs &a, hipStream_t s)
{
    return a.M <= 0 ? hipSuccess : dispatch_slab<true>(t, a, s);
}

}  // namespace aj
