// One (d_in, d_out) instantiation of the fused kernel, every mode and both
// activations; compiled once per shape (MOT_FUSED_D_IN, MOT_FUSED_D_OUT set
// by the build) so the instantiations build in parallel.
#include "k_bf16_fused_kernel.h"

#define MOT_CAT3(a, b, c) a##b##_##c
#define MOT_LAUNCH_NAME(a, b) MOT_CAT3(launch_fused_, a, b)

namespace mot {

hipError_t MOT_LAUNCH_NAME(MOT_FUSED_D_IN, MOT_FUSED_D_OUT)(const Problem& p, const UnitTab& ut, bool routed,
                                                           hipStream_t stream) {
    if (routed) return launch_t<MOT_FUSED_D_IN, MOT_FUSED_D_OUT, kFusedRouted>(p, ut, stream);
    return p.sp.parts > 1 ? launch_t<MOT_FUSED_D_IN, MOT_FUSED_D_OUT, kFusedSplit>(p, ut, stream)
                          : launch_t<MOT_FUSED_D_IN, MOT_FUSED_D_OUT, kFusedDense>(p, ut, stream);
}

}  // namespace mot
