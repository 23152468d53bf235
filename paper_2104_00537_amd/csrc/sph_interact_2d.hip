// The 2-D variants of the interaction (see sph_gather.h).
#include "sph_gather.h"

namespace sph {

template hipError_t launch_gather<2>(const KParams&, int64_t, const sph_state&,
                                     const uint32_t*, const uint32_t*, float*, float*, float*,
                                     uint32_t*, uint32_t, const InteractScratch&, hipStream_t);

}  // namespace sph
