// Backward-feature on scattered tiles for any group: the instantiations for 32 rows.
#include "tail_any.hpp"

namespace haste {

hipError_t bwd_x_any_2_12(const TailArgs &a, const int32_t *idx, const void *W, const void *dY, float *part,
                           size_t ws_bytes, hipStream_t s) {
    const AxGeom g = ax_geom(a, ws_bytes);
    return AxRun<2, 12>{a, g, idx, W, dY, part, s}.run();
}

}  // namespace haste
