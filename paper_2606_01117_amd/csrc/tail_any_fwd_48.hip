// Forward on scattered tiles for any group: the instantiations for up to 768 features.
#include "tail_any.hpp"

namespace haste {

hipError_t fwd_any_48(const TailArgs &a, const void *X, const int32_t *idx, const void *W, const float *bias, void *Y,
                      const int32_t *spos, int P, hipStream_t s) {
    const FaGeom g = fa_geom(a);
    return FaRun<48>{a, g, X, idx, W, bias, Y, spos, P, s}.run();
}

}  // namespace haste
