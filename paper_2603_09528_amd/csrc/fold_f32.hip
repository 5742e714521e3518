// Instantiations of the FP32 transforms of mirror-symmetric directions (the
// mixed modes: FP64 input of the first x pass, FP64 output of the last).
#include <algorithm>

#include "fold_impl.h"

namespace tpt {

hipError_t launch_fold_f32(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    if (g.ylines) {
        if (g.tin != DT_F32 || g.tout != DT_F32 || g.epi != EPI_STORE) return hipErrorInvalidValue;
        return g.inverse
                   ? launch_fold_typed<float, float, float, EPI_STORE, true, true, false>(g, list, total, shape, s)
                   : launch_fold_typed<float, float, float, EPI_STORE, true, false, false>(g, list, total, shape, s);
    }
    if (!g.inverse) {
        if (g.tout != DT_F32 || g.epi != EPI_STORE) return hipErrorInvalidValue;
        return g.tin == DT_F64
                   ? launch_fold_typed<float, double, float, EPI_STORE, false, false, false>(g, list, total, shape, s)
                   : launch_fold_typed<float, float, float, EPI_STORE, false, false, false>(g, list, total, shape, s);
    }
    if (g.tin != DT_F32 || g.tout != DT_F64) return hipErrorInvalidValue;
    return g.epi == EPI_ACCUM_F64
               ? launch_fold_typed<float, float, double, EPI_ACCUM_F64, false, true, false>(g, list, total, shape, s)
               : launch_fold_typed<float, float, double, EPI_STORE, false, true, false>(g, list, total, shape, s);
}

}  // namespace tpt
