// Fast transforms of several problems in one launch (see fft.hip).
#include "fft_impl.h"

namespace tpt {

hipError_t launch_fft_multi(const FftDesc& rep, const FftDesc* d_work, int nwork, long long blocks, hipStream_t s) {
    return launch_ut<true>(rep, d_work, nwork, blocks, s);
}

}  // namespace tpt
