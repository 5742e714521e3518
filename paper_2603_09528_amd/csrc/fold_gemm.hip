// Half-size products and whole products of one FP64 transform stage of a batch
// of small problems in one launch.  Apart, each of the two launches leaves most
// of the device idle, and the second waits for the first: the four stages of
// twelve problems of 29 to 100 cells a direction took 129 us in eight launches,
// 110 in four.  The first blocks walk the tiles of the work list, which take
// longest, the others those of the half-size products (16 x 64, the shape with
// four waves, as the work-list tile has).
#include "fold_impl.h"
#include "gemm_impl.h"

namespace tpt {

template <bool Y, bool INV>
__global__ __launch_bounds__(256) void fold_gemm_multi_kernel(const FoldDesc* __restrict__ fold, int nfold,
                                                              const unsigned* __restrict__ coarse, unsigned ftiles,
                                                              unsigned fblocks, const GemmDesc* __restrict__ gemm,
                                                              int ngemm, long long gtiles) {
    constexpr int BM = Y ? 64 : 128, BN = Y ? 128 : 64;
    constexpr int LF = FoldLds<double, Y, true, 16, 64>::TOTAL, LG = SmemF<double, BM, BN, !Y, 16, 2>::TOTAL;
    __shared__ __attribute__((aligned(16))) double smem[LF > LG ? LF : LG];
    __shared__ double red[2 * (256 / 64)];
    __shared__ unsigned lmax[3 * 64];
    const unsigned gblocks = gridDim.x - fblocks;
    if (blockIdx.x < gblocks)
        gemm_worklist_f<double, double, double, double, EPI_STORE, !Y, BM, BN>(gemm, ngemm, gtiles, smem, red, blockIdx.x, gblocks);
    else
        fold_tiles<double, double, double, EPI_STORE, Y, INV, true, true, 16, 64, 16, 16>(fold, nfold, coarse, ftiles, smem, red, lmax,
                                                                                          blockIdx.x - gblocks, fblocks);
}

hipError_t launch_fold_gemm(const FoldDesc& rep, const FoldList& list, long long ftiles, const GemmDesc* gemm, int ngemm,
                            long long gtiles, hipStream_t s) {
    if (ftiles <= 0 || gtiles <= 0 || ftiles > 0x3fffffff || rep.lines > 0x7fffffff) return hipErrorInvalidValue;
    if (rep.tin != DT_F64 || rep.tout != DT_F64 || rep.epi != EPI_STORE) return hipErrorInvalidValue;
    // what the device holds at three blocks a compute unit, and as much again
    // to take the places of blocks that are done
    const unsigned fb = (unsigned)std::min(ftiles, 768LL), gb = (unsigned)std::min(gtiles, 384LL);
#define TPT_FG(Y, INV)                                                                                              \
    TPT_KLAUNCH((fold_gemm_multi_kernel<Y, INV>), dim3(fb + gb), dim3(256), 0, s, list.work, list.nwork, list.coarse, \
                (unsigned)ftiles, fb, gemm, ngemm, gtiles)
    if (rep.ylines) {
        if (rep.inverse) TPT_FG(true, true);
        else TPT_FG(true, false);
    } else {
        if (rep.inverse) TPT_FG(false, true);
        else TPT_FG(false, false);
    }
#undef TPT_FG
    return hipGetLastError();
}

}  // namespace tpt
