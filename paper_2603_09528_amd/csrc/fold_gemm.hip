// Half-size products and whole products of one transform stage of a batch in
// one launch.  Apart, each of the two launches leaves part of the device idle,
// and the second waits for the first.  Every block walks its share of the
// work list's tiles and then its share of the half-size products' (the blocks
// after those with one work-list tile more come first), so both kinds spread
// evenly whatever their sizes.  Tiles of four waves, as the work list's: 32 x 64
// with remainders (16 x 64 in its place: twelve problems of 29 to 100 cells 162
// us a batch against 155, twenty of 40 to 120 403 against 343), 32 x 128 or
// 16 x 64 without (FP32).
#include "fold_impl.h"
#include "gemm_impl.h"

namespace tpt {

template <typename TM, typename TI, typename TO, int EPI, bool Y, bool INV, bool CORR, int PH, int DN, int WP, int WD>
__global__ __launch_bounds__(256, 3) void fold_gemm_multi_kernel(const FoldDesc* __restrict__ fold, int nfold,
                                                              const unsigned* __restrict__ coarse, unsigned ftiles,
                                                              const GemmDesc* __restrict__ gemm, int ngemm,
                                                              long long gtiles) {
    static_assert(FoldCfg<PH, DN, WP, WD>::NT == 256, "one block size");
    typedef typename std::conditional<Y, TM, TI>::type TA;
    typedef typename std::conditional<Y, TI, TM>::type TB;
    constexpr int BM = Y ? 64 : 128, BN = Y ? 128 : 64;
    constexpr int LF = FoldLds<TM, Y, CORR, PH, DN>::TOTAL, LG = SmemF<TM, BM, BN, !Y, 16, 2>::TOTAL;
    __shared__ __attribute__((aligned(16))) TM smem[LF > LG ? LF : LG];
    __shared__ double red[2 * (256 / 64)];
    __shared__ unsigned lmax[CORR ? 3 * DN : 1];
    gemm_worklist_f<TM, TA, TB, TO, EPI, !Y, BM, BN>(gemm, ngemm, gtiles, smem, red);
    __syncthreads();
    const unsigned g = gridDim.x, first = (unsigned)(gtiles % g);
    fold_tiles<TM, TI, TO, EPI, Y, INV, CORR, true, PH, DN, WP, WD>(fold, nfold, coarse, ftiles, smem, red, lmax,
                                                                    (blockIdx.x + g - first) % g, g);
}

template <typename TM, typename TI, typename TO, int EPI, bool Y, bool INV, bool CORR>
static hipError_t launch_fg(const FoldList& list, long long ftiles, int shape, const GemmDesc* gemm, int ngemm,
                            long long gtiles, hipStream_t s) {
    // three blocks a compute unit, as the work-list kernel
    const dim3 grid((unsigned)std::min(ftiles + gtiles, 768LL));
#define TPT_FG(PH_, DN_, WP_, WD_)                                                                                   \
    TPT_KLAUNCH((fold_gemm_multi_kernel<TM, TI, TO, EPI, Y, INV, CORR, PH_, DN_, WP_, WD_>), grid, dim3(256), 0, s,  \
                list.work, list.nwork, list.coarse, (unsigned)ftiles, gemm, ngemm, gtiles)
    if constexpr (CORR) {
        if (shape != FOLD_32x128) return hipErrorInvalidValue;
        TPT_FG(32, 64, 32, 16);
    } else {
        if (shape == FOLD_16x64) TPT_FG(16, 64, 16, 16);
        else if (shape == FOLD_32x128) TPT_FG(32, 128, 32, 32);
        else return hipErrorInvalidValue;
    }
#undef TPT_FG
    return hipGetLastError();
}

hipError_t launch_fold_gemm(const FoldDesc& rep, const FoldList& list, long long ftiles, int shape, const GemmDesc* gemm,
                            int ngemm, long long gtiles, hipStream_t s) {
    if (ftiles <= 0 || gtiles <= 0 || ftiles > 0x3fffffff || rep.lines > 0x7fffffff) return hipErrorInvalidValue;
#define TPT_FG(TM, TI, TO, EPI, Y, INV, CORR) \
    return launch_fg<TM, TI, TO, EPI, Y, INV, CORR>(list, ftiles, shape, gemm, ngemm, gtiles, s)
    const bool i64 = rep.tin == DT_F64, o64 = rep.tout == DT_F64;
    if (rep.prec == GP_F64) {
        if (!i64 || !o64 || rep.epi != EPI_STORE) return hipErrorInvalidValue;
        if (rep.ylines) {
            if (rep.inverse) TPT_FG(double, double, double, EPI_STORE, true, true, true);
            TPT_FG(double, double, double, EPI_STORE, true, false, true);
        }
        if (rep.inverse) TPT_FG(double, double, double, EPI_STORE, false, true, true);
        TPT_FG(double, double, double, EPI_STORE, false, false, true);
    }
    if (rep.prec != GP_F32) return hipErrorInvalidValue;
    if (rep.ylines) {
        if (i64 || o64 || rep.epi != EPI_STORE) return hipErrorInvalidValue;
        if (rep.inverse) TPT_FG(float, float, float, EPI_STORE, true, true, false);
        TPT_FG(float, float, float, EPI_STORE, true, false, false);
    }
    if (!rep.inverse) {
        if (o64 || rep.epi != EPI_STORE) return hipErrorInvalidValue;
        if (i64) TPT_FG(float, double, float, EPI_STORE, false, false, false);
        TPT_FG(float, float, float, EPI_STORE, false, false, false);
    }
    if (i64 || !o64) return hipErrorInvalidValue;
    if (rep.epi == EPI_ACCUM_F64) TPT_FG(float, float, double, EPI_ACCUM_F64, false, true, false);
    TPT_FG(float, float, double, EPI_STORE, false, true, false);
#undef TPT_FG
}

}  // namespace tpt
