// Instantiations of the FP64 transforms of mirror-symmetric directions, and
// the choice of their tile.
#include <algorithm>

#include "fold_impl.h"

namespace tpt {

bool fold_fits(int n, int nx, bool ylines, int prec) {
    const long long hp = ((n + 1) / 2 + FOLD_ROWS - 1) / FOLD_ROWS * FOLD_ROWS;
    const long long kp = ((n + 1) / 2 + fold_cols(prec) - 1) / fold_cols(prec) * fold_cols(prec);
    const long long lim = 0x7fffff00LL / 8;
    // (a K step and its mirror image have to lie in the line)
    if (n < std::max((int)FOLD_MIN_N, prec == GP_BF16X3 ? 32 : 0) || 2 * hp * kp > lim) return false;
    // a tile's lines: 128 x lines, or columns of at most 128 / nx + 2 slabs
    return ylines ? (long long)nx * n * (128 / nx + 2) <= lim : 128LL * n <= lim;
}

static void fold_dims(const FoldDesc& g, int shape, int* ph, int* dn) {
    *ph = shape == FOLD_64x128 ? 64 : shape == FOLD_32x128 ? 32 : 16;
    if (g.prec == GP_BF16X3) *dn = shape == FOLD_64x128 ? 128 : 64;
    else *dn = shape == FOLD_16x64 || (shape == FOLD_64x128 && g.corr) ? 64 : 128;
}

long long fold_tiles(FoldDesc& g, int shape) {
    int ph, dn;
    fold_dims(g, shape, &ph, &dn);
    g.tiles_p = (g.h + ph - 1) / ph;
    return (long long)g.tiles_p * ((g.lines + dn - 1) / dn);
}

long long fold_gemm_tiles(FoldDesc& g, int shape) {
    int ph, dn;
    fold_dims(g, shape, &ph, &dn);
    if (shape == FOLD_32x128 && g.corr) dn = 64;
    g.tiles_p = (g.h + ph - 1) / ph;
    return (long long)g.tiles_p * ((g.lines + dn - 1) / dn);
}

static int fold_shapes(int prec) { return prec == GP_BF16X3 ? 2 : (int)FOLD_NSHAPE; }

long long fold_max_tiles(int n, long long lines, int prec) {
    FoldDesc g{};
    g.n = n;
    g.h = (n + 1) / 2;
    g.prec = prec;
    g.lines = lines;
    long long most = 0;
    for (int v = 0; v < fold_shapes(prec); ++v) most = std::max(most, fold_tiles(g, v));
    return most;
}

// Relative time of a launch of `tiles` tiles: what the compute unit with most
// tiles has to do, over the rate the shape reaches when it has enough.  The
// padding of h to whole tiles and the idle units of a last round are in the
// tile count.  Rates from 256^3, 448 x 320 x 288, 512 x 383 x 256 and 640 x 640
// x 64 (64 x 64, 32 x 128 and 16 x 64 with remainders: 39, 34 and 23 TFLOP/s
// useful forward, 37, 31 and 20 inverse; 64 x 128, 32 x 128 and 16 x 64 without:
// 46, 45 and 36).  Cases it decides, with remainders: 448 x 320 x 288, x inverse
// 559 us in 64 x 64 against 599 in 32 x 128, y forward 414 against 399; 192 x 160
// x 128, x lines, 33-35 us in 32 x 128 against 39; 64 x 48 x 64, 5-7 us in 16 x
// 64 against 7-11.  Without: 192 x 160 x 128, x lines, 26 against 38 us in
// 64 x 128.
// Split BF16, 64 x 128 and 32 x 64: 128^3, 6.3-9.4 and 5.7-7.7 us; 256 x 200 x 100,
// x 17-19 and 16-17, y 14 and 17.
static double fold_cost(const FoldDesc& g, int shape, long long tiles) {
    // without remainders, with (forward, inverse), split BF16
    static const double rate[4][FOLD_NSHAPE] = {{1.0, 0.97, 0.78}, {1.0, 0.89, 0.58}, {1.0, 0.83, 0.55}, {1.0, 0.7, 0.0}};
    int ph, dn;
    fold_dims(g, shape, &ph, &dn);
    return (double)((tiles + 255) / 256) * ph * dn / rate[g.prec == GP_BF16X3 ? 3 : g.corr ? 1 + g.inverse : 0][shape];
}

int fold_shape(const FoldDesc* g, int count) {
    int best = 0;
    double cost = 0.0;
    for (int v = 0; v < fold_shapes(g[0].prec); ++v) {
        long long tiles = 0;
        for (int i = 0; i < count; ++i) {
            FoldDesc t = g[i];
            tiles += fold_tiles(t, v);
        }
        const double c = fold_cost(g[0], v, tiles);
        if (v == 0 || c < cost) {
            best = v;
            cost = c;
        }
    }
    return best;
}

long long fold_grid(const FoldDesc& g, int shape, long long total) {
    long long percu = shape == FOLD_64x128 || (shape == FOLD_32x128 && g.corr) ? 2 : shape == FOLD_32x128 ? 3 : 5;
    if (g.prec == GP_BF16X3 && shape == FOLD_32x128) percu = 4;
    return std::min(total, 256 * percu);
}

std::vector<unsigned> fold_coarse(const std::vector<FoldDesc>& g, long long total) {
    std::vector<unsigned> c;
    size_t i = 0;
    for (long long v = 0; v < total; v += FOLD_COARSE) {
        while (i + 1 < g.size() && g[i + 1].block_begin <= v) ++i;
        c.push_back((unsigned)i);
    }
    return c;
}

static hipError_t launch_any(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    return g.prec == GP_F64   ? launch_fold_f64(g, list, total, shape, s)
           : g.prec == GP_F32 ? launch_fold_f32(g, list, total, shape, s)
                              : launch_fold_bf16(g, list, total, shape, s);
}

hipError_t launch_fold(FoldDesc g, hipStream_t s) {
    const int shape = fold_shape(&g, 1);
    const long long total = fold_tiles(g, shape);
    return launch_any(g, nullptr, total, shape, s);
}

hipError_t launch_fold_multi(const FoldDesc& rep, const FoldList& list, long long total, int shape, hipStream_t s) {
    return launch_any(rep, &list, total, shape, s);
}

template <bool CORR>
static hipError_t launch_f64(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    typedef double D;
    constexpr int E = EPI_STORE;
    if (g.ylines)
        return g.inverse ? launch_fold_typed<D, D, D, E, true, true, CORR>(g, list, total, shape, s)
                         : launch_fold_typed<D, D, D, E, true, false, CORR>(g, list, total, shape, s);
    return g.inverse ? launch_fold_typed<D, D, D, E, false, true, CORR>(g, list, total, shape, s)
                     : launch_fold_typed<D, D, D, E, false, false, CORR>(g, list, total, shape, s);
}

hipError_t launch_fold_f64(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    if (g.tin != DT_F64 || g.tout != DT_F64 || g.epi != EPI_STORE) return hipErrorInvalidValue;
    return g.corr ? launch_f64<true>(g, list, total, shape, s)
               : launch_f64<false>(g, list, total, shape, s);
}

}  // namespace tpt
