// Split-BF16 x3 transforms of mirror-symmetric directions: the half-size
// products of fold_impl.h with every operand x = hi + lo and three BF16
// products (lo hi, hi lo, hi hi, FP32 accumulation), as gemm_tile_b does for
// whole bases.  The bases arrive split; the sums and differences of the data
// are split on their way to LDS.
//
// Bound by memory and LDS: two planes of two halves of both operands make 60 KB
// a K step of 32, single buffered (the next step waits in registers), two
// blocks of eight waves a CU.  Half the dense product's K steps, the data still
// loaded once a tile.  At 448 x 384 x 256, dense and now, us a pass: x forward
// 185 and 160 (3.3 TB/s), x inverse with the sum onto the solution 309 and 185,
// y 157 and 103, inverse 136 and 90 (3.9 TB/s).
#include <algorithm>

#include "fold_impl.h"

namespace tpt {

template <int PH, int DN> struct FoldLdsB {
    static constexpr int BK = 32, PR = BK + 8;                 // row stride (16-byte padding)
    static constexpr int P_PL = PH * PR, D_PL = DN * PR;       // one plane of one parity
    static constexpr int TOTAL = 4 * (P_PL + D_PL);            // [parity][hi, lo]
};

template <typename TI, typename TO, int EPI, bool Y, bool INV, bool MULTI, int PH, int DN, int WP, int WD>
__device__ __forceinline__ void fold_tiles_b(const FoldDesc* __restrict__ work, int nwork,
                                             const unsigned* __restrict__ coarse, unsigned total, uint16_t* smem,
                                             double* red) {
    typedef FoldLdsB<PH, DN> S;
    constexpr int BK = S::BK, PR = S::PR, NT = 4 * DN, MP = WP / 16, MD = WD / 16;
    constexpr int LP = 2 * 2 * PH * 4 / NT;  // 16-byte pieces of the basis planes per thread
    static_assert(NT == 64 * (PH / WP) * (DN / WD) && LP * NT == 16 * PH, "tile and threads do not match");
    constexpr int ei = (int)sizeof(TI);
    auto desc = [&](const FoldTile& t) -> const FoldDesc& { return MULTI ? work[t.prob] : *work; };
    const int tid = threadIdx.x;
    const int w = tid / 64, l = tid % 64, lr = l % 16, lg = l / 16;
    const int wd = w % (DN / WD), wp = w / (DN / WD);
    // a thread's data: columns dk .. dk + 7 of one line
    const int line = Y ? tid % DN : tid / 4, dk = (Y ? tid / DN : tid % 4) * 8;
    const int prow = tid / 4 % PH, pc = tid % 4 * 8, pp = tid / (4 * PH);  // basis piece: row, columns, parity and plane

    struct Offs {
        unsigned p, d0, d1;
    };
    auto setup = [&](const FoldTile& t, __amdgpu_buffer_rsrc_t& rP, __amdgpu_buffer_rsrc_t& rD, Offs& o) {
        const FoldDesc& g = desc(t);
        rP = buf_rsrc(g.P);
        o.p = (unsigned)(((pp * g.hp + prow) * BK + pc) * 2);
        if constexpr (Y) {
            const unsigned inner = (unsigned)g.inner, b0 = t.d0 / inner;
            const unsigned c = t.d0 + (unsigned)line, b = c / inner, slab = inner * (unsigned)g.n;
            rD = buf_rsrc_n((const TI*)g.in + (long long)b0 * slab,
                            (long long)((unsigned)g.lines / inner - b0) * slab * ei);
            const unsigned co = (b - b0) * slab + (c - b * inner);
            o.d0 = (co + (unsigned)dk * inner) * ei;
            o.d1 = INV ? o.d0 : (co + (unsigned)(BK - 8 - dk) * inner) * ei;
        } else {
            rD = buf_rsrc_n((const TI*)g.in + (long long)t.d0 * g.n, (g.lines - t.d0) * g.n * ei);
            o.d0 = (unsigned)(line * g.n + dk) * ei;
            o.d1 = INV ? o.d0 : (unsigned)(line * g.n + BK - 8 - dk) * ei;
        }
    };
    // [column of the step][first value, second value] as fold_tiles: row k0 + r
    // of the line and its mirror, or the even and the odd mode of slot k0 + r
    TI r0[8], r1[8];
    u32x4_t rp[LP];
    auto load8 = [&](TI (&v)[8], __amdgpu_buffer_rsrc_t r, unsigned off, unsigned so, unsigned step, bool wide) {
        if (!Y && wide) {
#pragma unroll
            for (int e = 0; e < 8; e += 16 / ei) {
                const u32x4_t q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(off + (unsigned)(e * ei)), (int)so, 0);
                typedef TI vec __attribute__((ext_vector_type(16 / sizeof(TI))));
                const vec x = __builtin_bit_cast(vec, q);
#pragma unroll
                for (int c = 0; c < 16 / ei; ++c) v[e + c] = x[c];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = BufIO<TI>::ld(r, Y ? off : off + (unsigned)(e * ei), Y ? so + e * step : so);
        }
    };
    auto gload = [&](const FoldTile& t, __amdgpu_buffer_rsrc_t rP, __amdgpu_buffer_rsrc_t rD, const Offs& o, int k0) {
        const FoldDesc& g = desc(t);
        const unsigned sp = (unsigned)((k0 * 4 * g.hp + t.p0 * BK) * 2);
#pragma unroll
        for (int q = 0; q < LP; ++q)
            rp[q] = __builtin_amdgcn_raw_buffer_load_b128(rP, (int)o.p, (int)(sp + (unsigned)(q * (4 / LP) * g.hp * BK * 2)), 0);
        const unsigned step = (unsigned)(Y ? g.inner : 1) * ei;
        const unsigned s0 = (unsigned)k0 * step, s1 = (unsigned)(INV ? g.n - g.h + k0 : g.n - BK - k0) * step;
        const bool tail = INV && k0 + BK > g.h;  // odd modes past the line's last: by elements, masked
        load8(r0, rD, o.d0, s0, step, true);
        load8(r1, rD, o.d1, s1, step, !tail);
        if (tail) {
#pragma unroll
            for (int e = 0; e < 8; ++e) r1[e] = k0 + dk + e < g.h ? r1[e] : (TI)0;
        }
    };
    uint16_t* const Ps = smem;
    uint16_t* const Ds = smem + 4 * S::P_PL;
    auto sstore = [&]() {
#pragma unroll
        for (int q = 0; q < LP; ++q) *(u32x4_t*)(Ps + (pp + q * (4 / LP)) * S::P_PL + prow * PR + pc) = rp[q];
        u32x4_t h[2], lo[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float a[2], b[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int i = 2 * e + c;
                a[c] = INV ? (float)r0[i] : (float)(r0[i] + r1[7 - i]);
                b[c] = INV ? (float)r1[i] : (float)(r0[i] - r1[7 - i]);
            }
            uint32_t hh, ll;
            split_bf16x2(a[0], a[1], hh, ll);
            h[0][e] = hh;
            lo[0][e] = ll;
            split_bf16x2(b[0], b[1], hh, ll);
            h[1][e] = hh;
            lo[1][e] = ll;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            *(u32x4_t*)(Ds + (2 * q) * S::D_PL + line * PR + dk) = h[q];
            *(u32x4_t*)(Ds + (2 * q + 1) * S::D_PL + line * PR + dk) = lo[q];
        }
    };

    const unsigned grid = gridDim.x;
    unsigned v = blockIdx.x;
    if (v >= total) return;
    auto find = [&](unsigned b) {
        return fold_find<MULTI, PH, DN>(work, nwork, coarse, MULTI ? b : xcd_block32(b, total));
    };
    unsigned lv = v;
    FoldTile lt = find(lv), cur = lt;  // the loader's tile is at most one ahead
    int lk = 0, lnk = (desc(lt).h + BK - 1) / BK;
    __amdgpu_buffer_rsrc_t rP, rD;
    Offs off;
    setup(lt, rP, rD, off);
    auto load_next = [&]() {
        if (lk == lnk) {
            lk = 0;
            if (lv + grid < total) {
                lv += grid;
                lt = find(lv);
                lnk = (desc(lt).h + BK - 1) / BK;
                setup(lt, rP, rD, off);
            }  // else past the last tile: its K steps again, never used
        }
        gload(lt, rP, rD, off, lk * BK);
        ++lk;
    };
    load_next();
    for (; v < total; v += grid) {
        const FoldDesc& g = desc(cur);
        const int nk = (g.h + BK - 1) / BK;
        f4 acc[2][MP][MD];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < MP; ++i)
#pragma unroll
                for (int j = 0; j < MD; ++j) acc[q][i][j] = (f4){0.f, 0.f, 0.f, 0.f};
        for (int kt = 0; kt < nk; ++kt) {
            __syncthreads();  // every wave is done with the step before
            sstore();
            __syncthreads();
            load_next();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                bf16x8 ph[MP], pl[MP], dh[MD], dl[MD];
                const uint16_t* P = Ps + 2 * q * S::P_PL + (wp * WP + lr) * PR + lg * 8;
                const uint16_t* D = Ds + 2 * q * S::D_PL + (wd * WD + lr) * PR + lg * 8;
#pragma unroll
                for (int i = 0; i < MP; ++i) {
                    ph[i] = __builtin_bit_cast(bf16x8, *(const u16x8*)(P + i * 16 * PR));
                    pl[i] = __builtin_bit_cast(bf16x8, *(const u16x8*)(P + S::P_PL + i * 16 * PR));
                }
#pragma unroll
                for (int j = 0; j < MD; ++j) {
                    dh[j] = __builtin_bit_cast(bf16x8, *(const u16x8*)(D + j * 16 * PR));
                    dl[j] = __builtin_bit_cast(bf16x8, *(const u16x8*)(D + S::D_PL + j * 16 * PR));
                }
                auto mul = [&](const bf16x8 (&a)[MP], const bf16x8 (&b)[MD]) {
#pragma unroll
                    for (int i = 0; i < MP; ++i)
#pragma unroll
                        for (int j = 0; j < MD; ++j)
                            acc[q][i][j] = Y ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[q][i][j], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[q][i][j], 0, 0, 0);
                };
                mul(pl, dh);  // small products first
                mul(ph, dl);
                mul(ph, dh);
            }
        }
        double se = 0.0, sx = 0.0;
        fold_store<float, TO, EPI, Y, INV, MP, MD>(g, cur, acc, cur.p0 + wp * WP, wd * WD, lr, lg, se, sx);
        if constexpr (EPI == EPI_ACCUM_F64) {
            block_sum2<NT>(se, sx, red);
            if (tid == 0) {
                g.partials[2 * cur.lb] = se;
                g.partials[2 * cur.lb + 1] = sx;
            }
        }
        cur = lt;
    }
}

#define TPT_FOLD_TEMPLATE template <typename TI, typename TO, int EPI, bool Y, bool INV, int PH, int DN, int WP, int WD>
TPT_FOLD_TEMPLATE
__global__ __launch_bounds__(4 * DN, 4) void fold_bf16_kernel(const FoldDesc g, unsigned total) {
    __shared__ __attribute__((aligned(16))) uint16_t smem[FoldLdsB<PH, DN>::TOTAL];
    __shared__ double red[2 * (4 * DN / 64)];
    fold_tiles_b<TI, TO, EPI, Y, INV, false, PH, DN, WP, WD>(&g, 1, nullptr, total, smem, red);
}
TPT_FOLD_TEMPLATE
__global__ __launch_bounds__(4 * DN, 4) void fold_bf16_multi_kernel(const FoldDesc* __restrict__ work, int nwork,
                                                                    const unsigned* __restrict__ coarse, unsigned total) {
    __shared__ __attribute__((aligned(16))) uint16_t smem[FoldLdsB<PH, DN>::TOTAL];
    __shared__ double red[2 * (4 * DN / 64)];
    fold_tiles_b<TI, TO, EPI, Y, INV, true, PH, DN, WP, WD>(work, nwork, coarse, total, smem, red);
}
#undef TPT_FOLD_TEMPLATE

template <typename TI, typename TO, int EPI, bool Y, bool INV>
static hipError_t launch_bf16(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    if (total <= 0) return hipSuccess;
    if (total > 0x3fffffff || g.lines > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)fold_grid(g, shape, total));
#define TPT_FOLD(PH_, DN_, WP_, WD_)                                                                                \
    do {                                                                                                            \
        if (list)                                                                                                   \
            TPT_KLAUNCH((fold_bf16_multi_kernel<TI, TO, EPI, Y, INV, PH_, DN_, WP_, WD_>), grid, dim3(4 * DN_), 0,  \
                        s, list->work, list->nwork, list->coarse, (unsigned)total);                                 \
        else                                                                                                        \
            TPT_KLAUNCH((fold_bf16_kernel<TI, TO, EPI, Y, INV, PH_, DN_, WP_, WD_>), grid, dim3(4 * DN_), 0, s, g, \
                        (unsigned)total);                                                                           \
    } while (0)
    if (shape == FOLD_64x128) TPT_FOLD(64, 128, 32, 32);
    else if (shape == FOLD_32x128) TPT_FOLD(32, 64, 32, 16);
    else return hipErrorInvalidValue;
#undef TPT_FOLD
    return hipGetLastError();
}

hipError_t launch_fold_bf16(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    if (g.ylines) {
        if (g.tin != DT_F32 || g.tout != DT_F32 || g.epi != EPI_STORE) return hipErrorInvalidValue;
        return g.inverse ? launch_bf16<float, float, EPI_STORE, true, true>(g, list, total, shape, s)
                         : launch_bf16<float, float, EPI_STORE, true, false>(g, list, total, shape, s);
    }
    if (!g.inverse) {
        if (g.tout != DT_F32 || g.epi != EPI_STORE) return hipErrorInvalidValue;
        return g.tin == DT_F64 ? launch_bf16<double, float, EPI_STORE, false, false>(g, list, total, shape, s)
                               : launch_bf16<float, float, EPI_STORE, false, false>(g, list, total, shape, s);
    }
    if (g.tin != DT_F32 || g.tout != DT_F64) return hipErrorInvalidValue;
    return g.epi == EPI_ACCUM_F64 ? launch_bf16<float, double, EPI_ACCUM_F64, false, true>(g, list, total, shape, s)
                                  : launch_bf16<float, double, EPI_STORE, false, true>(g, list, total, shape, s);
}

}  // namespace tpt
