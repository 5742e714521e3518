// Eigenbasis transforms of a mirror-symmetric direction.  Included by the
// per-precision translation units.
//
// A direction with the same condition at both walls on faces that are
// symmetric about the middle (a tanh-stretched channel; every uniform
// periodic direction with the half-shifted Fourier basis) has eigenvectors
// that are even or odd under i -> N-1-i.  With H = ceil(N/2) slots of an even
// and an odd vector, the forward transform splits into two products of half
// the size,
//   even modes: E_a = sum_{k<H} P0[a][k] (f_k + f_{N-1-k}),
//   odd modes:  O_a = sum_{k<H} P1[a][k] (f_k - f_{N-1-k}),
// and the inverse joins two of them,
//   e_k = sum_{a<H} P0[k][a] E_a,  o_k = sum_{a<H} P1[k][a] O_a,
//   u_k = e_k + o_k,  u_{N-1-k} = e_k - o_k:
// half the multiplications of the dense product (2 N^2 per line becomes N^2),
// the field read and written once as before.  A line keeps its modes even ones
// first (position a; odd ones at N-H+a), so both halves are contiguous; the
// plan orders the eigenvalues to match.  For odd N slot 0 has no odd mode.
//
// Faces given as doubles are symmetric only up to the rounding of their
// coordinates, which near the walls is 1e-14 .. 1e-13 of a cell.  The vectors
// are then symmetric to about 1e-13 after a rotation within each slot (it
// undoes the mixing of pairs whose eigenvalues agree to that), and CORR adds
// what is left:
//   E += X0 (f_k - f_{N-1-k}),  O += X1 (f_k + f_{N-1-k}),  then the rotation,
// and the same, backwards, in the inverse.  X is at most 5e-12 of P, so two
// BF16 terms of it and of the data (16 bits each) leave 2^-55 of a vector:
// all four products of the terms of eight columns are one K = 32 BF16 product
// in FP32 accumulators, an eighth of the FP64 products' time.  Together P, X
// and the rotation are the dense basis to the rounding of a double (one term
// would leave 2e-16 .. 7e-15 on tanh grids); without X, errors of 1e-13 would
// be left where the dense product has 1e-15.
// FP32 sums hold fields of any size: a tile with a line whose largest value lies
// outside 2^-90 .. 2^100 is multiplied again, with the copies of such a line over
// a power of two (its largest exponent), so a scaled field has the scaled result.
// Whether and how is up to the line alone: every tile shape gives the same bits.
//
// P0, P1 are padded with zero rows and columns (rows to 64, row length to
// 16), so basis loads need no bounds and the K loop no tail, and stored by
// K step, [step][parity][row][columns of the step]: every block reads the same
// step at about the same time, and from rows N / 2 elements apart that would
// be a few of the L2's channels (448 x 320 x 288, x pass: 533 us by rows, 503 by steps); the data operand
// is read through buffer resources that end at its last line, so lines past
// it read zero.  Data rows past H in the last K step meet zero basis columns:
// forward and even inverse they belong to the same line (a NaN or an infinity
// there is in that line's sums already), odd inverse ones may not and are
// masked.
#pragma once
#include <type_traits>

#include "device_common.h"
#include "mfma_tile.h"

namespace tpt {

// LDS of one tile, double buffered.  A K step is BK = 64 bytes of elements;
// its columns k are kept in the order (k % 4, k / 4), so that the 16 bytes a
// lane reads are its operands of all the step's MFMAs (column 4 m + l / 16 of
// the m-th): P as [parity][PH][BK], the data as [parity][4][DN][BK / 4] (y
// lines) or [parity][DN][BK] (x lines), rows padded by 16 bytes.
// CORR keeps the remainders, [parity][PH][16], and the data's BF16 copies,
// [parity][DN][16], a row the high terms of the step's columns and then the low
// ones, the other way round in every second eight rows: sixteen rows' high (or
// low) terms, read together, then lie in different banks.
template <typename TM, bool Y, bool CORR, int PH, int DN> struct FoldLds {
    static constexpr int BK = 64 / (int)sizeof(TM), NK = BK / 4;
    static constexpr int PP = BK + NK;
    static constexpr int PD = Y ? DN * NK : BK + NK;
    static constexpr int P_HALF = PH * PP, D_HALF = (Y ? 4 : DN) * PD;
    static constexpr int BUF = 2 * (P_HALF + D_HALF);
    static constexpr int PB = 16, B_HALF = DN * PB, X_HALF = PH * PB;  // in bf16
    static constexpr int B_BUF = 2 * (B_HALF + X_HALF);
    static constexpr int TOTAL = 2 * BUF + (CORR ? 2 * B_BUF * 2 / (int)sizeof(TM) : 0);
};

// A tile: PH slots over DN lines.  A wave holds WP x WD of both parities: the
// inverse needs e and o of the same element, the rotation both modes of a
// slot, the remainders both halves of the data.
template <int PH, int DN, int WP, int WD> struct FoldCfg {
    static constexpr int WAVES_P = PH / WP, WAVES_D = DN / WD;
    static constexpr int NT = 64 * WAVES_P * WAVES_D;
    static constexpr int MP = WP / 16, MD = WD / 16;
    // waves per SIMD: two blocks of eight waves, three of four, or four and more
    static constexpr int WPE = PH == 32 && NT == 256 ? 3 : 4;
};

struct FoldTile {
    int prob;      // problem of the work list
    unsigned lb;   // tile within the problem
    unsigned d0;   // first line
    int p0;        // first slot
};

// Tile v of the list.  coarse[v / FOLD_COARSE]: the problem of the first tile of
// that group (a search by bisection would be a chain of loads for every tile).
template <bool MULTI, int PH, int DN>
__device__ __forceinline__ FoldTile fold_find(const FoldDesc* __restrict__ work, int nwork,
                                              const unsigned* __restrict__ coarse, unsigned v) {
    FoldTile t;
    t.prob = 0;
    if constexpr (MULTI) {
        t.prob = (int)coarse[v / FOLD_COARSE];
        while (t.prob + 1 < nwork && (unsigned)work[t.prob + 1].block_begin <= v) ++t.prob;
        v -= (unsigned)work[t.prob].block_begin;
    }
    t.lb = v;
    // the tiles of one set of lines are neighbours: they share its data in L2
    const unsigned tp = (unsigned)work[t.prob].tiles_p, td = v / tp;
    t.p0 = (int)(v - td * tp) * PH;
    t.d0 = td * DN;
    return t;
}

// The high word of |x|: orders doubles by size, in steps of 2^-20.
__device__ __forceinline__ unsigned fold_size(double x) {
    return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) & 0x7fffffffu;
}
// The power of two over which a line with this largest size has its remainders
// formed: below 2^100 FP32 sums don't overflow (the terms of X / xs are below
// one), above 2^-90 what underflows is 2^-36 of them.  (Zero has none; infinities
// and NaN are lost on the line anyway.)
__device__ __forceinline__ int fold_shift(unsigned m) {
    const bool in = m == 0 || m >= 0x7ff00000u || (m >= (1023u - 90) << 20 && m < (1023u + 100) << 20);
    return in ? 0 : (int)(m >> 20) - 1023;
}
// Offset in its row of the high (t = 0) or low (t = 1) terms.
__device__ __forceinline__ int fold_term(int row, int t) { return ((row >> 3) & 1) == t ? 0 : 8; }
__device__ __forceinline__ bf16x8 fold_frag(const uint16_t* p) { return __builtin_bit_cast(bf16x8, *(const u16x8*)p); }

// The FP32 MFMA leaves rows 4 g + r of a 16 x 16 result in lane group g (of
// 16 lanes), register r; the FP64 one rows g + 4 r.  Transposing (g, r) makes
// the two agree.
__device__ __forceinline__ f4 fold_transpose(f4 v) {
    uint32_t a[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = __float_as_uint(v[r]);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const auto t = __builtin_amdgcn_permlane32_swap(a[r], a[r + 2], false, false);
        a[r] = t[0];
        a[r + 2] = t[1];
    }
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const auto t = __builtin_amdgcn_permlane16_swap(a[r], a[r + 1], false, false);
        a[r] = t[0];
        a[r + 1] = t[1];
    }
    return (f4){__uint_as_float(a[0]), __uint_as_float(a[1]), __uint_as_float(a[2]), __uint_as_float(a[3])};
}

// Results of a wave: acc[0], acc[1] of slots p0 .. and lines l0 .. of the tile
// (FP32 and FP64 MFMA results; y lines: rows of the result are slots, its
// columns lines; x lines the other way round).  se, sx: sums of EPI_ACCUM_F64.
template <typename TM, typename TO, int EPI, bool Y, bool INV, int MP, int MD>
__device__ __forceinline__ void fold_store(const FoldDesc& g, const FoldTile& cur,
                                           const typename Mfma<TM>::acc (&acc)[2][MP][MD], int p0, int l0, int lr, int lg,
                                           double& se, double& sx) {
    typedef Mfma<TM> MM;
    constexpr int eo = (int)sizeof(TO);
    const int ho = g.n - g.h;       // position of odd slot 0
    const int odd = g.n & 1;        // slot 0 has no odd mode, row H-1 is its own mirror
    // two results of an element: positions p and ho + p (modes), or rows p
    // and n - 1 - p.  An offset past any buffer drops the store.
    constexpr unsigned NOWHERE = 0xffffffffu;
    const unsigned step = (unsigned)(Y ? g.inner : 1) * eo;   // between positions of a line
    const unsigned lstep = (unsigned)(Y ? 1 : g.n) * eo;      // between lines of the tile (y: of a slab)
    __amdgpu_buffer_rsrc_t rC;
    unsigned inner = 1, b0 = 0;
    if constexpr (Y) {
        inner = (unsigned)g.inner;
        b0 = cur.d0 / inner;
        const unsigned slab = inner * (unsigned)g.n;
        rC = buf_rsrc_n((TO*)g.out + (long long)b0 * slab, (long long)((unsigned)g.lines / inner - b0) * slab * eo);
    } else {
        rC = buf_rsrc_n((TO*)g.out + (long long)cur.d0 * g.n, (g.lines - cur.d0) * g.n * eo);
    }
    const int p00 = p0 + (Y ? MM::row(lg, 0) : lr);
    const unsigned l00 = cur.d0 + (unsigned)(l0 + (Y ? lr : MM::row(lg, 0)));
    const unsigned first = (unsigned)p00 * step;
    const unsigned second = INV ? (unsigned)(g.n - 1 - p00) * step : (unsigned)(p00 + ho) * step;
#pragma unroll
    for (int j = 0; j < MD; ++j) {
        unsigned lo = 0;  // offset of the line (y: the lane's; x: of its register 0)
        if constexpr (Y) {
            const unsigned c = l00 + (unsigned)(j * 16), b = c / inner;
            lo = ((b - b0) * inner * (unsigned)g.n + (c - b * inner)) * eo;
        } else {
            lo = (l00 - cur.d0 + (unsigned)(j * 16)) * lstep;
        }
#pragma unroll
        for (int i = 0; i < MP; ++i) {
            unsigned at[4][2];
            TM val[4][2];
            [[maybe_unused]] double old[4][2];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int dp = i * 16 + (Y ? MM::row(0, r) : 0);
                const unsigned dl = Y ? 0u : (unsigned)MM::row(0, r);
                const int p = p00 + dp;
                const bool ok = p < g.h && l00 + (unsigned)(j * 16) + dl < (unsigned)g.lines;
                const bool ok2 = ok && (INV ? p < ho : !(odd && p == 0));
                const unsigned base = lo + dl * lstep, ds = (unsigned)dp * step;
                at[r][0] = ok ? base + first + ds : NOWHERE;
                at[r][1] = ok2 ? base + (INV ? second - ds : second + ds) : NOWHERE;
                const TM e = acc[0][i][j][r], o = acc[1][i][j][r];
                val[r][0] = INV ? e + o : e;
                val[r][1] = INV ? e - o : o;
                if (EPI == EPI_ACCUM_F64 && !ok2) val[r][1] = (TM)0;  // not summed
            }
            if constexpr (EPI == EPI_ACCUM_F64) {
                // the eight reads of a register group together
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q) old[r][q] = BufIO<double>::ld(rC, at[r][q], 0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const double x = old[r][q] + (double)val[r][q];
                        BufIO<double>::st(x, rC, at[r][q], 0);
                        se += (double)val[r][q] * (double)val[r][q];
                        sx += x * x;
                    }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < 2; ++q) BufIO<TO>::st((TO)val[r][q], rC, at[r][q], 0);
            }
        }
    }
}

template <typename TM, typename TI, typename TO, int EPI, bool Y, bool INV, bool CORR, bool MULTI, int PH, int DN,
          int WP, int WD>
__device__ __forceinline__ void fold_tiles(const FoldDesc* __restrict__ work, int nwork,
                                           const unsigned* __restrict__ coarse, unsigned total, TM* smem,
                                           double* red, [[maybe_unused]] unsigned* lmax,
                                           unsigned block = blockIdx.x, unsigned blocks = gridDim.x) {
    typedef FoldLds<TM, Y, CORR, PH, DN> S;
    static_assert(!CORR || std::is_same<TM, double>::value, "remainders are for FP64");  // (BK = 8)
    typedef FoldCfg<PH, DN, WP, WD> C;
    typedef Mfma<TM> MM;
    constexpr int BK = S::BK, NT = C::NT, MP = C::MP, MD = C::MD;
    constexpr int NK = S::NK;
    constexpr int LP = 2 * PH * 4 / NT > 0 ? 2 * PH * 4 / NT : 1, LD = DN * BK / NT;  // basis loads are 16 bytes
    typedef TM vec __attribute__((ext_vector_type(NK)));
    static_assert(sizeof(vec) == 16 && LD >= 1 && NT % BK == 0 && NT % DN == 0 && NT % (4 * PH) == 0, "tile too small for its threads");
    // (a single problem's descriptor stays in the kernel arguments)
    auto desc = [&](const FoldTile& t) -> const FoldDesc& { return MULTI ? work[t.prob] : *work; };
    constexpr int ei = (int)sizeof(TI), em = (int)sizeof(TM);
    const int tid = threadIdx.x;
    const int w = tid / 64, l = tid % 64, lr = l % 16, lg = l / 16;
    const int wd = w % C::WAVES_D, wp = w / C::WAVES_D;

    // A thread loads LP quarter rows of the basis, PROWS rows apart, and LD elements of
    // data, so it keeps one offset per operand and the rest is uniform (scalar
    // offsets) or immediate.  Data: consecutive rows of one column (y), one
    // column of lines XL apart (x), or (x, CORR) consecutive columns of a line.
    constexpr int PROWS = NT / 4;
    constexpr bool ACROSS = !Y && !CORR;
    constexpr int XL = NT / BK;
    const int prow = tid / 4 % (2 * PH), pcol = tid % 4;
    const int dline = Y ? tid % DN : ACROSS ? tid / BK : tid / (BK / LD);
    const int dk = Y ? tid / DN * LD : ACROSS ? tid % BK : tid % (BK / LD) * LD;
    constexpr int LK = ACROSS ? 1 : LD;  // consecutive columns
    // operands of a tile: basis and data resources, and the thread's offsets
    // of the basis, of the first values (rows k0 + dk .. of the line) and of
    // the second: their mirrors (forward) or the odd modes of slots k0 + dk ..
    // (inverse)
    struct Offs {
        unsigned p, d0, d1, x;
    };
    auto setup = [&](const FoldTile& t, __amdgpu_buffer_rsrc_t& rP, __amdgpu_buffer_rsrc_t& rD, Offs& o) {
        const FoldDesc& g = desc(t);
        rP = buf_rsrc(g.P);
        o.p = (unsigned)((((prow / PH) * g.hp + prow % PH) * BK + pcol * NK) * em);
        // remainders: a quarter row of both terms per thread
        if constexpr (CORR) o.x = (unsigned)((((prow / PH) * g.hp + prow % PH) * 2 * BK + pcol * 4) * 2);
        const int km = BK - LK - dk;  // the mirrors of rows dk .. dk + LK - 1, ascending
        if constexpr (Y) {
            // column c = slab * inner + i; offsets from the tile's first slab
            const unsigned inner = (unsigned)g.inner, b0 = t.d0 / inner;
            const unsigned c = t.d0 + (unsigned)dline, b = c / inner;
            const unsigned slab = inner * (unsigned)g.n;
            rD = buf_rsrc_n((const TI*)g.in + (long long)b0 * slab, (long long)((unsigned)g.lines / inner - b0) * slab * ei);
            const unsigned co = (b - b0) * slab + (c - b * inner);
            o.d0 = (co + (unsigned)dk * inner) * ei;
            o.d1 = INV ? o.d0 : (co + (unsigned)km * inner) * ei;
        } else {
            rD = buf_rsrc_n((const TI*)g.in + (long long)t.d0 * g.n, (g.lines - t.d0) * g.n * ei);
            o.d0 = (unsigned)(dline * g.n + dk) * ei;
            o.d1 = INV ? o.d0 : (unsigned)(dline * g.n + km) * ei;
        }
    };
    vec rp[LP];
    TI r0[LD], r1[LD];
    [[maybe_unused]] double2 rr[CORR && INV ? LD : 1];
    [[maybe_unused]] u32x2_t rx = {0, 0};
    auto gload = [&](const FoldTile& t, __amdgpu_buffer_rsrc_t rP, __amdgpu_buffer_rsrc_t rD, const Offs& o, int k0) {
        const FoldDesc& g = desc(t);
        const unsigned sp = (unsigned)((k0 * 2 * g.hp + t.p0 * BK) * em);
#pragma unroll
        for (int q = 0; q < LP; ++q) {
            const unsigned row = (unsigned)(((q * PROWS / PH) * g.hp + (q * PROWS) % PH) * BK * em);
            rp[q] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(rP, (int)o.p, (int)(sp + row), 0));
        }
        const unsigned step = (unsigned)(Y ? g.inner : 1) * ei;
        const unsigned s0 = (unsigned)k0 * step, s1 = (unsigned)(INV ? g.n - g.h + k0 : g.n - BK - k0) * step;
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            const int m = INV || ACROSS ? q : LD - 1 - q;
            const unsigned qs = ACROSS ? (unsigned)(XL * g.n * ei) : step;
            r0[q] = BufIO<TI>::ld(rD, o.d0, s0 + (unsigned)q * qs);
            r1[q] = BufIO<TI>::ld(rD, o.d1, s1 + (unsigned)m * qs);
            const int k = k0 + dk + (ACROSS ? 0 : q);
            if (INV && k0 + BK > g.h) r1[q] = k < g.h ? r1[q] : (TI)0;
            if constexpr (CORR && INV) rr[q] = g.rot[k];
        }
        if constexpr (CORR) {
            const __amdgpu_buffer_rsrc_t rX = buf_rsrc(g.X);
            rx = __builtin_amdgcn_raw_buffer_load_b64(rX, (int)o.x, (int)((k0 * 2 * g.hp + t.p0 * BK) * 4), 0);
        }
    };
    [[maybe_unused]] unsigned mx = 0;  // size of the largest value stored of this thread's line
    [[maybe_unused]] int sh = 0;       // less the power of two of its copies
    auto sstore = [&](int buf) {
        TM* P = smem + buf * S::BUF + prow * S::PP + pcol * NK;
        TM* D = smem + buf * S::BUF + 2 * S::P_HALF;
        if (NT <= 8 * PH || tid < 8 * PH) {
#pragma unroll
            for (int q = 0; q < LP; ++q) *(vec*)(P + q * PROWS * S::PP) = rp[q];
        }
        [[maybe_unused]] float c0[LD], c1[LD];
#pragma unroll
        for (int q = 0; q < LD; ++q) {
            const int k = dk + (ACROSS ? 0 : q), line = dline + (ACROSS ? q * XL : 0);
            const int o = Y ? (k % 4) * S::PD + line * NK + k / 4 : line * S::PD + (k % 4) * NK + k / 4;
            TM a, b;
            if constexpr (CORR && INV) {
                // (written as multiply-adds: the same bits in every tile shape)
                a = __builtin_fma(rr[q].x, (double)r0[q], -(rr[q].y * r1[q]));
                b = __builtin_fma(rr[q].x, (double)r1[q], rr[q].y * r0[q]);
            } else {
                a = INV ? (TM)r0[q] : (TM)(r0[q] + r1[q]);
                b = INV ? (TM)r1[q] : (TM)(r0[q] - r1[q]);
            }
            D[o] = a;
            D[S::D_HALF + o] = b;
            if constexpr (CORR) {
                c0[q] = (float)__builtin_ldexp(a, sh);
                c1[q] = (float)__builtin_ldexp(b, sh);
                mx = max(mx, max(fold_size(a), fold_size(b)));
            }
        }
        if constexpr (CORR) {
            uint16_t* C = (uint16_t*)(smem + 2 * S::BUF) + buf * S::B_BUF;
            uint16_t* B = C + dline * S::PB + dk + fold_term(dline, 0);
            uint16_t* D = C + dline * S::PB + dk + fold_term(dline, 1);
            if (NT == 8 * PH || tid < 8 * PH)
                *(u32x2_t*)(C + 2 * S::B_HALF + prow * S::PB + fold_term(prow, pcol >> 1) + (pcol & 1) * 4) = rx;
            uint32_t hi, lo;
            if constexpr (LD == 1) {
                split_bf16x2(c0[0], c1[0], hi, lo);
                B[0] = (uint16_t)hi;
                D[0] = (uint16_t)lo;
                B[S::B_HALF] = (uint16_t)(hi >> 16);
                D[S::B_HALF] = (uint16_t)(lo >> 16);
            } else {
#pragma unroll
                for (int q = 0; q < LD; q += 2) {
                    split_bf16x2(c0[q], c0[q + 1], hi, lo);
                    *(uint32_t*)(B + q) = hi;
                    *(uint32_t*)(D + q) = lo;
                    split_bf16x2(c1[q], c1[q + 1], hi, lo);
                    *(uint32_t*)(B + S::B_HALF + q) = hi;
                    *(uint32_t*)(D + S::B_HALF + q) = lo;
                }
            }
        }
    };

    const unsigned grid = blocks;
    unsigned v = block;
    if (v >= total) return;
    // (neighbouring tiles on one XCD)
    auto find = [&](unsigned b) {
        return fold_find<MULTI, PH, DN>(work, nwork, coarse, MULTI ? b : xcd_block32(b, total));
    };
    // The loader runs ahead of the products: a K step is loaded while the one
    // before it is staged and multiplied, across tile ends too, so a load has a
    // whole K step of MFMAs to arrive.
    unsigned lv = v;                     // tile of the next K step to load
    FoldTile lt = find(lv), cur = lt, nxt = lt, nxt2 = lt;  // the loader's, the one multiplied, the (up to) two after it
    int ahead = 0;
    int lk = 0, lnk = (desc(lt).h + BK - 1) / BK;
    __amdgpu_buffer_rsrc_t rP, rD;
    Offs off;
    setup(lt, rP, rD, off);
    [[maybe_unused]] int held = 0;       // K step (of its tile) in the registers
    auto load_next = [&]() {
        if (lk == lnk) {
            lk = 0;
            if (lv + grid < total) {
                lv += grid;
                lt = find(lv);
                lnk = (desc(lt).h + BK - 1) / BK;
                setup(lt, rP, rD, off);
                if (ahead == 0) nxt = lt;
                else nxt2 = lt;
                ++ahead;
            }  // else past the last tile: its K steps again, never used
        }
        held = lk;
        gload(lt, rP, rD, off, lk * BK);
        ++lk;
    };
    // the lines' sizes go to LDS with the last K step of their tile: three sets,
    // so that the next tile's may be written, and the one before's cleared,
    // while a tile's are read
    [[maybe_unused]] int ws = 0, rs = 0;
    [[maybe_unused]] bool again = false;  // the tile's second time
    auto next_set = [](int q) { return q == 2 * DN ? 0 : q + DN; };
    auto stage_held = [&](int buf) {
        sstore(buf);
        if (CORR && held + 1 == lnk) {
            atomicMax(lmax + ws + dline, mx);
            ws = next_set(ws);
        }
        load_next();
    };
    auto stage = [&](int buf) {
        if (CORR && held == 0) mx = sh = 0;  // the next tile's first
        stage_held(buf);
    };
    if constexpr (CORR) {
        for (int q = tid; q < 3 * DN; q += NT) lmax[q] = 0;
        __syncthreads();
    }
    load_next();
    int buf = 0;
    stage_held(0);
    __syncthreads();
    while (v < total) {
        const FoldDesc& g = desc(cur);
        const int nk = (g.h + BK - 1) / BK;
        typename MM::acc acc[2][MP][MD];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int i = 0; i < MP; ++i)
#pragma unroll
                for (int j = 0; j < MD; ++j) acc[q][i][j] = MM::zero();
        // remainders: FP32 accumulators
        [[maybe_unused]] f4 cacc[CORR ? 2 : 1][MP][MD];
        if constexpr (CORR) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < MP; ++i)
#pragma unroll
                    for (int j = 0; j < MD; ++j) cacc[q][i][j] = (f4){0.f, 0.f, 0.f, 0.f};
        }
        for (int kt = 0; kt < nk; ++kt) {
            const TM* P = smem + buf * S::BUF + (wp * WP + lr) * S::PP + lg * NK;
            const TM* D = smem + buf * S::BUF + 2 * S::P_HALF +
                          (Y ? lg * S::PD + (wd * WD + lr) * NK : (wd * WD + lr) * S::PD + lg * NK);
            vec fp[2][MP], fd[2][MD];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
#pragma unroll
                for (int i = 0; i < MP; ++i) fp[q][i] = *(const vec*)(P + (q * PH + i * 16) * S::PP);
#pragma unroll
                for (int j = 0; j < MD; ++j) fd[q][j] = *(const vec*)(D + q * S::D_HALF + j * 16 * (Y ? NK : S::PD));
            }
            auto multiply = [&](int kk) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int i = 0; i < MP; ++i)
#pragma unroll
                        for (int j = 0; j < MD; ++j)
                            acc[q][i][j] = Y ? MM::mma(fp[q][i][kk], fd[q][j][kk], acc[q][i][j])
                                             : MM::mma(fd[q][j][kk], fp[q][i][kk], acc[q][i][j]);
            };
#pragma unroll
            for (int kk = 0; kk < NK / 2; ++kk) multiply(kk);
            // the next K step goes to the other buffer between the two halves of
            // the MFMAs, so that the wait for its loads overlaps them, and the
            // loads of the one after it are issued
            stage(buf ^ 1);
#pragma unroll
            for (int kk = NK / 2; kk < NK; ++kk) multiply(kk);
            if constexpr (CORR) {
                // (moved up between the MFMAs above, their operands would spill)
                __builtin_amdgcn_sched_barrier(0);
                // K = 32: the columns by (high, low, high, low) terms of the
                // remainders and (high, high, low, low) ones of the data
                const uint16_t* C = (const uint16_t*)(smem + 2 * S::BUF) + buf * S::B_BUF;
                const uint16_t* B = C + (wd * WD + lr) * S::PB + fold_term(lr, lg >> 1);
                const uint16_t* X = C + 2 * S::B_HALF + (wp * WP + lr) * S::PB + fold_term(lr, lg & 1);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    bf16x8 xv[MP];
#pragma unroll
                    for (int i = 0; i < MP; ++i) xv[i] = fold_frag(X + (1 - q) * S::X_HALF + i * 16 * S::PB);
#pragma unroll
                    for (int j = 0; j < MD; ++j) {
                        const bf16x8 dv = fold_frag(B + q * S::B_HALF + j * 16 * S::PB);
#pragma unroll
                        for (int i = 0; i < MP; ++i)
                            cacc[1 - q][i][j] =
                                Y ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[i], dv, cacc[1 - q][i][j], 0, 0, 0)
                                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(dv, xv[i], cacc[1 - q][i][j], 0, 0, 0);
                    }
                }
            }
            if (kt + 1 < nk) {
                __syncthreads();
                buf ^= 1;
            }
        }
        double se = 0.0, sx = 0.0;
        if constexpr (CORR) {
            const double xs = g.xs;
            const double2* rot = g.rot + cur.p0 + wp * WP;
            constexpr int LR = Y ? 1 : 4;  // lines of a lane's results
            bool out = false;  // (the same answer in every wave)
#pragma unroll
            for (int q = 0; q < DN; q += 64) out = out || fold_shift(lmax[rs + q + l]) != 0;
            double f[MD][LR];
#pragma unroll
            for (int j = 0; j < MD; ++j)
#pragma unroll
                for (int r = 0; r < LR; ++r) f[j][r] = xs;
            if (__builtin_expect(__any(out) != 0, 0)) {
                if (!again) {
                    // back to the tile's first K step
                    __syncthreads();
                    again = true;
                    mx = 0;
                    sh = -fold_shift(lmax[rs + dline]);
                    if (tid < DN) lmax[next_set(rs) + tid] = 0;  // (the next tile may have been here)
                    ws = rs;
                    lv = v;
                    lt = cur;
                    lk = 0;
                    lnk = nk;
                    ahead = 0;
                    setup(lt, rP, rD, off);
                    load_next();
                    stage_held(buf);
                    __syncthreads();
                    continue;
                }
#pragma unroll
                for (int j = 0; j < MD; ++j)
#pragma unroll
                    for (int r = 0; r < LR; ++r)
                        f[j][r] = ldexp(xs, fold_shift(lmax[rs + wd * WD + j * 16 + (Y ? lr : MM::row(lg, r))]));
            }
#pragma unroll
            for (int i = 0; i < MP; ++i)
#pragma unroll
                for (int j = 0; j < MD; ++j)
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const f4 t = fold_transpose(cacc[q][i][j]);
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[q][i][j][r] += (double)t[r] * f[j][r % LR];
                    }
            if constexpr (!INV) {
                // from the slot's vectors to its eigenvectors
#pragma unroll
                for (int i = 0; i < MP; ++i)
#pragma unroll
                    for (int j = 0; j < MD; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const double2 cs = rot[i * 16 + (Y ? MM::row(lg, r) : lr)];
                            const double e = acc[0][i][j][r], o = acc[1][i][j][r];
                            acc[0][i][j][r] = __builtin_fma(cs.x, e, cs.y * o);
                            acc[1][i][j][r] = __builtin_fma(cs.x, o, -(cs.y * e));
                        }
            }
        }
        fold_store<TM, TO, EPI, Y, INV, MP, MD>(g, cur, acc, cur.p0 + wp * WP, wd * WD, lr, lg, se, sx);
        if constexpr (EPI == EPI_ACCUM_F64) {
            block_sum2<NT>(se, sx, red);
            if (threadIdx.x == 0) {
                g.partials[2 * cur.lb] = se;
                g.partials[2 * cur.lb + 1] = sx;
            }
        }
        __syncthreads();
        if constexpr (CORR) {
            if (tid < DN) lmax[rs + tid] = 0;  // (used again two tiles on)
            rs = next_set(rs);
            again = false;
        }
        buf ^= 1;
        cur = nxt;
        nxt = nxt2;
        --ahead;
        v += grid;
    }
}

// One problem (descriptor by value) or a work list.
#define TPT_FOLD_TEMPLATE \
    template <typename TM, typename TI, typename TO, int EPI, bool Y, bool INV, bool CORR, int PH, int DN, int WP, int WD>
#define TPT_FOLD_CFG FoldCfg<PH, DN, WP, WD>
TPT_FOLD_TEMPLATE
__global__ __launch_bounds__((TPT_FOLD_CFG::NT), (TPT_FOLD_CFG::WPE)) void fold_kernel(const FoldDesc g, unsigned total) {
    __shared__ __attribute__((aligned(16))) TM smem[FoldLds<TM, Y, CORR, PH, DN>::TOTAL];
    __shared__ double red[2 * (TPT_FOLD_CFG::NT / 64)];
    __shared__ unsigned lmax[CORR ? 3 * DN : 1];
    fold_tiles<TM, TI, TO, EPI, Y, INV, CORR, false, PH, DN, WP, WD>(&g, 1, nullptr, total, smem, red, lmax);
}
TPT_FOLD_TEMPLATE
__global__ __launch_bounds__((TPT_FOLD_CFG::NT), (TPT_FOLD_CFG::WPE)) void fold_multi_kernel(
    const FoldDesc* __restrict__ work, int nwork, const unsigned* __restrict__ coarse, unsigned total) {
    __shared__ __attribute__((aligned(16))) TM smem[FoldLds<TM, Y, CORR, PH, DN>::TOTAL];
    __shared__ double red[2 * (TPT_FOLD_CFG::NT / 64)];
    __shared__ unsigned lmax[CORR ? 3 * DN : 1];
    fold_tiles<TM, TI, TO, EPI, Y, INV, CORR, true, PH, DN, WP, WD>(work, nwork, coarse, total, smem, red, lmax);
}
#undef TPT_FOLD_TEMPLATE
#undef TPT_FOLD_CFG

template <typename TM, typename TI, typename TO, int EPI, bool Y, bool INV, bool CORR>
hipError_t launch_fold_typed(const FoldDesc& g, const FoldList* list, long long total, int shape, hipStream_t s) {
    if (total <= 0) return hipSuccess;
    if (total > 0x3fffffff || g.lines > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)fold_grid(g, shape, total));
#define TPT_FOLD(PH_, DN_, WP_, WD_)                                                                              \
    do {                                                                                                          \
        const dim3 nt(FoldCfg<PH_, DN_, WP_, WD_>::NT);                                                           \
        if (list)                                                                                                 \
            TPT_KLAUNCH((fold_multi_kernel<TM, TI, TO, EPI, Y, INV, CORR, PH_, DN_, WP_, WD_>), grid, nt, 0, s,   \
                        list->work, list->nwork, list->coarse, (unsigned)total);                                                   \
        else                                                                                                      \
            TPT_KLAUNCH((fold_kernel<TM, TI, TO, EPI, Y, INV, CORR, PH_, DN_, WP_, WD_>), grid, nt, 0, s, g,      \
                        (unsigned)total);                                                                         \
    } while (0)
    switch (shape) {
        case FOLD_64x128:
            if constexpr (CORR) TPT_FOLD(64, 64, 32, 16);
            else TPT_FOLD(64, 128, 32, 32);
            break;
        case FOLD_32x128:
            if constexpr (CORR) TPT_FOLD(32, 128, 32, 16);
            else TPT_FOLD(32, 128, 32, 32);
            break;
        case FOLD_16x64: TPT_FOLD(16, 64, 16, 16); break;
        default: return hipErrorInvalidValue;
    }
#undef TPT_FOLD
    return hipGetLastError();
}

}  // namespace tpt
