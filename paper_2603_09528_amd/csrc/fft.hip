// Fast transforms for uniform directions.  On a uniform grid the eigenbases
// of §2.2.1 are known in closed form: the real Fourier basis (periodic), the
// cosine basis DCT-II (Neumann-Neumann, cell centres) and the sine basis
// DST-II (Dirichlet-Dirichlet, cell centres); §3 lets such a direction use
// FFT-based transforms in place of the dense eigenbasis product.
//
// Bases (orthonormal; the column order of the plan's analytic bases):
//   Fourier: column 0 = 1/sqrt(N); columns 2m-1, 2m (m = 1 .. N/2-1) =
//            sqrt(2/N) cos(2 pi m i/N), sqrt(2/N) sin(2 pi m i/N); column N-1
//            = (-1)^i / sqrt(N).
//   DCT-II:  column k = c_k cos(pi k (i + 1/2)/N), c_0 = sqrt(1/N), else sqrt(2/N).
//   DST-II:  column k-1 = c_k sin(pi k (i + 1/2)/N), k = 1..N, c_N = sqrt(1/N).
// Forward fhat = Q^{-1} f = sqrt(h) Q~^T f; inverse phi = Q phihat = Q~ phihat / sqrt(h).
//
// Each transform is one real length-N FFT (N a power of two) done as an
// N/2-point complex FFT of z_n = v_2n + i v_2n+1 in LDS, with the half
// spectrum V_m = (Z_m + conj Z_{M-m})/2 - i W^m (Z_m - conj Z_{M-m})/2
// (W = e^{-2 pi i/N}, M = N/2):
//   Fourier: v = f; the outputs are the real and imaginary parts of V_m.
//   DCT-II (Makhoul's reordering): v_n = f_2n, v_{N-1-n} = f_2n+1; then
//            X_k = Re(e^{-i pi k/2N} V_k) and X_{N-k} = -Im(e^{-i pi k/2N} V_k).
//   DST-II:  the DCT-II of (-1)^i f_i with the output order reversed, since
//            sin(pi k (2i+1)/2N) = (-1)^i cos(pi (N-k) (2i+1)/2N).
// The inverses run the same steps backwards: build the half spectrum, fold it
// into Z, inverse complex FFT (conjugate twiddles), unpack.  Arithmetic is
// FP64 whatever the storage types.
//
// Complex FFT of M = 2^m points: radix-2 decimation in time grouped into
// passes of up to three stages.  A thread holds the 8 points one pass
// combines in registers (the 2^q points base + k 2^h of a radix-2^q group,
// pre-multiplied by W_{2^(h+q)}^(b bitrev(k)), b = base mod 2^h, then q
// radix-2 stages with constant twiddles); the passes exchange points through
// LDS.  The first pass takes the natural-order input at stride M/2^q, which
// is where the bit-reversed order of the usual in-place algorithm puts a
// group, so no separate reordering is needed and the output comes out in
// natural order.  LDS positions are padded by one complex per sixteen, which
// keeps the power-of-two strides of the passes off a single bank, and lines
// are an odd number of points apart.
//
// Lines are either contiguous (x direction, element stride 1) or strided (y
// direction: the lines of one z slab are its Nx columns, element stride Nx).
// A block holds LPB lines, M/8 threads per line (one thread for M <= 8),
// 256 threads (128 for N = 2048, one line): 2048 complex points, 34 KB of LDS
// plus the twiddle tables (four blocks per CU at N = 256).  Eight points per
// thread rather than sixteen: the register and LDS footprint per thread then
// allows twice the resident waves, which the memory-bound pass needs more
// than the fewer LDS round trips of radix 16.  Loads and stores walk the lines so that
// consecutive lanes touch consecutive addresses: along a line for x (16-byte
// pairs), across lines for y.  The pass moves 16 B per unknown in FP64.
//
// Lines of 64 and more have kernels for their length and direction: with the
// length known only at run time half the time of a pass went into index
// arithmetic (84 vector instructions per 64 unknowns, 52 % of the cycles at
// 256^3) and the registers allowed four waves per SIMD; compiled for the
// length, addresses are one register and constant offsets, and LDS sets the
// occupancy.  256^3 periodic, FP64, us: x 68 -> 60 (with the check; 4.5 TB/s)
// and inverse 53 -> 47, y 65 -> 58 and 67 -> 49; x lines of 1024 (2.7e8
// unknowns) 1133 -> 965 and 1027 -> 872 (4.9 TB/s).
#include "fft_impl.h"

namespace tpt {

bool fft_supported(int n) { return n >= 8 && n <= 2048 && (n & (n - 1)) == 0; }

int fft_lines_per_block(int n) { return ut_lines_per_block(n); }

// y lines of 512 and more in blocks of 512 threads: 16, 8 and 4 lines a block in
// place of 8, 4 and 1, so the rows that a block reads and writes are 128, 64 and
// 32 bytes instead of 64, 32 and 8, and more waves fit a compute unit.  At
// 1024 x 1024 x 256 (FP64 DCT) 1297 -> 1099 us forward, 1277 -> 1137 inverse;
// FP32 1486 -> 1172; 512 x 2048 x 32, 375 -> 248; 256 x 512 x 128, 72 -> 64.
// Lines of 256 have 128-byte rows already (wider ones: 65 -> 68 us at 256^3).
// Only with two blocks for every compute unit: below that narrow ones spread
// further.
int fft_wide(const FftDesc& d) {
    return d.ylines && d.n >= 512 && d.lines >= 2LL * 256 * ut_lines_per_block(d.n, true);
}

long long fft_blocks(const FftDesc& d) {
    const int lpb = ut_lines_per_block(d.n, d.wide);
    return (d.lines + lpb - 1) / lpb;
}

hipError_t launch_fft(const FftDesc& d, long long blocks, hipStream_t s) {
    return launch_ut<false>(d, nullptr, 0, blocks, s);
}

}  // namespace tpt
