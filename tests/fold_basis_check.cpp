// How far the half-size products' basis is from the eigenvectors: for each grid
// on the command line (cells, stretching, lower end, length, condition 1 N 2 D
// 0 periodic, location), the largest 2-norm over the vectors of what the device
// holds less the vector, forward and inverse, in units of 2^-53, and whether
// remainders are applied.  In long double.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "host_ops.h"

using namespace tpt;
typedef long double real;

static double held(double x, double s) {
    uint16_t hi, lo;
    fold_split(x, s, hi, lo);
    return ((double)host_bf16_to_f(hi) + (double)host_bf16_to_f(lo)) * s;
}

int main(int argc, char** argv) {
    for (int q = 1; q + 5 < argc; q += 6) {
        const int nc = std::atoi(argv[q]), bc = std::atoi(argv[q + 4]), loc = std::atoi(argv[q + 5]);
        const double beta = std::atof(argv[q + 1]), lo = std::atof(argv[q + 2]), len = std::atof(argv[q + 3]);
        std::vector<double> x(nc + 1);
        for (int i = 0; i <= nc; ++i) {
            const double xi = (double)i / nc;
            const double u = beta == 0.0 ? xi : 0.5 * (1.0 + std::tanh(beta * (xi - 0.5)) / std::tanh(0.5 * beta));
            x[i] = lo + len * (i == 0 ? 0.0 : i == nc ? 1.0 : u);
        }
        Op1D op;
        Eig1D e;
        FoldBasis f;
        if (!build_op1d(nc, x.data(), bc, bc, loc, op).empty() || !eig_op1d(op, e).empty()) return 1;
        const int n = op.n, h = (n + 1) / 2, odd = n & 1, hp = (h + 63) / 64 * 64, kp = (h + 15) / 16 * 16;
        if (!op.mirror || !fold_basis(op, e, hp, kp, f)) {
            std::printf("whole\n");
            continue;
        }
        const size_t half = (size_t)hp * kp;
        real worst = 0.0L;
        for (int a = 0; a < h; ++a) {
            // the pair of a slot as products with it give it, and the vectors
            // (periodic: of the same span, the cosine and sine about the middle)
            const int pe = 2 * a, po = odd ? 2 * a - 1 : 2 * a + 1;
            const real c = f.rot[2 * a], s = f.rot[2 * a + 1];
            for (int inv = 0; inv < 2; ++inv) {
                real d2[2] = {0.0L, 0.0L};
                for (int i = 0; i < n; ++i) {
                    const int k = i < h ? i : n - 1 - i;
                    const bool mid = 2 * k == n - 1;
                    const real sg = i < h ? 1.0L : -1.0L, sv = std::sqrt((real)op.vol[i]), w = inv ? 1.0L / sv : sv;
                    const size_t at = inv ? (size_t)k * kp + a : (size_t)a * kp + k;
                    // forward: e = P0 +- X0, o = +-P1 + X1; inverse: X0 belongs to o, X1 to e
                    const double xe = inv ? f.xinv[half + at] : f.xfwd[at], xo = inv ? f.xinv[at] : f.xfwd[half + at];
                    const double sc = inv ? f.sinv : f.sfwd;
                    const real he = (f.rotated ? held(xe, sc) : 0.0), ho = (f.rotated ? held(xo, sc) : 0.0);
                    const real p0 = (inv ? f.inv : f.fwd)[at], p1 = (inv ? f.inv : f.fwd)[half + at];
                    const real m = mid && !inv ? 2.0L : 1.0L;
                    const real ev = mid ? m * p0 : p0 + sg * he, ov = mid ? m * ho : sg * p1 + ho;
                    const real pi = 3.14159265358979323846264338327950288L;
                    real ve = e.Qt[(size_t)i * n + pe], vo = po >= 0 ? e.Qt[(size_t)i * n + po] : 0.0;
                    if (op.periodic) {
                        const int me = a, mo = (po + 1) / 2;
                        ve = std::sqrt((me == 0 ? 1.0L : 2.0L) / n) * std::cos(pi * (real)(((long long)me * (2 * i + 1)) % (2LL * n)) / n);
                        vo = po < 0 ? 0.0L
                                    : std::sqrt((2 * mo == n ? 1.0L : 2.0L) / n) *
                                          std::sin(pi * (real)(((long long)mo * (2 * i + 1)) % (2LL * n)) / n);
                    }
                    const real de = (c * ev + s * ov) / w - ve, dn = po >= 0 ? (-s * ev + c * ov) / w - vo : 0.0L;
                    d2[0] += de * de;
                    d2[1] += dn * dn;
                }
                worst = std::max(worst, std::sqrt(std::max(d2[0], d2[1])));
            }
        }
        std::printf("%.3f %d\n", (double)(worst * 9007199254740992.0L), f.rotated ? 1 : 0);
    }
    return 0;
}
