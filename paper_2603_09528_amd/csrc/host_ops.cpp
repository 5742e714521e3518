// 1-D operators and their eigendecomposition (host side of a plan).
//
// §2.2.1, Eq. poisson-fd2 / tridiagonal-coefficients: a_i = 1/(dx_i dx_{i-1/2}),
// c_i = 1/(dx_i dx_{i+1/2}), b_i = -(a_i + c_i), dx_i the control volume of
// unknown i and dx_{i+1/2} the distance to the next unknown.  Boundary rows
// (the paper leaves them unspecified) come from ghost values: a Neumann wall
// drops the wall coupling and keeps only the interior flux; a Dirichlet wall
// at a cell-centred direction mirrors the ghost (u_0 = -u_1 at distance dx_1),
// i.e. b_1 = -c_1 - 2/dx_1^2; face-located unknowns between Dirichlet walls
// are the interior faces with zero wall values; periodic directions close
// with the cyclic corners.  D T is symmetric (dx_i c_i = dx_{i+1} a_{i+1}), so
// T~ = D^{1/2} T D^{-1/2} is symmetric (Eq. reverse-similarity-transform).
#include "host_ops.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <numeric>

namespace tpt {

typedef long double real;

static bool nearly_equal(double x, double y, double tol) { return std::fabs(x - y) <= tol * std::fabs(y); }

std::string build_op1d(int ncells, const double* faces, int bc_lo, int bc_hi, int loc, Op1D& op) {
    if (ncells < 2) return "need at least 2 cells per direction";
    if (!faces) return "faces pointer is NULL";
    for (int i = 0; i < ncells; ++i)
        if (!(faces[i + 1] > faces[i])) return "faces must be strictly increasing";
    const bool per = bc_lo == BC_P;
    if (per != (bc_hi == BC_P)) return "periodic boundaries must be set on both sides";
    auto okbc = [](int b) { return b == BC_P || b == BC_N || b == BC_D; };
    if (!okbc(bc_lo) || !okbc(bc_hi)) return "unknown boundary condition";
    if (loc != LOC_C && loc != LOC_F) return "unknown location";
    std::vector<double> w(ncells);
    for (int i = 0; i < ncells; ++i) w[i] = faces[i + 1] - faces[i];
    op = Op1D();
    op.periodic = per;
    op.bc_lo = bc_lo;
    op.bc_hi = bc_hi;
    op.loc = loc;
    // dist_lo[i] = distance to unknown i-1, dist_hi[i] = distance to unknown i+1
    std::vector<double> vol, dlo, dhi;
    if (loc == LOC_C) {
        const int n = ncells;
        vol = w;
        dlo.resize(n);
        dhi.resize(n);
        for (int i = 0; i + 1 < n; ++i) {
            double d = 0.5 * (w[i] + w[i + 1]);  // centre-to-centre
            dhi[i] = d;
            dlo[i + 1] = d;
        }
        if (per) {
            dlo[0] = dhi[n - 1] = 0.5 * (w[0] + w[n - 1]);
        } else {
            dlo[0] = w[0];       // mirrored ghost at distance of one cell width
            dhi[n - 1] = w[n - 1];
        }
    } else {
        if (per) {
            const int n = ncells;  // unknown m on face x_{m+1} (x_n == x_0)
            vol.resize(n);
            dlo.resize(n);
            dhi.resize(n);
            for (int m = 0; m < n; ++m) {
                double wa = w[(m + 1) % n];
                vol[m] = 0.5 * (w[m] + wa);
                dlo[m] = w[m];
                dhi[m] = wa;
            }
        } else if (bc_lo == BC_D && bc_hi == BC_D) {
            const int n = ncells - 1;  // interior faces
            vol.resize(n);
            dlo.resize(n);
            dhi.resize(n);
            for (int m = 0; m < n; ++m) {
                vol[m] = 0.5 * (w[m] + w[m + 1]);
                dlo[m] = w[m];
                dhi[m] = w[m + 1];
            }
        } else {
            return "face-located unknowns need periodic or Dirichlet-Dirichlet walls";
        }
    }
    const int n = (int)vol.size();
    op.n = n;
    op.vol = vol;
    op.a.resize(n);
    op.b.resize(n);
    op.c.resize(n);
    for (int i = 0; i < n; ++i) {
        op.a[i] = 1.0 / (vol[i] * dlo[i]);
        op.c[i] = 1.0 / (vol[i] * dhi[i]);
        op.b[i] = -(op.a[i] + op.c[i]);
    }
    if (!per) {
        if (loc == LOC_C) {
            // lower wall
            if (bc_lo == BC_N) op.b[0] += op.a[0];
            else op.b[0] -= op.a[0];
            if (bc_hi == BC_N) op.b[n - 1] += op.c[n - 1];
            else op.b[n - 1] -= op.c[n - 1];
        }
        op.a[0] = 0.0;
        op.c[n - 1] = 0.0;
    }
    op.null_mode = per || (loc == LOC_C && bc_lo == BC_N && bc_hi == BC_N);
    // uniform: equal control volumes and equal neighbour distances
    bool uni = true;
    for (int i = 0; i < n && uni; ++i) {
        uni = nearly_equal(vol[i], vol[0], 1e-12) && nearly_equal(dlo[i], vol[0], 1e-12) &&
              nearly_equal(dhi[i], vol[0], 1e-12);
    }
    // a Dirichlet mirrored ghost at a cell-centred wall sits at distance dx_1: still uniform
    op.uniform = uni;
    if (per) {
        op.mirror = uni;
    } else if (bc_lo == bc_hi) {
        // twice the spacing of the doubles just above 1, times the largest
        // coordinate (a tanh-stretched grid has up to 1.3 times)
        const double tol = 2.0 * std::numeric_limits<double>::epsilon() *
                           std::max(std::fabs(faces[0]), std::fabs(faces[ncells]));
        op.mirror = true;
        for (int k = 1; k < ncells; ++k)
            if (!(std::fabs((faces[k] - faces[0]) - (faces[ncells] - faces[ncells - k])) <= tol)) op.mirror = false;
        op.mirror = op.mirror || uni;
    }
    // (the closed-form basis of a uniform direction is symmetric: its volumes
    // have to be, which faces like i / 383 leave to the rounding)
    op.mirror_exact = op.mirror;
    for (int i = 0; i < n && op.mirror_exact; ++i) {
        const int m = n - 1 - i;
        op.mirror_exact = vol[i] == vol[m] && (uni || (op.b[i] == op.b[m] && op.a[i] == op.c[m]));
    }
    return "";
}

// ---------------------------------------------------------------------------
// Analytic orthonormal eigenbases of the uniform operators (Fourier,
// cosine and sine bases; the modified wavenumbers are -(4/h^2) sin^2(theta)).
// ---------------------------------------------------------------------------
static bool analytic_basis(const Op1D& op, Eig1D& e) {
    if (!op.uniform) return false;
    const int n = op.n;
    const real h = op.vol[0];
    const real s4 = 4.0L / (h * h);
    e.n = n;
    e.lam.assign(n, 0.0);
    e.Qt.assign((size_t)n * n, 0.0);
    auto Q = [&](int i, int p) -> double& { return e.Qt[(size_t)i * n + p]; };
    const real pi = 3.14159265358979323846264338327950288L;
    if (op.periodic) {
        // real Fourier basis: p = 0 constant; pairs (cos, sin) of wavenumber m;
        // for even n the alternating vector.
        int p = 0;
        for (int i = 0; i < n; ++i) Q(i, 0) = (double)(1.0L / std::sqrt((real)n));
        e.lam[0] = 0.0;
        p = 1;
        for (int m = 1; 2 * m < n; ++m) {
            real th = pi * m / n;
            real lam = -s4 * std::sin(th) * std::sin(th);
            real nc = std::sqrt(2.0L / n);
            for (int i = 0; i < n; ++i) {
                real ang = 2.0L * pi * (real)(((long long)m * i) % n) / (real)n;
                Q(i, p) = (double)(nc * std::cos(ang));
                Q(i, p + 1) = (double)(nc * std::sin(ang));
            }
            e.lam[p] = e.lam[p + 1] = (double)lam;
            p += 2;
        }
        if (n % 2 == 0) {
            for (int i = 0; i < n; ++i) Q(i, p) = (double)(((i % 2) ? -1.0L : 1.0L) / std::sqrt((real)n));
            e.lam[p] = (double)(-s4);
            ++p;
        }
        e.null_index = 0;
        e.analytic = true;
        return true;
    }
    if (op.loc == LOC_C && op.bc_lo == BC_N && op.bc_hi == BC_N) {
        // cosine basis cos(pi k (i + 1/2) / n)
        for (int k = 0; k < n; ++k) {
            real nc = (k == 0) ? std::sqrt(1.0L / n) : std::sqrt(2.0L / n);
            // angle pi k (2i+1) / (2n), reduced exactly modulo 2 pi first
            for (int i = 0; i < n; ++i)
                Q(i, k) = (double)(nc * std::cos(pi * (real)(((long long)k * (2 * i + 1)) % (4LL * n)) / (2.0L * n)));
            real th = pi * k / (2.0L * n);
            e.lam[k] = (double)(-s4 * std::sin(th) * std::sin(th));
        }
        e.lam[0] = 0.0;
        e.null_index = 0;
        e.analytic = true;
        return true;
    }
    if (op.loc == LOC_C && op.bc_lo == BC_D && op.bc_hi == BC_D) {
        // sine basis sin(pi k (i + 1/2) / n), k = 1..n
        for (int k = 1; k <= n; ++k) {
            real nc = (k == n) ? std::sqrt(1.0L / n) : std::sqrt(2.0L / n);
            for (int i = 0; i < n; ++i)
                Q(i, k - 1) =
                    (double)(nc * std::sin(pi * (real)(((long long)k * (2 * i + 1)) % (4LL * n)) / (2.0L * n)));
            real th = pi * k / (2.0L * n);
            e.lam[k - 1] = (double)(-s4 * std::sin(th) * std::sin(th));
        }
        e.null_index = -1;
        e.analytic = true;
        return true;
    }
    if (op.loc == LOC_F && op.bc_lo == BC_D) {
        // interior faces of n+1 cells: sin(pi k (i + 1) / (n + 1)), k = 1..n
        const int m = n + 1;
        for (int k = 1; k <= n; ++k) {
            real nc = std::sqrt(2.0L / m);
            for (int i = 0; i < n; ++i)
                Q(i, k - 1) = (double)(nc * std::sin(pi * (real)(((long long)k * (i + 1)) % (2LL * m)) / m));
            real th = pi * k / (2.0L * m);
            e.lam[k - 1] = (double)(-s4 * std::sin(th) * std::sin(th));
        }
        e.null_index = -1;
        e.analytic = true;
        return true;
    }
    return false;  // mixed Neumann/Dirichlet: numerical
}

// ---------------------------------------------------------------------------
// Implicit QL for a symmetric tridiagonal matrix (Golub & Van Loan §8.3:
// implicit symmetric QR step with Wilkinson shift, run bottom-up).  The
// eigenvector matrix is kept column-major (one contiguous row per vector) so
// that each Givens rotation updates two contiguous arrays.
//
// The numerical eigensolvers run in 80-bit extended precision (long double)
// and round to double at the end: a double-precision eigensolver fixes an
// eigenvector only to about eps ||T|| / gap, i.e. 1e-12..1e-11 for the smooth
// low modes of a stretched operator with N ~ 10^2..10^3, and those modes carry
// the solution of a Poisson problem.
// ---------------------------------------------------------------------------
static bool tridiag_ql(int n, std::vector<real>& d, std::vector<real>& e, std::vector<real>& Zt) {
    if (n <= 1) return true;
    e.resize(n);
    e[n - 1] = 0.0L;
    const real eps = std::numeric_limits<real>::epsilon();
    for (int l = 0; l < n; ++l) {
        int iter = 0;
        for (;;) {
            // find the first negligible off-diagonal at or below l
            int m = l;
            for (; m < n - 1; ++m) {
                real dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
                if (std::fabs(e[m]) <= eps * dd) break;
            }
            if (m == l) break;
            if (++iter > 60) return false;
            // shift from the leading 2x2 block of the unreduced part (d[l], e[l], d[l+1])
            real g = (d[l + 1] - d[l]) / (2.0L * e[l]);
            real r = std::hypot(g, (real)1.0L);
            g = d[m] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
            real s = 1.0L, c = 1.0L, p = 0.0L;
            int i = m - 1;
            bool underflow = false;
            for (; i >= l; --i) {
                real f = s * e[i];
                real b = c * e[i];
                r = std::hypot(f, g);
                e[i + 1] = r;
                if (r == 0.0L) {  // deflation by underflow
                    d[i + 1] -= p;
                    e[m] = 0.0L;
                    underflow = true;
                    break;
                }
                s = f / r;
                c = g / r;
                g = d[i + 1] - p;
                r = (d[i] - g) * s + 2.0L * c * b;
                p = s * r;
                d[i + 1] = g + p;
                g = c * r - b;
                // rotate eigenvector columns i and i+1
                real* zi = &Zt[(size_t)i * n];
                real* zj = &Zt[(size_t)(i + 1) * n];
                for (int k = 0; k < n; ++k) {
                    real t = zj[k];
                    zj[k] = s * zi[k] + c * t;
                    zi[k] = c * zi[k] - s * t;
                }
            }
            if (underflow) continue;
            d[l] -= p;
            e[l] = g;
            e[m] = 0.0L;
        }
    }
    return true;
}

// Householder reduction to tridiagonal form (Golub & Van Loan §8.3.1):
// for k = 0..n-3 reflect A[k+1:, k] onto e_1, update the trailing block with
// the symmetric rank-2 form, accumulate Z = H_0 H_1 ... .  Zt is returned
// column-major (Zt[p*n + i] = Z[i][p]).
static void householder_tridiag(int n, std::vector<real> A, std::vector<real>& d, std::vector<real>& e,
                                std::vector<real>& Zt) {
    auto a = [&](int i, int j) -> real& { return A[(size_t)i * n + j]; };
    std::vector<real> Z((size_t)n * n, 0.0L);
    for (int i = 0; i < n; ++i) Z[(size_t)i * n + i] = 1.0L;
    std::vector<real> v(n), pv(n), wv(n);
    for (int k = 0; k + 2 < n; ++k) {
        const int m = n - k - 1;  // length of x = A[k+1:, k]
        real alpha = 0.0L;
        for (int i = 0; i < m; ++i) alpha += a(k + 1 + i, k) * a(k + 1 + i, k);
        alpha = std::sqrt(alpha);
        if (alpha == 0.0L) continue;
        real x0 = a(k + 1, k);
        real sgn = x0 >= 0 ? 1.0L : -1.0L;
        // v = x + sgn*alpha*e1, H = I - beta v v^T, beta = 2 / v^T v
        for (int i = 0; i < m; ++i) v[i] = a(k + 1 + i, k);
        v[0] += sgn * alpha;
        real vtv = 0.0L;
        for (int i = 0; i < m; ++i) vtv += v[i] * v[i];
        if (vtv == 0.0L) continue;
        real beta = 2.0L / vtv;
        // p = beta * A22 v
        for (int i = 0; i < m; ++i) {
            real sum = 0.0L;
            const real* row = &A[(size_t)(k + 1 + i) * n + (k + 1)];
            for (int j = 0; j < m; ++j) sum += row[j] * v[j];
            pv[i] = beta * sum;
        }
        real ptv = 0.0L;
        for (int i = 0; i < m; ++i) ptv += pv[i] * v[i];
        real kk = 0.5L * beta * ptv;
        for (int i = 0; i < m; ++i) wv[i] = pv[i] - kk * v[i];
        // A22 -= v w^T + w v^T
        for (int i = 0; i < m; ++i) {
            real* row = &A[(size_t)(k + 1 + i) * n + (k + 1)];
            for (int j = 0; j < m; ++j) row[j] -= v[i] * wv[j] + wv[i] * v[j];
        }
        // column k / row k below the diagonal become (-sgn*alpha, 0, ...)
        a(k + 1, k) = -sgn * alpha;
        a(k, k + 1) = -sgn * alpha;
        for (int i = 1; i < m; ++i) {
            a(k + 1 + i, k) = 0.0L;
            a(k, k + 1 + i) = 0.0L;
        }
        // Z <- Z H  (columns k+1..n-1)
        for (int r = 0; r < n; ++r) {
            real* zr = &Z[(size_t)r * n + (k + 1)];
            real sum = 0.0L;
            for (int j = 0; j < m; ++j) sum += zr[j] * v[j];
            sum *= beta;
            for (int j = 0; j < m; ++j) zr[j] -= sum * v[j];
        }
    }
    d.assign(n, 0.0L);
    e.assign(n, 0.0L);
    for (int i = 0; i < n; ++i) d[i] = a(i, i);
    for (int i = 0; i + 1 < n; ++i) e[i] = a(i + 1, i);
    Zt.assign((size_t)n * n, 0.0L);
    for (int i = 0; i < n; ++i)
        for (int p = 0; p < n; ++p) Zt[(size_t)p * n + i] = Z[(size_t)i * n + p];
}

// Numerical eigenbasis of an exactly mirror-symmetric wall-bounded operator.
// With H = ceil(n/2), the even vectors (x_0 .. x_{H-1}, mirrored) and the odd
// ones diagonalise two tridiagonal matrices of half the size: a quarter of the
// work of the full problem, and vectors that are even or odd exactly (the full
// QL leaves arbitrary mixtures of the pairs whose eigenvalues differ by less
// than its rounding, the wall-bound modes of a strongly stretched grid).
// Eigenvalues of the two interlace, even first, so vector p has parity p % 2.
static std::string mirror_eig(const Op1D& op, Eig1D& e) {
    const int n = op.n, h = (n + 1) / 2, ho = n - h;
    std::vector<real> s(n), d(h), off(h, 0.0L);
    for (int i = 0; i < n; ++i) s[i] = std::sqrt((real)op.vol[i]);
    for (int i = 0; i < h; ++i) d[i] = op.b[i];
    auto coup = [&](int i) { return std::sqrt((real)op.c[i] * (real)op.a[i + 1]); };  // of unknowns i and i + 1
    for (int i = 0; i + 1 < h; ++i) off[i] = coup(i);
    e.lam.assign(n, 0.0);
    e.Qt.assign((size_t)n * n, 0.0);
    const real rt = std::sqrt(0.5L);
    for (int par = 0; par < 2; ++par) {
        const int m = par ? ho : h;
        if (m == 0) continue;
        std::vector<real> dd(d.begin(), d.begin() + m), ee(off.begin(), off.begin() + m), Zt((size_t)m * m, 0.0L);
        for (int i = 0; i < m; ++i) Zt[(size_t)i * m + i] = 1.0L;
        if (n % 2 == 0) dd[m - 1] += par ? -coup(m - 1) : coup(m - 1);
        else if (!par && m > 1) ee[m - 2] *= std::sqrt(2.0L);  // the middle unknown is its own mirror
        if (!tridiag_ql(m, dd, ee, Zt)) return "QL eigensolver did not converge";
        std::vector<int> idx(m);
        std::iota(idx.begin(), idx.end(), 0);
        std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return dd[x] > dd[y]; });
        // the exact null vector D^{1/2} 1 in this half's coordinates
        std::vector<real> v0;
        if (op.null_mode && !par) {
            v0.resize(m);
            real q2 = 0.0L;
            for (int i = 0; i < m; ++i) {
                v0[i] = (2 * i == n - 1) ? s[i] : s[i] / rt;
                q2 += v0[i] * v0[i];
            }
            for (int i = 0; i < m; ++i) v0[i] /= std::sqrt(q2);
        }
        for (int q = 0; q < m; ++q) {
            const int p = 2 * q + par;
            real* z = &Zt[(size_t)idx[q] * m];
            real lam = dd[idx[q]];
            if (!v0.empty()) {
                if (q == 0) {
                    lam = 0.0L;
                    std::copy(v0.begin(), v0.end(), z);
                } else {
                    real dot = 0.0L, q2 = 0.0L;
                    for (int i = 0; i < m; ++i) dot += v0[i] * z[i];
                    for (int i = 0; i < m; ++i) {
                        z[i] -= dot * v0[i];
                        q2 += z[i] * z[i];
                    }
                    for (int i = 0; i < m; ++i) z[i] /= std::sqrt(q2);
                }
            }
            e.lam[p] = (double)lam;
            for (int i = 0; i < m; ++i) {
                if (2 * i == n - 1) {
                    e.Qt[(size_t)i * n + p] = (double)z[i];
                } else {
                    e.Qt[(size_t)i * n + p] = (double)(z[i] * rt);
                    e.Qt[(size_t)(n - 1 - i) * n + p] = (double)(par ? -z[i] * rt : z[i] * rt);
                }
            }
        }
    }
    if (op.null_mode) e.null_index = 0;
    return "";
}

bool fold_basis(const Op1D& op, const Eig1D& e, int hp, int kp, FoldBasis& f) {
    const int n = op.n, h = (n + 1) / 2, odd = n & 1;
    const size_t half = (size_t)hp * kp;
    f = FoldBasis();
    f.hp = hp;
    f.kp = kp;
    f.rotated = !op.mirror_exact;
    f.fwd.assign(2 * half, 0.0);
    f.inv.assign(2 * half, 0.0);
    f.xfwd.assign(2 * half, 0.0);
    f.xinv.assign(2 * half, 0.0);
    f.rot.assign(2 * (size_t)std::max(hp, kp), 0.0);
    for (size_t a = 0; 2 * a < f.rot.size(); ++a) f.rot[2 * a] = 1.0;
    std::vector<real> s(n), ve(n), vo(n);
    for (int i = 0; i < n; ++i) s[i] = std::sqrt((real)op.vol[i]);
    const real pi = 3.14159265358979323846264338327950288L;
    for (int a = 0; a < h; ++a) {
        const int pe = 2 * a, po = odd ? 2 * a - 1 : 2 * a + 1;  // po = -1: no odd vector in this slot
        for (int i = 0; i < n; ++i) {
            ve[i] = e.Qt[(size_t)i * n + pe];
            vo[i] = po >= 0 ? e.Qt[(size_t)i * n + po] : 0.0;
        }
        if (op.periodic) {
            // Fourier basis about the middle: with the angles at i + 1/2 every
            // cosine is even and every sine odd (mode 2m - 1 the sine, mode 2m
            // the cosine of wavenumber m; even n: the alternating vector, odd,
            // last)
            const int me = a, mo = (po + 1) / 2;
            const real ne = std::sqrt((me == 0 ? 1.0L : 2.0L) / n), no = std::sqrt((2 * mo == n ? 1.0L : 2.0L) / n);
            for (int i = 0; i < n; ++i) {
                ve[i] = ne * std::cos(pi * (real)(((long long)me * (2 * i + 1)) % (2LL * n)) / (real)n);
                vo[i] = po >= 0 ? no * std::sin(pi * (real)(((long long)mo * (2 * i + 1)) % (2LL * n)) / (real)n) : 0.0L;
            }
        }
        if (f.rotated && po >= 0) {
            // e = c v_even - s v_odd with the largest symmetric part
            real m11 = 0.0L, m12 = 0.0L, m22 = 0.0L;
            for (int i = 0; i < n; ++i) {
                const real x = 0.5L * (ve[i] + ve[n - 1 - i]), y = 0.5L * (vo[i] + vo[n - 1 - i]);
                m11 += x * x;
                m12 += x * y;
                m22 += y * y;
            }
            const real th = 0.5L * std::atan2(-2.0L * m12, m11 - m22), c = std::cos(th), sn = std::sin(th);
            f.rot[2 * a] = (double)c;
            f.rot[2 * a + 1] = (double)sn;
            for (int i = 0; i < n; ++i) {
                const real x = ve[i], y = vo[i];
                ve[i] = c * x - sn * y;
                vo[i] = sn * x + c * y;
            }
        }
        // what the symmetry of e and the antisymmetry of o leave
        real xe = 0.0L, xo = 0.0L;
        for (int k = 0; k < h; ++k) {
            const int m = n - 1 - k;
            const bool mid = m == k;
            const real fe = ve[k] * s[k], fm = ve[m] * s[m], oe = vo[k] * s[k], om = vo[m] * s[m];  // Q^{-1} = Q~^T D^{1/2}
            const real ie = ve[k] / s[k], im = ve[m] / s[m], je = vo[k] / s[k], jm = vo[m] / s[m];  // Q = D^{-1/2} Q~
            const size_t ak = (size_t)a * kp + k, ka = (size_t)k * kp + a;
            f.fwd[ak] = (double)((mid ? 0.25L : 0.5L) * (fe + fm));
            f.fwd[half + ak] = (double)(0.5L * (oe - om));
            f.inv[ka] = (double)(0.5L * (ie + im));
            f.inv[half + ka] = (double)(0.5L * (je - jm));
            if (!f.rotated) continue;
            const real re = std::max(std::fabs(fe - fm) / s[k], std::fabs(ie - im) * s[k]);
            const real ro = std::max(std::fabs(oe + om) / s[k], std::fabs(je + jm) * s[k]);
            xe += 0.5L * re * re;
            xo += (mid ? 0.25L : 0.5L) * ro * ro;
            f.xfwd[ak] = (double)(0.5L * (fe - fm));
            f.xfwd[half + ak] = (double)((mid ? 0.25L : 0.5L) * (oe + om));
            f.xinv[ka] = (double)(0.5L * (je + jm));
            f.xinv[half + ka] = (double)(0.5L * (ie - im));
        }
        // the kernel's two BF16 terms of remainders and data, 16 bits each, lose
        // 2^-17 of a remainder at most: of 5e-12 of the vector 2^-54.5, where
        // rounding the vector itself to doubles takes 2^-53
        if (!(xe <= 2.5e-23L && xo <= 2.5e-23L)) return false;
    }
    auto scale = [](const std::vector<double>& x) {
        double m = 0.0;
        for (double v : x) m = std::max(m, std::fabs(v));
        int e = 0;
        std::frexp(m, &e);
        return std::ldexp(1.0, e);
    };
    if (f.rotated) {
        f.sfwd = scale(f.xfwd);
        f.sinv = scale(f.xinv);
    }
    return true;
}

uint16_t host_bf16(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

float host_bf16_to_f(uint16_t h) {
    uint32_t u = ((uint32_t)h) << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

void fold_split(double x, double s, uint16_t& hi, uint16_t& lo) {
    hi = host_bf16((float)(x / s));
    lo = host_bf16((float)(x / s - (double)host_bf16_to_f(hi)));
}

std::string eig_op1d(const Op1D& op, Eig1D& e) {
    e = Eig1D();
    const int n = op.n;
    e.n = n;
    if (analytic_basis(op, e)) return "";
    if (op.mirror_exact && !op.periodic) return mirror_eig(op, e);
    std::vector<real> s(n);
    for (int i = 0; i < n; ++i) s[i] = std::sqrt((real)op.vol[i]);
    std::vector<real> d(n), off(n, 0.0L), Zt;
    for (int i = 0; i < n; ++i) d[i] = op.b[i];
    if (!op.periodic) {
        // symmetric tridiagonal T~: off-diagonal sqrt(c_i a_{i+1})
        for (int i = 0; i + 1 < n; ++i) off[i] = std::sqrt((real)op.c[i] * (real)op.a[i + 1]);
        Zt.assign((size_t)n * n, 0.0L);
        for (int i = 0; i < n; ++i) Zt[(size_t)i * n + i] = 1.0L;
    } else {
        // cyclic: dense T~ with corners, reduced by Householder first
        std::vector<real> A((size_t)n * n, 0.0L);
        auto put = [&](int i, int j, double v) { A[(size_t)i * n + j] += (real)v * s[i] / s[j]; };
        for (int i = 0; i < n; ++i) {
            put(i, i, op.b[i]);
            put(i, (i + n - 1) % n, op.a[i]);
            put(i, (i + 1) % n, op.c[i]);
        }
        for (int i = 0; i < n; ++i)
            for (int j = i + 1; j < n; ++j) {
                real m = 0.5L * (A[(size_t)i * n + j] + A[(size_t)j * n + i]);
                A[(size_t)i * n + j] = A[(size_t)j * n + i] = m;
            }
        householder_tridiag(n, A, d, off, Zt);
    }
    if (!tridiag_ql(n, d, off, Zt)) return "QL eigensolver did not converge";
    // order by eigenvalue, largest (0 for a null mode) first
    std::vector<int> idx(n);
    std::iota(idx.begin(), idx.end(), 0);
    std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return d[x] > d[y]; });
    std::vector<real> lam(n), Q((size_t)n * n);
    for (int p = 0; p < n; ++p) {
        lam[p] = d[idx[p]];
        const real* z = &Zt[(size_t)idx[p] * n];
        for (int i = 0; i < n; ++i) Q[(size_t)i * n + p] = z[i];
    }
    if (op.null_mode) {
        // exact null vector D^{1/2} 1 / ||D^{1/2} 1||, eigenvalue exactly 0; the
        // other vectors are made orthogonal to it
        int k0 = 0;
        for (int p = 1; p < n; ++p)
            if (std::fabs(lam[p]) < std::fabs(lam[k0])) k0 = p;
        real nrm = 0.0L;
        for (int i = 0; i < n; ++i) nrm += (real)op.vol[i];
        nrm = std::sqrt(nrm);
        std::vector<real> v0(n);
        for (int i = 0; i < n; ++i) v0[i] = s[i] / nrm;
        lam[k0] = 0.0L;
        for (int i = 0; i < n; ++i) Q[(size_t)i * n + k0] = v0[i];
        for (int p = 0; p < n; ++p) {
            if (p == k0) continue;
            real dot = 0.0L;
            for (int i = 0; i < n; ++i) dot += v0[i] * Q[(size_t)i * n + p];
            real q2 = 0.0L;
            for (int i = 0; i < n; ++i) {
                real& q = Q[(size_t)i * n + p];
                q -= dot * v0[i];
                q2 += q * q;
            }
            real inv = 1.0L / std::sqrt(q2);
            for (int i = 0; i < n; ++i) Q[(size_t)i * n + p] *= inv;
        }
        e.null_index = k0;
    }
    e.lam.resize(n);
    e.Qt.resize((size_t)n * n);
    for (int p = 0; p < n; ++p) e.lam[p] = (double)lam[p];
    for (size_t k = 0; k < (size_t)n * n; ++k) e.Qt[k] = (double)Q[k];
    return "";
}

}  // namespace tpt
