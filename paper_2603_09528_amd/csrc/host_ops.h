// Host-side building blocks of a plan: 1-D operators with boundary rows and
// the eigendecomposition of the symmetrised operator (§2.2.1).
#pragma once
#include <cstdint>
#include <string>
#include <vector>

namespace tpt {

enum Bc { BC_P = 0, BC_N = 1, BC_D = 2 };
enum Loc { LOC_C = 0, LOC_F = 1 };

// One-dimensional operator T of one direction: row i is
// a[i] u[i-1] + b[i] u[i] + c[i] u[i+1]; for a periodic direction a[0] couples
// to u[N-1] and c[N-1] to u[0] (the cyclic corners).  vol = diagonal of D.
struct Op1D {
    int n = 0;             // unknowns
    bool periodic = false;
    bool null_mode = false;  // T 1 = 0 (periodic, or Neumann-Neumann at cell centres)
    bool uniform = false;    // all control volumes and neighbour distances equal
    int bc_lo = BC_N, bc_hi = BC_N, loc = LOC_C;
    std::vector<double> a, b, c, vol;
    // The operator is its own mirror image (i -> n-1-i) up to the rounding of
    // the face coordinates: the same condition at both walls on faces
    // symmetric about the middle, or a uniform periodic direction.  exact:
    // to the last bit (of a uniform direction the volumes).
    bool mirror = false, mirror_exact = false;
};

// Returns an empty string on success, else the reason.
std::string build_op1d(int ncells, const double* faces, int bc_lo, int bc_hi, int loc, Op1D& op);

// Eigendecomposition of T~ = D^{1/2} T D^{-1/2}: lam[p], Qt[i*n + p] (column p
// is eigenvector p), orthonormal.  null_index = column of the exact null
// vector (lam = 0) or -1.  analytic = closed-form basis was used.
struct Eig1D {
    int n = 0;
    std::vector<double> lam, Qt;
    int null_index = -1;
    bool analytic = false;
};

std::string eig_op1d(const Op1D& op, Eig1D& e);

// A basis as products of half the size read it (fold_impl.h): h = (n + 1) / 2
// pairs of an even and an odd vector, slot a holding even mode 2a and odd mode
// 2a + 1 (even n) or 2a - 1 (odd n, whose slot 0 has no odd vector: then the
// modes that come in nearly degenerate pairs share a slot).  The vectors of a
// slot are eigenvectors v up to a rotation,
//   v_even = c e + s o,  v_odd = -s e + c o,  (c, s) = rot[a],
// that leaves e as symmetric and o as antisymmetric as possible.
// fwd / inv: [2][hp][kp] main parts, fwd[par][a][k] and inv[par][k][a]; xfwd /
// xinv: what is left, the antisymmetric part of e's row (par 0) and the
// symmetric part of o's (par 1) (forward; inverse: the symmetric part of o and
// the antisymmetric part of e).  The middle column of an odd n is halved in
// fwd.  All zero beyond h.
struct FoldBasis {
    int hp = 0, kp = 0;
    bool rotated = false;            // rot and xfwd / xinv are not trivial
    std::vector<double> fwd, inv, xfwd, xinv, rot;
    double sfwd = 1.0, sinv = 1.0;   // powers of two: the largest |xfwd| / sfwd, |xinv| / sinv in [0.5, 1)
};
// BF16 of a float (round to nearest even, infinities and NaN kept), and back.
uint16_t host_bf16(float x);
float host_bf16_to_f(uint16_t h);
// The remainders are held as two BF16 terms: x / s = hi + lo.
void fold_split(double x, double s, uint16_t& hi, uint16_t& lo);
// Whether the basis splits like this with xfwd, xinv small enough for the
// kernel's split of them (always for an exact mirror operator).
bool fold_basis(const Op1D& op, const Eig1D& e, int hp, int kp, FoldBasis& f);

}  // namespace tpt
