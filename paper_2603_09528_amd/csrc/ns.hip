// One Runge–Kutta substep of the incompressible Navier–Stokes solver on the
// staggered grid (§2.1, Eq. rk3): the explicit terms and the predictor, the
// Helmholtz solve of each velocity component, the pressure Poisson solve,
// the correction of the velocity and the update of the pressure.
//
// Per substep k (alpha_k, beta_k, gamma_k; c = gamma_k nu dt / 2):
//   E^k   = A u^k + nu L_E u^k                         (kept for substep k+1)
//   rhs   = u^k + dt (alpha_k E^k + beta_k E^{k-1} - gamma_k G P) + c L_I u^k
//   (I - c L_I) u* = rhs                               (u* = rhs if L_I = 0)
//   L Phi = D u* / (gamma_k dt),   u^{k+1} = u* - gamma_k dt G Phi
//   P    += Phi - c L_I Phi
// (the right-hand side folds the predictor u** and the -c L_I u^k of the
// Helmholtz equation into one expression).
//
// Advection A u = -div(u (x) u) in the symmetry-preserving finite-volume
// form (the paper states second order and semi-discrete kinetic-energy
// conservation): the control volume of a face unknown is the half cells on
// both sides of the face; through its faces the mass flux is the mean of
// the two normal velocities along the component's own direction and the
// cell-width weighted mean of the two transverse velocities elsewhere (the
// fluxes for which the volume's discrete continuity is the half-sum of its
// two cells'), and the transported velocity is the plain mean of the two
// neighbouring unknowns.  The operator is then skew-symmetric for a
// discretely divergence-free field.
//
// Velocity walls: no penetration (wall faces carry no normal velocity and
// are not stored) and no slip (tangential components vanish on the wall:
// the Dirichlet rows of the 1-D operators, face-located along the
// component's own direction).
//
// Memory-bound.  One kernel forms the explicit terms and right-hand sides of
// all three components: u, v, w, P and the three E^{k-1} are read and the E^k
// and the right-hand sides written once, 104 B per cell (80 B for k = 1; a
// kernel for each component moves 168).  512 x 256 x 256, no implicit
// diffusion: 1726 us a substep in three kernels, 877 in one (3.8 TB/s).  A
// thread marches one (i, j) column of cells through a chunk of z planes with
// the z neighbours in registers; x neighbours come from the lanes beside
// (as loads they took the first-level cache's time: 1146 us), y neighbours
// are cache hits of the adjacent rows.  The pressure update rides in the gradient
// update's pass (which reads Phi anyway): 16 B per cell more there, P read
// and written.
#include <algorithm>
#include <cmath>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "device_common.h"

#include "host_ops.h"
#include "internal.h"
#include "projection.h"

namespace tpt {

struct NsDesc {
    int N[3];                   // cells per direction
    int nf[3];                  // face unknowns per direction (N periodic, N - 1 walls)
    int per[3];
    const double* w[3];         // cell widths
    const double* h[3];         // face spacings: distance of the centres of cells m, m+1
    const double* ca[2][3];     // 1-D operators [at cells, at faces][direction]
    const double* cb[2][3];
    const double* cc[2][3];
    const double* q[3];         // u, v, w (u^k)
    const double* P;            // P^{k-1/2}
    double* e[3];               // E^{k-1} in (if use_prev), E^k out
    double* rhs[3];             // Helmholtz right-hand sides (u* for L_I = 0)
    double dt, nu, alpha, beta, gamma, cn;
    int use_prev;
    int rz;                     // z planes one thread marches through
};

namespace {

constexpr int NS_NT = 256;

// Planes of a thread's chunk: 32 (each chunk reads a plane of the one below it
// again: 928 us in chunks of 8, 877 in 32 at 512 x 256 x 256), fewer where
// that leaves less than two rounds of the three blocks a compute unit holds
// (192 x 160 x 128: 120 us in chunks of 32, 110 in 11), down to 4.
inline int ns_chunk(long long ncb, int nz) {
    const long long n = std::min<long long>(std::max<long long>((2 * 3 * 256 + ncb - 1) / ncb, (nz + 31) / 32), (nz + 3) / 4);
    return (int)((nz + n - 1) / n);
}

// Read-only memory through the scalar cache (uniform indices): the stores of
// the kernel may not alias it.
typedef const double __attribute__((address_space(4)))* cptr;
__device__ __forceinline__ cptr as_const(const double* p) { return (cptr)p; }

// Value of the lane below / above.
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
    const int2 v = __builtin_bit_cast(int2, x);
    const int2 r = {__builtin_amdgcn_update_dpp(0, v.x, CTRL, 0xf, 0xf, false),
                    __builtin_amdgcn_update_dpp(0, v.y, CTRL, 0xf, 0xf, false)};
    return __builtin_bit_cast(double, r);
}
constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138;  // from lane + 1, from lane - 1

// 1-D operator row applied along a direction.
struct Row {
    double a, b, c;
    __device__ __forceinline__ double operator()(double m, double q, double p) const { return b * q + a * m + c * p; }
};

// The diffusion of a component split into its implicit and explicit parts,
// the last NI of the directions x, y, z being implicit.
template <int NI>
__device__ __forceinline__ void ns_diffusion(double lx, double ly, double lz, double& li, double& le) {
    li = (NI > 2 ? lx : 0.0) + (NI > 1 ? ly : 0.0) + (NI > 0 ? lz : 0.0);
    le = (NI > 2 ? 0.0 : lx) + (NI > 1 ? 0.0 : ly) + (NI > 0 ? 0.0 : lz);
}

// Explicit terms and right-hand sides of u on face i, v on face j and w on
// face k of the cells (i, j, k) of a thread's column.  Every value is loaded
// where it exists and from a valid neighbouring address where it does not (a
// wall), then replaced by zero.  A plane takes 11 loads of velocity and
// pressure, seven of them cache hits of the rows next to this one
// (neighbouring rows run on one XCD); what plane k + 1 needs of plane k and
// of itself at k is carried: u at faces i and i - 1, v at j and j - 1, w at
// (i, j), (i + 1, j) and (i, j + 1), and P.
template <int NI>
__global__ __launch_bounds__(NS_NT, 3) void ns_explicit_kernel(NsDesc d) {
    const int nx = d.N[0], ny = d.N[1], nz = d.N[2], nux = d.nf[0], nvy = d.nf[1], nwz = d.nf[2];
    const long long pxy = (long long)nx * ny, uxy = (long long)nux * ny, vxy = (long long)nx * nvy;
    const long long ncb = (pxy + NS_NT - 1) / NS_NT;
    const long long lb = xcd_block(blockIdx.x, gridDim.x);
    const long long zc = lb / ncb;
    const unsigned col = (unsigned)(lb - zc * ncb) * NS_NT + threadIdx.x;  // (a plane has fewer than 2^31 cells)
    if (col >= pxy) return;
    const int j = (int)(col / (unsigned)nx), i = (int)(col - (unsigned)j * nx);
    const int k0 = (int)zc * d.rz, k1 = min(nz, k0 + d.rz);
    // neighbours: cells i +- 1, j +- 1 and faces; wrapped, or clamped at a wall
    const bool hu = i < nux, hv = j < nvy;             // the faces above the cell
    const bool cxm = i > 0 || d.per[0], cxp = i + 1 < nx || d.per[0];   // cells beside
    const bool cym = j > 0 || d.per[1], cyp = j + 1 < ny || d.per[1];
    const bool fxp = i + 1 < nux || d.per[0], fyp = j + 1 < nvy || d.per[1];   // faces beside (below: cxm, cym)
    const int im = i > 0 ? i - 1 : (d.per[0] ? nx - 1 : 0), ip = i + 1 < nx ? i + 1 : (d.per[0] ? 0 : i);
    const int jm = j > 0 ? j - 1 : (d.per[1] ? ny - 1 : 0), jp = j + 1 < ny ? j + 1 : (d.per[1] ? 0 : j);
    const int fi = min(i, nux - 1), fim = min(im, nux - 1), fip = min(ip, nux - 1);
    const int fj = min(j, nvy - 1), fjm = min(jm, nvy - 1), fjp = min(jp, nvy - 1);
    unsigned u00 = (unsigned)j * nux + fi, um0 = (unsigned)j * nux + fim, up0 = (unsigned)j * nux + fip;
    unsigned u0m = (unsigned)jm * nux + fi, u0p = (unsigned)jp * nux + fi, ump = (unsigned)jp * nux + fim;
    unsigned v00 = (unsigned)fj * nx + i, v0m = (unsigned)fjm * nx + i, v0p = (unsigned)fjp * nx + i;
    unsigned vm0 = (unsigned)fj * nx + im, vp0 = (unsigned)fj * nx + ip, vpm = (unsigned)fjm * nx + ip;
    unsigned cm0 = (unsigned)j * nx + im, cp0 = (unsigned)j * nx + ip;
    unsigned c0m = (unsigned)jm * nx + i, c0p = (unsigned)jp * nx + i;
    // the x neighbours come from the lanes beside, at the end of a wave and of a row from memory
    const int lane = threadIdx.x % 64;
    const bool inl = lane > 0 && i > 0, inr = lane < 63 && i + 1 < nx;
    const bool edl = !inl && cxm, edr = !inr && cxp;
    auto zrow = [&](int face, int k) { return Row{as_const(d.ca[face][2])[k], as_const(d.cb[face][2])[k], as_const(d.cc[face][2])[k]}; };
    const cptr wz = as_const(d.w[2]), hz = as_const(d.h[2]);
    auto row = [&](int face, int dir, int m) { return Row{d.ca[face][dir][m], d.cb[face][dir][m], d.cc[face][dir][m]}; };
    const Row rfx = row(1, 0, fi), rcx = row(0, 0, i), rfy = row(1, 1, fj), rcy = row(0, 1, j);
    const double wx0 = d.w[0][i], wx1 = d.w[0][ip], wy0 = d.w[1][j], wy1 = d.w[1][jp];
    const double rhx = 1.0 / d.h[0][fi], rhy = 1.0 / d.h[1][fj], rwx = 1.0 / wx0, rwy = 1.0 / wy0;
    const double* U = d.q[0] + (long long)k0 * uxy;
    const double* V = d.q[1] + (long long)k0 * vxy;
    const double* W = d.q[2] + (long long)k0 * pxy;
    const double* P = d.P + (long long)k0 * pxy;
    // plane k0 and what it needs of the plane below
    double u = hu ? U[u00] : 0.0, ul = cxm ? U[um0] : 0.0;   // ul: face i - 1
    double v = hv ? V[v00] : 0.0, vl = cym ? V[v0m] : 0.0;
    double w = k0 < nwz ? W[col] : 0.0, p = P[col];
    const bool below = k0 > 0 || d.per[2];
    const long long kb = k0 > 0 ? -1 : (below ? nz - 1 : 0);
    double ub = hu && below ? U[kb * uxy + u00] : 0.0;
    double vb = hv && below ? V[kb * vxy + v00] : 0.0;
    const double* Wb = W + (k0 > 0 ? -1 : (below ? nwz - 1 : 0)) * pxy;
    double wb = below ? Wb[col] : 0.0, wbx = below ? Wb[cp0] : 0.0, wby = below ? Wb[c0p] : 0.0;
    for (int k = k0; k < k1; ++k) {
        // keep the offsets in 32 bits: as 64-bit loop invariants they cost a third resident block
        asm("" : "+v"(u00), "+v"(um0), "+v"(up0), "+v"(u0m), "+v"(u0p), "+v"(ump), "+v"(v00), "+v"(v0m));
        asm("" : "+v"(v0p), "+v"(vm0), "+v"(vp0), "+v"(vpm), "+v"(cm0), "+v"(cp0), "+v"(c0m), "+v"(c0p));
        const bool hw = k < nwz, up = k + 1 < nz || d.per[2], wup = k + 1 < nwz || d.per[2];
        // the plane above (wrapped; this plane again above a wall)
        const long long ka = k + 1 < nz ? 1 : (d.per[2] ? 1 - nz : 0), kw = wup ? ka : 0;
        const double* Ua = U + ka * uxy;
        const double* Va = V + ka * vxy;
        const double* Wk = hw ? W : W - pxy;   // (a plane that exists; zeroed below)
        const double ua_ = Ua[u00], va_ = Va[v00], vla_ = Va[v0m], wa_ = (Wk + kw * pxy)[col], pa = P[ka * pxy + col];
        const double uym_ = U[u0m], uyp_ = U[u0p], vyp_ = V[v0p], wym_ = Wk[c0m], wyp_ = Wk[c0p], pyp = P[c0p];
        double lua = 0.0, luy = 0.0, lv = 0.0, lw = 0.0, ru = 0.0, rv = 0.0, rvl = 0.0, rw = 0.0, rp = 0.0;
        if (edl) {
            lua = Ua[um0];
            luy = U[ump];
            lv = V[vm0];
            lw = Wk[cm0];
        }
        if (edr) {
            ru = U[up0];
            rv = V[vp0];
            rvl = V[vpm];
            rw = Wk[cp0];
            rp = P[cp0];
        }
        const long long ou = (long long)k * uxy + u00, ov = (long long)k * vxy + v00, ow = (long long)k * pxy + col;
        double eu = 0.0, ev = 0.0, ew = 0.0;
        if (d.use_prev) {
            eu = d.e[0][ou];
            ev = d.e[1][ov];
            if (hw) ew = d.e[2][ow];
        }
        const double ua = hu && up ? ua_ : 0.0, va = hv && up ? va_ : 0.0, vla = cym && up ? vla_ : 0.0, wa = wup ? wa_ : 0.0;
        const double uym = cym ? uym_ : 0.0, uyp = hu && cyp ? uyp_ : 0.0, vyp = fyp ? vyp_ : 0.0;
        const double wym = hw && cym ? wym_ : 0.0, wyp = hw && cyp ? wyp_ : 0.0;
        auto left = [&](double q, double edge) {
            const double x = lane_shift<DPP_WAVE_SHR1>(q);  // (with every lane of the wave)
            return inl ? x : edge;
        };
        auto right = [&](double q, double edge) {
            const double x = lane_shift<DPP_WAVE_SHL1>(q);  // (with every lane of the wave)
            return inr ? x : edge;
        };
        const double ula = left(ua, up ? lua : 0.0), uly = left(uyp, luy), vxm = left(v, lv), wxm = left(w, hw ? lw : 0.0);
        const double uxp = right(u, fxp ? ru : 0.0), vxp = right(v, hv ? rv : 0.0), vlx = right(vl, cym ? rvl : 0.0);
        const double wxp = right(w, hw ? rw : 0.0), pxp = right(p, rp);
        const double rwz = 1.0 / wz[k];
        // transport of q by the fluxes fp, fm through the faces above and below
        auto flux = [](double q, double qp, double qm, double fp, double fm) {
            return fp * (0.5 * (q + qp)) - fm * (0.5 * (q + qm));
        };
        auto own = [](double q, double qp, double qm) {  // along the component's own direction
            const double l = 0.5 * (qm + q), h = 0.5 * (q + qp);
            return h * h - l * l;
        };
        auto mean = [](double w0, double q0, double w1, double q1) { return 0.5 * (w0 * q0 + w1 * q1); };
        auto put = [&](int c, long long o, double q, double adv, double li, double le, double gp, double e) {
            const double ek = d.nu * le - adv;
            double r = q + d.dt * (d.alpha * ek - d.gamma * gp) + d.cn * li;
            if (d.use_prev) r += d.dt * d.beta * e;
            d.e[c][o] = ek;
            d.rhs[c][o] = r;
        };
        double li, le;
        if (hu) {
            ns_diffusion<NI>(rfx(ul, u, uxp), rcy(uym, u, uyp), zrow(0, k)(ub, u, ua), li, le);
            const double ft = mean(wx0, v, wx1, vxp), fb = mean(wx0, vl, wx1, vlx);
            const double gt = mean(wx0, w, wx1, wxp), gb = mean(wx0, wb, wx1, wbx);
            const double adv = (own(u, uxp, ul) + flux(u, uyp, uym, ft, fb) * rwy + flux(u, ua, ub, gt, gb) * rwz) * rhx;
            put(0, ou, u, adv, li, le, (pxp - p) * rhx, eu);
        }
        if (hv) {
            ns_diffusion<NI>(rcx(vxm, v, vxp), rfy(vl, v, vyp), zrow(0, k)(vb, v, va), li, le);
            const double ft = mean(wy0, u, wy1, uyp), fb = mean(wy0, ul, wy1, uly);
            const double gt = mean(wy0, w, wy1, wyp), gb = mean(wy0, wb, wy1, wby);
            const double adv = (own(v, vyp, vl) + flux(v, vxp, vxm, ft, fb) * rwx + flux(v, va, vb, gt, gb) * rwz) * rhy;
            put(1, ov, v, adv, li, le, (pyp - p) * rhy, ev);
        }
        if (hw) {
            const double rhz = 1.0 / hz[k], w0 = wz[k], w1 = wz[k + 1 < nz ? k + 1 : 0];
            ns_diffusion<NI>(rcx(wxm, w, wxp), rcy(wym, w, wyp), zrow(1, k)(wb, w, wa), li, le);
            const double ft = mean(w0, u, w1, ua), fb = mean(w0, ul, w1, ula);
            const double gt = mean(w0, v, w1, va), gb = mean(w0, vl, w1, vla);
            const double adv = (own(w, wa, wb) + flux(w, wxp, wxm, ft, fb) * rwx + flux(w, wyp, wym, gt, gb) * rwy) * rhz;
            put(2, ow, w, adv, li, le, (pa - p) * rhz, ew);
        }
        ub = u;
        vb = v;
        wb = w;
        wbx = wxp;
        wby = wyp;
        u = ua;
        ul = ula;
        v = va;
        vl = vla;
        w = wa;
        p = pa;
        U += uxy;
        V += vxy;
        W += pxy;
        P += pxy;
    }
}

constexpr double kAlpha[3] = {8.0 / 15.0, 5.0 / 12.0, 3.0 / 4.0};
constexpr double kBeta[3] = {0.0, -17.0 / 60.0, -5.0 / 12.0};

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

hipError_t launch_ns_explicit(NsDesc d, int nimpl, hipStream_t s) {
    const long long ncb = ((long long)d.N[0] * d.N[1] + NS_NT - 1) / NS_NT;
    d.rz = ns_chunk(ncb, d.N[2]);
    const long long nb = ncb * ((d.N[2] + d.rz - 1) / d.rz);
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nb), block(NS_NT);
    if (nimpl == 0) TPT_KLAUNCH(ns_explicit_kernel<0>, grid, block, 0, s, d);
    else if (nimpl == 1) TPT_KLAUNCH(ns_explicit_kernel<1>, grid, block, 0, s, d);
    else if (nimpl == 2) TPT_KLAUNCH(ns_explicit_kernel<2>, grid, block, 0, s, d);
    else TPT_KLAUNCH(ns_explicit_kernel<3>, grid, block, 0, s, d);
    return hipGetLastError();
}

}  // namespace tpt

using namespace tpt;

struct tpt_ns_s {
    tpt_plan pressure = nullptr;
    double nu = 0.0, dt = 0.0;
    int implicit = TPT_IMPLICIT_NONE;
    int impl[3] = {0, 0, 0};
    int device = 0;
    int N[3] = {0, 0, 0}, nf[3] = {0, 0, 0}, per[3] = {0, 0, 0};
    long long count[3] = {0, 0, 0};    // unknowns of u, v, w
    tpt_plan helm[3][3] = {};          // [substep][component], implicit diffusion only
    double* coef = nullptr;            // a, b, c of each component's 1-D operators
    const double* ca[3][3] = {};       // [component][direction]
    const double* cb[3][3] = {};
    const double* cc[3][3] = {};
    ~tpt_ns_s() {
        for (auto& row : helm)
            for (auto& p : row)
                if (p) tpt_plan_destroy(p);
        if (coef) (void)hipFree(coef);
    }
};

namespace {

size_t ns_solve_ws(const tpt_ns_s* ns) {
    size_t b = plan_workspace_bytes(ns->pressure);
    for (auto& row : ns->helm)
        for (auto* p : row)
            if (p) b = std::max(b, plan_workspace_bytes(p));
    return b;
}

size_t ns_ws_bytes(const tpt_ns_s* ns) {
    size_t b = 0;
    for (int c = 0; c < 3; ++c) b += align256((size_t)ns->count[c] * 8);
    return b + align256((size_t)ns->pressure->dof * 8) + ns_solve_ws(ns);
}

}  // namespace

extern "C" {

int tpt_ns_create(tpt_plan pressure, double nu, double dt, int implicit, tpt_ns* out) {
    if (!pressure || !out) return fail(TPT_ERR_INVALID, "NULL argument");
    *out = nullptr;
    ProjDesc pd;
    int rc = proj_desc(pressure, pd);
    if (rc) return rc;
    if (!(std::isfinite(nu) && nu >= 0.0)) return fail(TPT_ERR_INVALID, "nu must be finite and >= 0");
    if (!(std::isfinite(dt) && dt > 0.0)) return fail(TPT_ERR_INVALID, "dt must be finite and > 0");
    if (implicit < TPT_IMPLICIT_XYZ || implicit > TPT_IMPLICIT_NONE)
        return fail(TPT_ERR_INVALID, "unknown implicit directions");
    if (implicit != TPT_IMPLICIT_NONE && !(nu > 0.0))
        return fail(TPT_ERR_INVALID, "implicit diffusion needs nu > 0");
    std::unique_ptr<tpt_ns_s> ns(new (std::nothrow) tpt_ns_s);
    if (!ns) return fail(TPT_ERR_OOM, "host allocation");
    ns->pressure = pressure;
    ns->nu = nu;
    ns->dt = dt;
    ns->implicit = implicit;
    ns->device = pressure->device;
    ns->impl[2] = implicit != TPT_IMPLICIT_NONE;
    ns->impl[1] = implicit == TPT_IMPLICIT_YZ || implicit == TPT_IMPLICIT_XYZ;
    ns->impl[0] = implicit == TPT_IMPLICIT_XYZ;
    for (int d = 0; d < 3; ++d) {
        ns->N[d] = pressure->N[d];
        ns->per[d] = pressure->op[d].periodic ? 1 : 0;
        ns->nf[d] = ns->per[d] ? ns->N[d] : ns->N[d] - 1;
    }
    for (int c = 0; c < 3; ++c) {
        long long n = 1;
        for (int d = 0; d < 3; ++d) n *= d == c ? ns->nf[d] : ns->N[d];
        ns->count[c] = n;
        if (n >= (1LL << 31)) return fail(TPT_ERR_UNSUPPORTED, "velocity component of 2^31 or more unknowns");
    }
    if (pressure->dof >= (1LL << 31)) return fail(TPT_ERR_UNSUPPORTED, "pressure grid of 2^31 or more cells");
    int cur = 0;
    if (hipGetDevice(&cur) == hipSuccess && cur != ns->device) TPT_HIP(hipSetDevice(ns->device));
    // 1-D operators of the velocity components: face-located along their own
    // direction, Dirichlet (no slip / no penetration) at walls
    Op1D ops[3][3];
    size_t total = 0;
    for (int c = 0; c < 3; ++c)
        for (int d = 0; d < 3; ++d) {
            const int bc = ns->per[d] ? BC_P : BC_D;
            std::string err = build_op1d(ns->N[d], pressure->faces[d].data(), bc, bc, d == c ? LOC_F : LOC_C,
                                         ops[c][d]);
            if (!err.empty()) return fail(TPT_ERR_INVALID, "velocity operator: " + err);
            total += 3 * (size_t)ops[c][d].n;
        }
    std::vector<double> h(total);
    size_t off = 0;
    size_t offs[3][3];
    for (int c = 0; c < 3; ++c)
        for (int d = 0; d < 3; ++d) {
            const Op1D& op = ops[c][d];
            offs[c][d] = off;
            std::copy(op.a.begin(), op.a.end(), h.begin() + off);
            std::copy(op.b.begin(), op.b.end(), h.begin() + off + op.n);
            std::copy(op.c.begin(), op.c.end(), h.begin() + off + 2 * op.n);
            off += 3 * (size_t)op.n;
        }
    if (hipMalloc(&ns->coef, total * sizeof(double)) != hipSuccess) {
        ns->coef = nullptr;
        return fail(TPT_ERR_OOM, "NS coefficients");
    }
    TPT_HIP(hipMemcpy(ns->coef, h.data(), total * sizeof(double), hipMemcpyHostToDevice));
    for (int c = 0; c < 3; ++c)
        for (int d = 0; d < 3; ++d) {
            const int n = ops[c][d].n;
            ns->ca[c][d] = ns->coef + offs[c][d];
            ns->cb[c][d] = ns->coef + offs[c][d] + n;
            ns->cc[c][d] = ns->coef + offs[c][d] + 2 * n;
        }
    // the Helmholtz problems of the velocity components, one per substep
    // coefficient gamma_k nu dt / 2 (eigenbases shared through the cache)
    if (implicit != TPT_IMPLICIT_NONE) {
        for (int k = 0; k < 3; ++k)
            for (int c = 0; c < 3; ++c) {
                tpt_plan_desc hd;
                tpt_plan_desc_init(&hd);
                for (int d = 0; d < 3; ++d) {
                    hd.n[d] = ns->N[d];
                    hd.faces[d] = pressure->faces[d].data();
                    const int bc = ns->per[d] ? TPT_BC_PERIODIC : TPT_BC_DIRICHLET;
                    hd.bc[d][0] = hd.bc[d][1] = bc;
                    hd.loc[d] = d == c ? TPT_LOC_FACE : TPT_LOC_CENTER;
                }
                hd.kind = TPT_HELMHOLTZ;
                hd.alpha = (kAlpha[k] + kBeta[k]) * nu * dt / 2.0;
                hd.precision = TPT_FP64;
                hd.nrhs = 1;
                hd.flags = TPT_FLAG_NO_CHECK;
                hd.implicit = implicit;
                if ((rc = tpt_plan_create(&hd, &ns->helm[k][c]))) return rc;
            }
    }
    *out = ns.release();
    return TPT_OK;
}

int tpt_ns_destroy(tpt_ns ns) {
    delete ns;
    return TPT_OK;
}

int tpt_ns_workspace_bytes(tpt_ns ns, size_t* bytes) {
    if (!ns || !bytes) return fail(TPT_ERR_INVALID, "NULL argument");
    *bytes = ns_ws_bytes(ns);
    return TPT_OK;
}

int tpt_ns_substep(tpt_ns ns, int k, double* u, double* v, double* w, double* eu, double* ev, double* ew,
                   double* p, double* phi, void* workspace, size_t workspace_bytes, void* stream) {
    if (!ns || !u || !v || !w || !eu || !ev || !ew || !p || !phi || !workspace)
        return fail(TPT_ERR_INVALID, "NULL argument");
    if (k < 1 || k > 3) return fail(TPT_ERR_INVALID, "substep k must be 1, 2 or 3");
    const size_t need = ns_ws_bytes(ns);
    if (workspace_bytes < need) return fail(TPT_ERR_WORKSPACE, "NS workspace too small: need " + std::to_string(need));
    int cur = 0;
    if (hipGetDevice(&cur) == hipSuccess && cur != ns->device) TPT_HIP(hipSetDevice(ns->device));
    hipStream_t s = (hipStream_t)stream;
    const double alpha = kAlpha[k - 1], beta = kBeta[k - 1], gamma = alpha + beta;
    const double cn = ns->implicit == TPT_IMPLICIT_NONE ? 0.0 : gamma * ns->nu * ns->dt / 2.0;
    double* vel[3] = {u, v, w};
    double* ex[3] = {eu, ev, ew};
    char* base = (char*)workspace;
    double* rhs[3];
    for (int c = 0; c < 3; ++c) {
        rhs[c] = (double*)base;
        base += align256((size_t)ns->count[c] * 8);
    }
    double* div = (double*)base;
    base += align256((size_t)ns->pressure->dof * 8);
    void* sws = base;
    const size_t sws_bytes = workspace_bytes - (size_t)(base - (char*)workspace);
    // explicit terms and the right-hand sides of the three components (all
    // read u^k, so the velocity is overwritten only after the last one)
    const tpt_plan_s* pp = ns->pressure;
    NsDesc nd{};
    for (int e = 0; e < 3; ++e) {
        nd.N[e] = ns->N[e];
        nd.nf[e] = ns->nf[e];
        nd.per[e] = ns->per[e];
        for (int f = 0; f < 2; ++f) {  // the other components are cell-located along e, with one operator
            const int c = f ? e : (e + 1) % 3;
            nd.ca[f][e] = ns->ca[c][e];
            nd.cb[f][e] = ns->cb[c][e];
            nd.cc[f][e] = ns->cc[c][e];
        }
        nd.q[e] = vel[e];
        nd.e[e] = ex[e];
        nd.rhs[e] = rhs[e];
    }
    nd.w[0] = pp->buf.vx; nd.w[1] = pp->buf.vy; nd.w[2] = pp->buf.vz;
    nd.h[0] = pp->buf.dcx; nd.h[1] = pp->buf.dcy; nd.h[2] = pp->buf.dcz;
    nd.P = p;
    nd.dt = ns->dt;
    nd.nu = ns->nu;
    nd.alpha = alpha;
    nd.beta = beta;
    nd.gamma = gamma;
    nd.cn = cn;
    nd.use_prev = k > 1 ? 1 : 0;
    {
        TimedScope ts("ns_explicit", s);
        hipError_t e = launch_ns_explicit(nd, ns->impl[0] + ns->impl[1] + ns->impl[2], s);
        if (e != hipSuccess) return fail(TPT_ERR_HIP, std::string("NS explicit launch: ") + hipGetErrorString(e));
    }
    // implicit diffusion: (I - c L_I) u* = rhs, u* into the velocity arrays
    double* ustar[3] = {rhs[0], rhs[1], rhs[2]};
    int rc;
    if (ns->implicit != TPT_IMPLICIT_NONE) {
        for (int c = 0; c < 3; ++c)
            if ((rc = solve_one(ns->helm[k - 1][c], rhs[c], vel[c], sws, sws_bytes, s))) return rc;
        for (int c = 0; c < 3; ++c) ustar[c] = vel[c];
    }
    // projection: L Phi = D u* / (gamma dt), u = u* - gamma dt G Phi
    ProjDesc pd;
    if ((rc = proj_desc(pp, pd))) return rc;
    pd.u = ustar[0];
    pd.v = ustar[1];
    pd.w = ustar[2];
    pd.uo = u;
    pd.vo = v;
    pd.wo = w;
    pd.div = div;
    pd.phi = phi;
    pd.scale = 1.0 / (gamma * ns->dt);
    pd.gscale = gamma * ns->dt;
    {
        TimedScope ts("divergence", s);
        hipError_t e = launch_divergence(pd, s);
        if (e != hipSuccess) return fail(TPT_ERR_HIP, std::string("divergence launch: ") + hipGetErrorString(e));
    }
    if ((rc = solve_one(ns->pressure, div, phi, sws, sws_bytes, s))) return rc;
    // u = u* - gamma dt G Phi and, in the same pass,
    // P^{k+1/2} = P^{k-1/2} + Phi - c L_I Phi
    pd.P = p;
    pd.pcn = cn;
    const double* pa[3] = {pp->buf.ax, pp->buf.ay, pp->buf.az};
    const double* pb[3] = {pp->buf.bx, pp->buf.by, pp->buf.bz};
    const double* pc[3] = {pp->buf.cx, pp->buf.cy, pp->buf.cz};
    for (int e = 0; e < 3; ++e) {
        pd.pimpl[e] = ns->impl[e];
        pd.pca[e] = pa[e];
        pd.pcb[e] = pb[e];
        pd.pcc[e] = pc[e];
    }
    TimedScope ts("gradient_update", s);
    hipError_t e = launch_gradient_update(pd, s);
    if (e != hipSuccess) return fail(TPT_ERR_HIP, std::string("gradient update launch: ") + hipGetErrorString(e));
    return TPT_OK;
}

}  // extern "C"
