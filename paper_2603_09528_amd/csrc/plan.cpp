// Plans: initialization steps 1.1–1.3 of the three-dimensional procedure
// (§2.2.2) — 1-D operators, eigenbases of x and y, device copies — and the
// device-resident eigenbasis cache shared by plans with the same grid.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace tpt {

// ---- errors -----------------------------------------------------------------
static thread_local std::string g_last_error;
void set_error(const std::string& msg) { g_last_error = msg; }
int fail(int code, const std::string& msg) {
    g_last_error = msg;
    return code;
}
const char* last_error_cstr() { return g_last_error.c_str(); }

DirBasis::~DirBasis() {
    if (block) {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(device);
        (void)hipFree(block);
        (void)hipSetDevice(cur);
    }
}

// ---- eigenbasis cache ---------------------------------------------------------
static std::mutex g_cache_mu;
static std::map<std::string, std::weak_ptr<DirBasis>> g_cache;
static std::map<std::string, std::weak_ptr<const Eig1D>> g_eig_cache;

BasisForm basis_form(const Op1D& op, int prec, bool ylines, int nx, bool no_fast, bool need_dense, int* fast) {
    *fast = -1;
    if (!no_fast && op.uniform && fft_supported(op.n)) {
        if (op.periodic) *fast = UT_FOURIER;
        else if (op.loc == LOC_C && op.bc_lo == BC_N && op.bc_hi == BC_N) *fast = UT_DCT;
        else if (op.loc == LOC_C && op.bc_lo == BC_D && op.bc_hi == BC_D) *fast = UT_DST;
        if (*fast >= 0) return BF_FAST;
    }
    if (op.mirror && !need_dense && fold_fits(op.n, nx, ylines, prec)) return BF_FOLD;
    return BF_DENSE;
}

static std::string eig_key(const Op1D& op, int ncells, const double* faces) {
    std::string k;
    k.reserve(32 + 8 * (ncells + 1));
    int hdr[4] = {ncells, op.bc_lo, op.bc_hi, op.loc};
    k.append((const char*)hdr, sizeof(hdr));
    k.append((const char*)faces, sizeof(double) * (ncells + 1));
    return k;
}

std::shared_ptr<DirBasis> basis_cache_get(const Op1D& op, int ncells, const double* faces, int form, int prec, bool host_only,
                                          std::string& err) {
    int device = 0;
    if (!host_only) {
        if (hipGetDevice(&device) != hipSuccess) {
            err = "hipGetDevice failed";
            return nullptr;
        }
    }
    const std::string ekey = eig_key(op, ncells, faces);
    if (form != BF_FOLD) prec = GP_F64;  // one set for all precisions
    int hdr[4] = {device, host_only ? 1 : 0, form, prec};
    const std::string key = std::string((const char*)hdr, sizeof(hdr)) + ekey;
    std::lock_guard<std::mutex> lock(g_cache_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
        if (auto sp = it->second.lock()) return sp;
    }
    auto b = std::make_shared<DirBasis>();
    b->device = device;
    b->n = op.n;
    b->form = form;
    auto ie = g_eig_cache.find(ekey);
    if (ie != g_eig_cache.end()) b->eig = ie->second.lock();
    if (!b->eig) {
        auto e = std::make_shared<Eig1D>();
        err = eig_op1d(op, *e);
        if (!err.empty()) return nullptr;
        b->eig = e;
        g_eig_cache[ekey] = b->eig;
    }
    const Eig1D& eig = *b->eig;
    // an eigenbasis that does not split after all takes the dense product
    const int h = (op.n + 1) / 2;
    const int hp = (h + FOLD_ROWS - 1) / FOLD_ROWS * FOLD_ROWS, kp = (h + fold_cols(prec) - 1) / fold_cols(prec) * fold_cols(prec);
    FoldBasis fb;
    if (form == BF_FOLD && !fold_basis(op, eig, hp, kp, fb)) b->form = form = BF_DENSE;
    b->null_pos = form == BF_FOLD && eig.null_index >= 0 ? eig.null_index / 2 : eig.null_index;
    if (!host_only) {
        const int n = op.n;
        const size_t nn = (size_t)n * n;
        size_t total = 0;
        auto take = [&](size_t bytes) {
            const size_t o = total;
            total += (bytes + 255) & ~(size_t)255;
            return o;
        };
        const size_t o_lam = take(8 * (size_t)n);
        size_t o_qinv = 0, o_q = 0, o_sqinv = 0, o_sq = 0, o_hqinv = 0, o_lqinv = 0, o_hq = 0, o_lq = 0;
        size_t o_tw = 0, o_qtw = 0;
        // bf16 planes: rows padded to a multiple of 8 elements (16 bytes), so
        // the split-BF16 tiles load them as vectors whatever n is
        const int ldp = (n + 7) / 8 * 8;
        const size_t nf = 2 * (size_t)hp * kp;
        size_t o_xqinv = 0, o_xq = 0, o_rot = 0;
        if (form == BF_FAST) {
            o_tw = take(16 * (size_t)(n / 2));
            o_qtw = take(16 * (size_t)(n / 2 + 1));
        } else if (form == BF_FOLD) {
            const size_t es = prec == GP_F64 ? 8 : 4;  // (two bf16 planes: 4 bytes)
            o_qinv = take(es * nf);
            o_q = take(es * nf);
            if (prec == GP_F64) {
                o_xqinv = take(4 * nf);
                o_xq = take(4 * nf);
                o_rot = take(8 * fb.rot.size());
            }
        } else {
            const size_t np = (size_t)n * ldp;
            o_qinv = take(8 * nn);
            o_q = take(8 * nn);
            o_sqinv = take(4 * nn);
            o_sq = take(4 * nn);
            o_hqinv = take(2 * np);
            o_lqinv = take(2 * np);
            o_hq = take(2 * np);
            o_lq = take(2 * np);
        }
        std::vector<char> host(total, 0);
        double* lam = (double*)(host.data() + o_lam);
        // a folded basis keeps its even modes first
        for (int p = 0; p < n; ++p) lam[form == BF_FOLD ? p / 2 + (p & 1) * h : p] = eig.lam[p];
        if (form == BF_FAST) {
            // twiddles of the length-n real transform and the quarter-wave
            // factors of the cosine / sine transforms, in long double
            double* tw = (double*)(host.data() + o_tw);
            double* qw = (double*)(host.data() + o_qtw);
            const long double pi = 3.14159265358979323846264338327950288L;
            for (int k = 0; k < n / 2; ++k) {
                const long double a = 2.0L * pi * (long double)k / (long double)n;
                tw[2 * k] = (double)std::cos(a);
                tw[2 * k + 1] = (double)-std::sin(a);
            }
            for (int k = 0; k <= n / 2; ++k) {
                const long double a = pi * (long double)k / (2.0L * n);
                qw[2 * k] = (double)std::cos(a);
                qw[2 * k + 1] = (double)-std::sin(a);
            }
        } else if (form == BF_FOLD) {
            // by K step: [columns / w][parity][row][w], w = 64 bytes of
            // elements with column k of the step at (k % 4, k / 4); of the
            // remainders [step of 8][parity][row][high, low terms][8]
            auto at = [&](size_t e, int w) {
                const size_t par = e / ((size_t)hp * kp), row = e / kp % hp, c = e % kp, k = c % w;
                return ((c / w * 2 + par) * hp + row) * w + k % 4 * (w / 4) + k / 4;
            };
            double* dqinv = (double*)(host.data() + o_qinv);
            double* dq = (double*)(host.data() + o_q);
            float* sqinv = (float*)(host.data() + o_qinv);
            float* sq = (float*)(host.data() + o_q);
            uint16_t* bqinv = (uint16_t*)(host.data() + o_qinv);
            uint16_t* bq = (uint16_t*)(host.data() + o_q);
            for (size_t e = 0; e < nf; ++e) {
                if (prec == GP_F64) {
                    dqinv[at(e, 8)] = fb.fwd[e];
                    dq[at(e, 8)] = fb.inv[e];
                } else if (prec == GP_F32) {
                    sqinv[at(e, 16)] = (float)fb.fwd[e];
                    sq[at(e, 16)] = (float)fb.inv[e];
                } else {
                    // [step of 32][parity][hi, lo][row][32]
                    const size_t par = e / ((size_t)hp * kp), row = e / kp % hp, c = e % kp;
                    const size_t o = ((c / 32 * 2 + par) * 2 * hp + row) * 32 + c % 32;
                    const uint16_t hi = host_bf16((float)fb.fwd[e]), hj = host_bf16((float)fb.inv[e]);
                    bqinv[o] = hi;
                    bqinv[o + (size_t)hp * 32] = host_bf16((float)(fb.fwd[e] - (double)host_bf16_to_f(hi)));
                    bq[o] = hj;
                    bq[o + (size_t)hp * 32] = host_bf16((float)(fb.inv[e] - (double)host_bf16_to_f(hj)));
                }
            }
            if (prec == GP_F64) {
                uint16_t* xi = (uint16_t*)(host.data() + o_xqinv);
                uint16_t* xq = (uint16_t*)(host.data() + o_xq);
                for (size_t e = 0; e < nf; ++e) {
                    const size_t par = e / ((size_t)hp * kp), row = e / kp % hp, c = e % kp;
                    const size_t o = ((c / 8 * 2 + par) * hp + row) * 16 + c % 8;
                    fold_split(fb.xfwd[e], fb.sfwd, xi[o], xi[o + 8]);
                    fold_split(fb.xinv[e], fb.sinv, xq[o], xq[o + 8]);
                }
                std::memcpy(host.data() + o_rot, fb.rot.data(), 8 * fb.rot.size());
            }
        } else {
            double* qinv = (double*)(host.data() + o_qinv);
            double* q = (double*)(host.data() + o_q);
            float* sqinv = (float*)(host.data() + o_sqinv);
            float* sq = (float*)(host.data() + o_sq);
            uint16_t* hqinv = (uint16_t*)(host.data() + o_hqinv);
            uint16_t* lqinv = (uint16_t*)(host.data() + o_lqinv);
            uint16_t* hq = (uint16_t*)(host.data() + o_hq);
            uint16_t* lq = (uint16_t*)(host.data() + o_lq);
            for (int i = 0; i < n; ++i) {
                const double si = std::sqrt(op.vol[i]);
                for (int p = 0; p < n; ++p) {
                    const double qt = eig.Qt[(size_t)i * n + p];
                    qinv[(size_t)p * n + i] = qt * si;  // Q^{-1} = Q~^T D^{1/2}
                    q[(size_t)i * n + p] = qt / si;     // Q = D^{-1/2} Q~
                }
            }
            for (size_t e = 0; e < nn; ++e) {
                sqinv[e] = (float)qinv[e];
                sq[e] = (float)q[e];
                const size_t ep = e / n * ldp + e % n;  // padded position (padding stays 0)
                uint16_t hb = host_bf16((float)qinv[e]);
                hqinv[ep] = hb;
                lqinv[ep] = host_bf16((float)(qinv[e] - (double)host_bf16_to_f(hb)));
                hb = host_bf16((float)q[e]);
                hq[ep] = hb;
                lq[ep] = host_bf16((float)(q[e] - (double)host_bf16_to_f(hb)));
            }
        }
        b->h = op.vol[0];
        void* blk = nullptr;
        if (hipMalloc(&blk, total) != hipSuccess) {
            err = "out of device memory for an eigenbasis";
            (void)hipGetLastError();
            return nullptr;
        }
        if (hipMemcpy(blk, host.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(blk);
            err = "hipMemcpy of an eigenbasis failed";
            return nullptr;
        }
        char* d = (char*)blk;
        b->block = blk;
        b->bytes = total;
        b->d_lam = (double*)(d + o_lam);
        if (form == BF_FAST) {
            b->d_twiddle = (double2*)(d + o_tw);
            b->d_qtw = (double2*)(d + o_qtw);
        } else if (form == BF_FOLD) {
            b->hp = hp;
            b->kp = kp;
            if (prec == GP_F64) {
                b->fd_qinv = (double*)(d + o_qinv);
                b->fd_q = (double*)(d + o_q);
            } else if (prec == GP_F32) {
                b->fs_qinv = (float*)(d + o_qinv);
                b->fs_q = (float*)(d + o_q);
            } else {
                b->fb_qinv = (uint16_t*)(d + o_qinv);
                b->fb_q = (uint16_t*)(d + o_q);
            }
            if (prec == GP_F64) {
                b->f_corr = fb.rotated ? 1 : 0;
                b->fxs_qinv = fb.sfwd;
                b->fxs_q = fb.sinv;
                b->fx_qinv = (uint16_t*)(d + o_xqinv);
                b->fx_q = (uint16_t*)(d + o_xq);
                b->f_rot = (double2*)(d + o_rot);
            }
        } else {
            b->ldp = ldp;
            b->d_qinv = (double*)(d + o_qinv);
            b->d_q = (double*)(d + o_q);
            b->s_qinv = (float*)(d + o_sqinv);
            b->s_q = (float*)(d + o_sq);
            b->h_qinv = (uint16_t*)(d + o_hqinv);
            b->l_qinv = (uint16_t*)(d + o_lqinv);
            b->h_q = (uint16_t*)(d + o_hq);
            b->l_q = (uint16_t*)(d + o_lq);
        }
    }
    g_cache[key] = b;
    return b;
}

size_t basis_cache_bytes() {
    std::lock_guard<std::mutex> lock(g_cache_mu);
    size_t s = 0;
    for (auto& kv : g_cache)
        if (auto sp = kv.second.lock()) s += sp->bytes;
    return s;
}

int plan_gemm_prec(const tpt_plan_s* p) {
    switch (p->desc.precision) {
        case TPT_MIXED_FP32: return GP_F32;
        case TPT_MIXED_BF16X3: return GP_BF16X3;
        default: return GP_F64;
    }
}

// Bytes per unknown of the workspace: two transform buffers and the Thomas
// scratch (c', d' in FP64).  Mixed modes use FP32 transform buffers plus an
// FP32 residual; the tail holds partial sums.
static size_t partial_slots(const tpt_plan_s* p) {
    const long long dof = p->dof * p->desc.nrhs;
    // enough for the residual blocks of all rhs, for the x-inverse GEMM blocks
    // of its smallest tile (32 x 64) and for the tiles of the x-inverse
    // half-size products (those have fewer lines to a tile: few long x lines
    // make more of them)
    long long res = 0;
    for (int r = 0; r < p->desc.nrhs; ++r) res += (p->dof + 255) / 256;
    long long xi = ((long long)p->N[1] * p->N[2] * p->desc.nrhs + 31) / 32 * ((p->N[0] + 63) / 64);
    if (p->desc.precision != TPT_FP64)
        xi = std::max(xi, fold_max_tiles(p->N[0], (long long)p->N[1] * p->N[2], plan_gemm_prec(p)));
    // the x-inverse fast transform: at most one block per x line
    const long long fx = (long long)p->N[1] * p->N[2] * p->desc.nrhs;
    // the right-hand-side check: 4 doubles (two slots) per block
    CheckDesc c{};
    c.nx = p->N[0];
    c.ny = p->N[1];
    c.nz = p->N[2];
    long long chk = 2 * check_blocks(c) * p->desc.nrhs;
    if (fft_supported(p->N[0])) chk = std::max(chk, 2 * check_fused_blocks(p) * p->desc.nrhs);
    (void)dof;
    return (size_t)std::max(std::max(std::max(res, xi), fx), chk) + 8;
}

size_t plan_workspace_bytes(const tpt_plan_s* p) {
    const size_t n = (size_t)p->dof * p->desc.nrhs;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t tsc = 8 * (size_t)thomas_scratch_doubles(p->N[0], p->N[1], p->N[2], p->desc.nrhs, p->op[2].periodic ? 1 : 0);
    const size_t main = (p->desc.precision == TPT_FP64) ? 2 * al(8 * n) + al(tsc) : al(tsc) + 3 * al(4 * n);
    return main + 16 * partial_slots(p) + 256;
}

}  // namespace tpt

tpt_plan_s::~tpt_plan_s() {
    if (buf.block || own_ws || h_norms) {
        int cur = 0;
        (void)hipGetDevice(&cur);
        (void)hipSetDevice(device);
        if (buf.block) (void)hipFree(buf.block);
        if (own_ws) (void)hipFree(own_ws);
        if (h_norms) (void)hipHostFree(h_norms);
        (void)hipSetDevice(cur);
    }
}

using namespace tpt;

extern "C" {

void tpt_plan_desc_init(tpt_plan_desc* d) {
    if (!d) return;
    std::memset(d, 0, sizeof(*d));
    for (int i = 0; i < 3; ++i) {
        d->n[i] = 2;
        d->bc[i][0] = d->bc[i][1] = TPT_BC_NEUMANN;
        d->loc[i] = TPT_LOC_CENTER;
    }
    d->kind = TPT_POISSON;
    d->precision = TPT_FP64;
    d->rtol = 1e-12;
    d->max_refine = 8;
    d->fixed_refine = -1;
    d->nrhs = 1;
}

int tpt_plan_create(const tpt_plan_desc* desc, tpt_plan* out) {
    if (!desc || !out) return fail(TPT_ERR_INVALID, "NULL argument");
    *out = nullptr;
    if (desc->nrhs < 1) return fail(TPT_ERR_INVALID, "nrhs must be >= 1");
    if (desc->kind != TPT_POISSON && desc->kind != TPT_HELMHOLTZ) return fail(TPT_ERR_INVALID, "unknown kind");
    if (desc->kind == TPT_HELMHOLTZ && !(desc->alpha > 0.0))
        return fail(TPT_ERR_INVALID, "Helmholtz needs alpha > 0");
    if (desc->precision < TPT_FP64 || desc->precision > TPT_MIXED_BF16X3)
        return fail(TPT_ERR_INVALID, "unknown precision");
    if (desc->implicit < TPT_IMPLICIT_XYZ || desc->implicit > TPT_IMPLICIT_Z)
        return fail(TPT_ERR_INVALID, "unknown implicit directions");
    if (desc->implicit != TPT_IMPLICIT_XYZ && desc->kind != TPT_HELMHOLTZ)
        return fail(TPT_ERR_INVALID, "only a Helmholtz plan can leave directions explicit");
    if (desc->implicit != TPT_IMPLICIT_XYZ && desc->precision != TPT_FP64)
        return fail(TPT_ERR_UNSUPPORTED, "yz and z implicit plans are FP64 only");
    for (int d = 0; d < 3; ++d) {
        if (desc->n[d] < 2) return fail(TPT_ERR_INVALID, "need at least 2 cells per direction");
        if (!desc->faces[d]) return fail(TPT_ERR_INVALID, "faces pointer is NULL");
    }
    std::unique_ptr<tpt_plan_s> p(new tpt_plan_s());
    p->desc = *desc;
    if (p->desc.rtol <= 0.0) p->desc.rtol = 1e-12;
    if (p->desc.max_refine <= 0) p->desc.max_refine = 8;
    p->host_only = (desc->flags & TPT_FLAG_HOST_ONLY) != 0;
    p->seq_thomas = (desc->flags & TPT_FLAG_SEQ_THOMAS) != 0;
    p->check = (desc->flags & TPT_FLAG_NO_CHECK) == 0;
    p->tx = desc->implicit == TPT_IMPLICIT_XYZ;
    p->ty = desc->implicit != TPT_IMPLICIT_Z;
    if (!p->host_only && hipGetDevice(&p->device) != hipSuccess)
        return fail(TPT_ERR_HIP, "no HIP device");
    for (int d = 0; d < 3; ++d) {
        p->faces[d].assign(desc->faces[d], desc->faces[d] + desc->n[d] + 1);
        p->desc.faces[d] = p->faces[d].data();
        std::string err = build_op1d(desc->n[d], p->faces[d].data(), desc->bc[d][0], desc->bc[d][1], desc->loc[d],
                                     p->op[d]);
        if (!err.empty()) return fail(TPT_ERR_INVALID, "direction " + std::to_string(d) + ": " + err);
        p->N[d] = p->op[d].n;
    }
    p->dof = (long long)p->N[0] * p->N[1] * p->N[2];
    // one pass for the x transform and the y GEMM (FP64; x rows of 128 or
    // 256 points, whole 128-row tiles of y) reads whole y bases
    bool want_fuse = !p->host_only && p->tx && p->ty && desc->precision == TPT_FP64 && (desc->flags & TPT_FLAG_FUSE_XY) &&
                     (p->N[0] == 128 || p->N[0] == 256) && p->N[1] % 128 == 0;
    int fast[2] = {-1, -1}, form[2] = {BF_DENSE, BF_DENSE};
    for (int d = 0; d < 2 && !p->host_only; ++d)
        form[d] = basis_form(p->op[d], plan_gemm_prec(p.get()), d == 1, p->N[0],
                             (desc->flags & (d == 0 ? TPT_FLAG_DENSE_X : TPT_FLAG_DENSE_Y)) != 0,
                             d == 1 && want_fuse && fast[0] >= 0, &fast[d]);
    std::string err;
    p->bx = basis_cache_get(p->op[0], desc->n[0], p->faces[0].data(), form[0], plan_gemm_prec(p.get()), p->host_only, err);
    if (!p->bx) return fail(err.find("memory") != std::string::npos ? TPT_ERR_OOM : TPT_ERR_INVALID, "x basis: " + err);
    p->by = basis_cache_get(p->op[1], desc->n[1], p->faces[1].data(), form[1], plan_gemm_prec(p.get()), p->host_only, err);
    if (!p->by) return fail(err.find("memory") != std::string::npos ? TPT_ERR_OOM : TPT_ERR_INVALID, "y basis: " + err);
    if (desc->kind == TPT_POISSON) {
        p->sigma = 0.0;
        p->tau = 1.0;
    } else {
        p->sigma = 1.0;
        p->tau = -desc->alpha;
    }
    // the null line: lambda_x = lambda_y = 0 (both exact) and a singular T_z
    if (desc->kind == TPT_POISSON && p->bx->null_pos >= 0 && p->by->null_pos >= 0 && p->op[2].null_mode)
        p->null_line = p->bx->null_pos + p->N[0] * p->by->null_pos;
    p->info.null_line = p->null_line;
    p->run_check = p->check || (desc->precision != TPT_FP64 && p->null_line >= 0);
    {
        double ax = 0.0, ay = 0.0;
        for (double v : p->op[0].vol) ax += v;
        for (double v : p->op[1].vol) ay += v;
        p->last_area_inv = 1.0 / (ax * ay * p->op[2].vol[p->N[2] - 1]);
    }
    p->fast[0] = fast[0];
    p->fast[1] = fast[1];
    p->fuse_xy = want_fuse && p->fast[0] >= 0 && p->fast[1] < 0;
    p->info.rel_residual = -1.0;
    p->info.compat_defect = p->check ? 0.0 : -1.0;
    p->info.nonfinite = p->check ? 0 : -1;
    if (!p->host_only) {
        const size_t nx = p->N[0], ny = p->N[1], nz = p->N[2];
        const size_t nstat = (size_t)TPT_STATS * p->desc.nrhs;
        const size_t doubles = 5 * (nx + ny + nz) + ny * nz + std::max(nx, ny) + nstat + 64;
        void* blk = nullptr;
        if (hipMalloc(&blk, doubles * 8) != hipSuccess) {
            (void)hipGetLastError();
            return fail(TPT_ERR_OOM, "out of device memory for plan coefficients");
        }
        p->buf.block = blk;
        std::vector<double> h(doubles, 0.0);
        double* w = h.data();
        auto put = [&](const std::vector<double>& v) {
            std::memcpy(w, v.data(), 8 * v.size());
            w += v.size();
        };
        put(p->op[0].a); put(p->op[0].b); put(p->op[0].c);
        put(p->op[1].a); put(p->op[1].b); put(p->op[1].c);
        put(p->op[2].a); put(p->op[2].b); put(p->op[2].c);
        put(p->op[0].vol); put(p->op[1].vol); put(p->op[2].vol);
        for (size_t k = 0; k < nz; ++k)
            for (size_t j = 0; j < ny; ++j) *w++ = p->op[1].vol[j] * p->op[2].vol[k];
        w += std::max(nx, ny);  // zeros
        for (int d = 0; d < 3; ++d) {
            // centre distances, half the sum of the two cell widths (as the
            // operator's couplings use them, so that D G is its Laplacian)
            const std::vector<double>& fc = p->faces[d];
            const size_t nc = fc.size() - 1, n = p->N[d];
            for (size_t m = 0; m < n; ++m) {
                const double wm = fc[m + 1] - fc[m];
                const double wn = m + 1 < nc ? fc[m + 2] - fc[m + 1] : fc[1] - fc[0];
                *w++ = 0.5 * (wm + wn);
            }
        }
        TPT_HIP(hipMemcpy(blk, h.data(), doubles * 8, hipMemcpyHostToDevice));
        double* d = (double*)blk;
        p->buf.ax = d; d += nx; p->buf.bx = d; d += nx; p->buf.cx = d; d += nx;
        p->buf.ay = d; d += ny; p->buf.by = d; d += ny; p->buf.cy = d; d += ny;
        p->buf.az = d; d += nz; p->buf.bz = d; d += nz; p->buf.cz = d; d += nz;
        p->buf.vx = d; d += nx; p->buf.vy = d; d += ny; p->buf.vz = d; d += nz;
        p->buf.vyz = d; d += ny * nz;
        p->buf.zeros = d; d += std::max(nx, ny);
        p->buf.dcx = d; d += nx; p->buf.dcy = d; d += ny; p->buf.dcz = d; d += nz;
        p->buf.norms = d;
        if (hipHostMalloc((void**)&p->h_norms, (nstat + 8) * sizeof(double), hipHostMallocDefault) != hipSuccess) {
            p->h_norms = nullptr;
            return fail(TPT_ERR_OOM, "pinned host allocation failed");
        }
    }
    *out = p.release();
    return TPT_OK;
}

int tpt_plan_destroy(tpt_plan plan) {
    delete plan;
    return TPT_OK;
}

int tpt_plan_shape(tpt_plan p, int shape[3]) {
    if (!p || !shape) return fail(TPT_ERR_INVALID, "NULL argument");
    for (int d = 0; d < 3; ++d) shape[d] = p->N[d];
    return TPT_OK;
}

int tpt_plan_workspace_bytes(tpt_plan p, size_t* bytes) {
    if (!p || !bytes) return fail(TPT_ERR_INVALID, "NULL argument");
    *bytes = plan_workspace_bytes(p);
    return TPT_OK;
}

int tpt_plan_eigen(tpt_plan p, int dir, double* lam, double* Qt) {
    if (!p || !lam || dir < 0 || dir > 1) return fail(TPT_ERR_INVALID, "bad argument");
    const Eig1D& e = *(dir == 0 ? p->bx : p->by)->eig;
    std::memcpy(lam, e.lam.data(), sizeof(double) * e.n);
    if (Qt) std::memcpy(Qt, e.Qt.data(), sizeof(double) * (size_t)e.n * e.n);
    return TPT_OK;
}

int tpt_plan_operator(tpt_plan p, int dir, double* a, double* b, double* c, double* vol) {
    if (!p || dir < 0 || dir > 2) return fail(TPT_ERR_INVALID, "bad argument");
    const Op1D& op = p->op[dir];
    const size_t n = sizeof(double) * op.n;
    if (a) std::memcpy(a, op.a.data(), n);
    if (b) std::memcpy(b, op.b.data(), n);
    if (c) std::memcpy(c, op.c.data(), n);
    if (vol) std::memcpy(vol, op.vol.data(), n);
    return TPT_OK;
}

int tpt_plan_transforms(tpt_plan p, int kinds[2]) {
    if (!p || !kinds) return fail(TPT_ERR_INVALID, "NULL argument");
    for (int d = 0; d < 2; ++d) kinds[d] = p->fast[d] < 0 ? TPT_XFORM_GEMM : TPT_XFORM_FFT + p->fast[d];
    if (!p->tx) kinds[0] = TPT_XFORM_NONE;
    if (!p->ty) kinds[1] = TPT_XFORM_NONE;
    return TPT_OK;
}

int tpt_plan_fused(tpt_plan p, int* fused) {
    if (!p || !fused) return fail(TPT_ERR_INVALID, "NULL argument");
    *fused = p->fuse_xy ? 1 : 0;
    return TPT_OK;
}

const char* tpt_last_error(void) { return tpt::last_error_cstr(); }
const char* tpt_version(void) { return "tpt 0.1 (gfx950)"; }

}  // extern "C"
