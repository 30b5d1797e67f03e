// C ABI of the solver (include/hyperpower.h) and the host-side orchestration
// of the hyper-power preconditioner and the Krylov solvers.  Every numerical
// step runs in the HIP kernels of ops.hip, fd.hip and krylov.hip; this file
// only sequences them, holds the O(1)-per-iteration Krylov scalars and owns
// device memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <stdexcept>
#include <vector>

#include "hp_internal.h"
#include "vec.h"

using namespace hp;

namespace {

constexpr int KMAX = 6;  // largest number of hyper-power updates

#define HIPCHK(expr)                                   \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return HP_EHIP;          \
    } while (0)

// ---- buffers -------------------------------------------------------------------
struct Extra {
    // hyper-power temporaries
    double* hv = nullptr;  // 4 velocity vectors x max_rhs
    int pv_slot = 0;       // hv slot of the P_V Richardson residual (0: V block, 3: Q block)
    // the Q block of P_k (k > 1, eq. Pcq2, PCG) runs beside the V block: a second stream, fork/join
    // events and a second operator / fast-diagonalisation workspace
    hipStream_t side = nullptr;
    hipEvent_t fork_ev = nullptr, join_ev = nullptr;
    double* ws2 = nullptr;
    double* hq = nullptr;  // 3 pressure vectors per level x (KMAX+1) x max_rhs
    // inner PCG of the Schur variant HP_SCHUR_PCG: r, z, p, A p (velocity x
    // max_rhs each), per-rhs scalars, step coefficients and dot partials
    double* cgv = nullptr;
    CgScalars* cgsc = nullptr;
    double* cgcoef = nullptr;
    double* cgpart = nullptr;
    // Krylov vectors
    double* kv = nullptr;
    size_t kv_doubles = 0;
    double* dcoef = nullptr;  // device coefficient staging
    double* hcoef = nullptr;  // pinned host coefficients
    size_t coef_doubles = 0;
    // device-side MINRES state (two buffers, read and written alternately),
    // coefficient slots, dot partials
    MinresScalars* msc = nullptr;
    MinresScalars* hmsc[2] = {nullptr, nullptr};  // pinned host mirrors
    MinresScalars* dmsc[2] = {nullptr, nullptr};  // their device addresses
    double* mpart = nullptr;   // 2 x DOT partials per rhs
    // partials of the MINRES (z_new . v_new), written by the last
    // fast-diagonalisation launch of the V block (mfg) and of the Q block
    // (mfq), fd_dot_count per rhs each; zeroed once, slots no workgroup
    // reaches stay zero
    double* mfg = nullptr;
    double* mfq = nullptr;
    hipEvent_t mev[4] = {nullptr, nullptr, nullptr, nullptr};  // ring of iteration ends
    hipStream_t cap = nullptr;  // non-blocking stream used only for graph capture
    // cached iteration graphs (one per buffer-rotation phase)
    bool g_valid = false;
    hipGraphExec_t g_exec[6] = {};
    int g_q = 0, g_k = 0, g_nrhs = 0, g_var = 0, g_sched = 0, g_prec = 0;
    double g_tol = 0, g_nu = 0;
    const double* g_kv = nullptr;
    // device-side FGMRES state (restart length up to 128)
    FgScalars* fsc = nullptr;
    FgScalars* hfsc[2] = {nullptr, nullptr};
    FgScalars* dfsc[2] = {nullptr, nullptr};  // device addresses of the mapped mirrors
    double* fH = nullptr;      // R x 129 x 128
    double* fcs = nullptr;     // R x 128
    double* fsn = nullptr;     // R x 128
    double* fg = nullptr;      // R x 129
    double* fy = nullptr;      // R x 128
    double* fhc = nullptr;     // R x 129 Gram-Schmidt coefficients
    double* fvs = nullptr;     // R
    double* fpart = nullptr;   // partials for up to 129 pairs x R
    // quadrature-based forward operator (tables and scratch made on first use)
    QuadOp quad;
    bool f_valid = false;
    std::vector<hipGraphExec_t> f_exec;
    int f_q = 0, f_k = 0, f_nrhs = 0, f_var = 0, f_sched = 0, f_prec = 0, f_m = 0;
    double f_tol = 0, f_nu = 0;
    const double* f_kv = nullptr;
};

Extra* extra_of(hp_ctx* c);

struct CtxExtra {
    hp_ctx ctx;
    Extra ex;
};

Extra* extra_of(hp_ctx* c) { return &reinterpret_cast<CtxExtra*>(c)->ex; }

Fields full_fields(hp_ctx* c, const double* base) {
    Fields f{};
    for (int b = 0; b < 4; ++b) {
        f.f[b] = const_cast<double*>(base) + c->off[b];
        f.stride[b] = c->N;
    }
    return f;
}

// The forward problem y = K x of the Krylov loops: the Kronecker-factored
// operator kernels, or (forward = 1) the quadrature-based operator.
hipError_t launch_forward(hp_ctx* c, const double* x, double* y, int nrhs) {
    if (c->opts.forward == 1) {
        QuadOp* q = &extra_of(c)->quad;
        hipError_t e = quad_setup(c, q);
        if (e != hipSuccess) return e;
        return launch_quad_K(c, q, full_fields(c, x), full_fields(c, y), nrhs);
    }
    return launch_operator(c, OP_K, full_fields(c, x), full_fields(c, y), 1.0, 0.0, nullptr, nrhs);
}

Fields vel_fields(hp_ctx* c, const double* base, long long stride) {
    Fields f{};
    for (int b = 0; b < 3; ++b) {
        f.f[b] = const_cast<double*>(base) + c->off[b];
        f.stride[b] = stride;
    }
    f.f[3] = nullptr;
    f.stride[3] = 0;
    return f;
}

Fields pres_fields(hp_ctx* c, const double* base, long long stride) {
    Fields f{};
    f.f[3] = const_cast<double*>(base);
    f.stride[3] = stride;
    return f;
}

// velocity / pressure views of full vectors
Fields vel_of_full(hp_ctx* c, const double* base) { return vel_fields(c, base, c->N); }
Fields pres_of_full(hp_ctx* c, const double* base) {
    return pres_fields(c, base + c->off[3], c->N);
}

hp_status check_rhs(hp_ctx* c, int nrhs) {
    if (!c || nrhs < 1 || nrhs > c->opts.max_rhs) return HP_EINVAL;
    return HP_OK;
}

// device copy of strided block data: y_b = a x_b + b y_b for each rhs, per block
hipError_t fields_axpby(hp_ctx* c, const Fields& x, const Fields& y, double a, double b,
                        bool vel, bool pres, int nrhs) {
    for (int blk = vel ? 0 : 3; blk < (pres ? 4 : 3); ++blk) {
        long long n = c->dims[blk][0] * c->dims[blk][1] * c->dims[blk][2];
        hipError_t e = vec_axpbypcz(c->stream, n, nrhs, a, x.f[blk], x.stride[blk], b, y.f[blk],
                                    y.stride[blk], 0.0, nullptr, 0, y.f[blk], y.stride[blk]);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// out = a x + b y + g z on the pressure block (batched)
hipError_t pres_axpbypcz(hp_ctx* c, double a, const Fields& x, double b, const Fields& y, double g,
                         const Fields& z, const Fields& out, int nrhs) {
    return vec_axpbypcz(c->stream, c->nQ, nrhs, a, x.f[3], x.stride[3], b, y.f[3], y.stride[3], g,
                        z.f[3], z.stride[3], out.f[3], out.stride[3]);
}

// ---- hyper-power preconditioner (Secs. 2, 4.1) ------------------------------------

// The factor of P_{Q,0}^{-1} = 2 nu w M_q^{-1} (w: the damping factor p0_scale).
double q0_factor(const hp_ctx* c) { return 2.0 * c->nu * c->opts.p0_scale; }

// y = P_{V,level}^{-1} x: q^level Richardson steps y <- y + P_{V,0}^{-1}(x - A y)
// from y = 0, which equals the hyper-power recursion of eq. Pcv (its Neumann
// form, eq. neumann).  x, y: velocity views; must not alias each other.
hipError_t apply_PV(hp_ctx* c, int q, int level, const Fields& x, const Fields& y, int nrhs,
                    int prec, const FdDot* dot = nullptr) {
    Extra* ex = extra_of(c);
    long long steps = 1;
    for (int i = 0; i < level; ++i) steps *= q;
    // the dot partials come from the last fast-diagonalisation launch
    hipError_t e = launch_P0(c, x, y, true, false, false, prec, nrhs, steps == 1 ? dot : nullptr);
    if (e != hipSuccess) return e;
    Fields r = vel_fields(c, ex->hv + (size_t)ex->pv_slot * c->nV * c->opts.max_rhs, c->nV);
    for (long long j = 1; j < steps; ++j) {
        e = launch_operator(c, OP_A, y, r, -1.0, 1.0, &x, nrhs);  // r = x - A y
        if (e != hipSuccess) return e;
        e = launch_P0(c, r, y, true, false, true, prec, nrhs,    // y += P0^{-1} r
                      j + 1 == steps ? dot : nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// out = S~_l t = B^T P_{V,l}^{-1} B t  (pressure views).  With
// after_q0 the argument is s and t = P_{Q,0}^{-1} s is implied: B t = 2 nu D^T s
// (B = D^T M_q, P_{Q,0}^{-1} = 2 nu M_q^{-1}), which skips P_{Q,0} and M_q.
hipError_t apply_Stilde(hp_ctx* c, int q, int l, const Fields& t, const Fields& out, int nrhs,
                        int prec, bool after_q0 = false) {
    Extra* ex = extra_of(c);
    const long long nV = c->nV;
    Fields b1 = vel_fields(c, ex->hv + nV * c->opts.max_rhs, nV);       // slot 1
    Fields b2 = vel_fields(c, ex->hv + 2 * nV * c->opts.max_rhs, nV);   // slot 2
    hipError_t e = after_q0 ? launch_operator(c, OP_DT, t, b1, q0_factor(c), 0.0, nullptr, nrhs)
                            : launch_operator(c, OP_B, t, b1, 1.0, 0.0, nullptr, nrhs);
    if (e != hipSuccess) return e;
    e = apply_PV(c, q, l, b1, b2, nrhs, prec);
    if (e != hipSuccess) return e;
    return launch_operator(c, OP_BT, b2, out, 1.0, 0.0, nullptr, nrhs);
}

// out = S_pcg t = B' Y, Y the preconditioned conjugate-gradient iterate for
// A Y = B t from Y = 0 with P_{V,l}, l = opts.schur_level, after
// opts.schur_pcg_iters steps (a right-hand side stops early once
// sqrt(r.z) <= opts.schur_pcg_tol sqrt(r_0.z_0)): options (3) (l = 0) and
// (4) (l > 0) of Sec. 4.1.  after_q0 as for apply_Stilde.  Every step is a
// fixed launch sequence with device-side scalars (capturable in a graph).
hipError_t apply_Spcg(hp_ctx* c, int q, const Fields& t, const Fields& out, int nrhs, int prec,
                      bool after_q0 = false) {
    Extra* ex = extra_of(c);
    const long long nV = c->nV, R = c->opts.max_rhs;
    const int lv = c->opts.schur_level;
    hipStream_t st = c->stream;
    double* bv = ex->hv + nV * R;       // slot 1: B t
    double* y = ex->hv + 2 * nV * R;    // slot 2: the iterate
    double* r = ex->cgv;
    double* z = r + nV * R;
    double* pv = z + nV * R;
    double* qv = pv + nV * R;
    double* cx = ex->cgcoef;
    double* cr = cx + 2 * R;
    double* cp = cr + 2 * R;
    auto F = [&](double* b) { return vel_fields(c, b, nV); };
    hipError_t e = after_q0 ? launch_operator(c, OP_DT, t, F(bv), q0_factor(c), 0.0, nullptr, nrhs)
                            : launch_operator(c, OP_B, t, F(bv), 1.0, 0.0, nullptr, nrhs);
    if (e != hipSuccess) return e;
    const long long n = nV * nrhs;  // velocity vectors are contiguous per rhs
    if ((e = vec_copy(st, n, bv, r)) != hipSuccess) return e;
    if ((e = vec_zero(st, n, y)) != hipSuccess) return e;
    if ((e = apply_PV(c, q, lv, F(r), F(z), nrhs, prec)) != hipSuccess) return e;
    if ((e = vec_copy(st, n, z, pv)) != hipSuccess) return e;
    const int cnt = (int)vec_dot_partial_count(nV);
    if ((e = vec_dot_partials(st, nV, nV, r, z, nrhs, ex->cgpart)) != hipSuccess) return e;
    if ((e = cg_init(st, ex->cgsc, ex->cgpart, cnt, nrhs)) != hipSuccess) return e;
    for (int j = 0; j < c->opts.schur_pcg_iters; ++j) {
        if ((e = launch_operator(c, OP_A, F(pv), F(qv), 1.0, 0.0, nullptr, nrhs)) != hipSuccess)
            return e;
        if ((e = vec_dot_partials(st, nV, nV, pv, qv, nrhs, ex->cgpart)) != hipSuccess) return e;
        if ((e = cg_alpha(st, ex->cgsc, ex->cgpart, cnt, cx, cr, nrhs)) != hipSuccess) return e;
        const double* xy[2] = {y, pv};
        if ((e = vec_lincomb(st, nV, nV, nrhs, 2, xy, cx, y)) != hipSuccess) return e;
        const double* xr[2] = {r, qv};
        if ((e = vec_lincomb(st, nV, nV, nrhs, 2, xr, cr, r)) != hipSuccess) return e;
        if ((e = apply_PV(c, q, lv, F(r), F(z), nrhs, prec)) != hipSuccess) return e;
        if ((e = vec_dot_partials(st, nV, nV, r, z, nrhs, ex->cgpart)) != hipSuccess) return e;
        if ((e = cg_beta(st, ex->cgsc, ex->cgpart, cnt, cp, c->opts.schur_pcg_tol, nrhs)) != hipSuccess)
            return e;
        const double* xp[2] = {z, pv};
        if ((e = vec_lincomb(st, nV, nV, nrhs, 2, xp, cp, pv)) != hipSuccess) return e;
    }
    return launch_operator(c, OP_BT, F(y), out, 1.0, 0.0, nullptr, nrhs);
}

int l_of(const hp_ctx* c, int k) {
    if (c->opts.l_schedule == HP_L_LITERAL) return k == 1 ? 0 : k;
    return k - 1;
}

Fields hq_slot(hp_ctx* c, int level, int slot) {
    Extra* ex = extra_of(c);
    const long long nQ = c->nQ, R = c->opts.max_rhs;
    return pres_fields(c, ex->hq + ((long long)level * 3 + slot) * nQ * R, nQ);
}

// y = P^_{Q,level}^{-1} x by the recursion of eq. Pcq1:
//   X_k = X_{k-1} sum_{i<q} (I - S~_{l(k)} X_{k-1})^i
// (for HP_SCHUR_PCG the same recursion with the fixed S_pcg in place of
// S~_{l(k)}: eq. Pcq2 taken literally, as S_pcg is not linear),
// with the sum evaluated in Horner form, s_1 = x, s_{i+1} = x + (I - S X) s_i,
// so that y = X_{k-1} s_q (one fused update per term instead of two).
hipError_t apply_PQ1(hp_ctx* c, int q, int level, const Fields& x, const Fields& y, int nrhs,
                     int prec, const FdDot* dot = nullptr) {
    if (level == 0) return launch_P0(c, x, y, false, true, false, prec, nrhs, dot);
    Fields sa = hq_slot(c, level, 0), sb = hq_slot(c, level, 1), t = hq_slot(c, level, 2);
    const int lv = l_of(c, level);
    const bool pcg = c->opts.schur_variant == HP_SCHUR_PCG;  // fixed S_pcg (eq. Pcq2 form)
    const Fields* s = &x;  // s_1 = x
    hipError_t e = hipSuccess;
    for (int i = 1; i < q; ++i) {
        if (level == 1) {
            // X_0 = P_{Q,0}^{-1}: t = S~ X_0 s_i = B' P_{V,l}^{-1} (2 nu D' s_i)
            e = pcg ? apply_Spcg(c, q, *s, t, nrhs, prec, true)
                    : apply_Stilde(c, q, lv, *s, t, nrhs, prec, true);
        } else {
            e = apply_PQ1(c, q, level - 1, *s, t, nrhs, prec);  // t = X_{k-1} s_i
            if (e != hipSuccess) return e;
            // t = S~ t (B reads t first)
            e = pcg ? apply_Spcg(c, q, t, t, nrhs, prec) : apply_Stilde(c, q, lv, t, t, nrhs, prec);
        }
        if (e != hipSuccess) return e;
        if (level == 1 && i == q - 1) {
            // the last s_q = x + s_{q-1} - t is formed where the final
            // P_{Q,0}^{-1} reads it (the same arithmetic, one launch fewer)
            const FdComb comb{*s, t, 1.0, 1.0, -1.0};
            return launch_P0(c, x, y, false, true, false, prec, nrhs, dot, &comb);
        }
        const Fields* sn = (s == &sa) ? &sb : &sa;
        e = pres_axpbypcz(c, 1.0, x, 1.0, *s, -1.0, t, *sn, nrhs);  // s_{i+1} = x + s_i - t
        if (e != hipSuccess) return e;
        s = sn;
    }
    return apply_PQ1(c, q, level - 1, *s, y, nrhs, prec, dot);
}

// y = P_{Q,level}^{-1} x for eq. Pcq2 with the fixed S~_l, l = opts.schur_level
// (option (1) of Sec. 4.1 for l = 0, option (2) for l > 0): q^level
// Richardson steps.
hipError_t apply_PQ2(hp_ctx* c, int q, int level, const Fields& x, const Fields& y, int nrhs,
                     int prec, const FdDot* dot = nullptr) {
    long long steps = 1;
    for (int i = 0; i < level; ++i) steps *= q;
    hipError_t e = launch_P0(c, x, y, false, true, false, prec, nrhs, steps == 1 ? dot : nullptr);
    if (e != hipSuccess) return e;
    Fields t = hq_slot(c, 0, 0);
    for (long long j = 1; j < steps; ++j) {
        e = apply_Stilde(c, q, c->opts.schur_level, y, t, nrhs, prec);  // t = S~_l y
        if (e != hipSuccess) return e;
        e = fields_axpby(c, x, t, 1.0, -1.0, false, true, nrhs);    // t = x - t
        if (e != hipSuccess) return e;
        e = launch_P0(c, t, y, false, true, true, prec, nrhs,       // y += P_Q0^{-1} t
                      j + 1 == steps ? dot : nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// P_k^{-1} = blockdiag(P_{V,k}^{-1}, P_{Q,k}^{-1}) (Sec. 4): the two blocks are
// independent.  At k <= 1 they share their launches (apply_Pk_joint);
// otherwise the Q block is issued on a second stream with its own
// workspace and residual slot (fork/join through events, which also holds
// under stream capture) while the V block runs on the context stream.
// Optional dot product of the result with `with` (a full vector), as
// partials written by the last launch of each block: the velocity part into
// vpart, the pressure part into qpart (fd_dot_count(c, true / false) per rhs).
struct PkDot {
    const double* with;
    double* vpart;
    double* qpart;
};

// The Q block of P_k (and the pressure part of the dot) on c->stream.
hipError_t pk_q_block(hp_ctx* c, int q, int k, const double* x, double* y, int nrhs,
                      const PkDot* pd) {
    const int prec = c->opts.precision;
    const FdDot qdot = pd ? FdDot{pd->with, pd->qpart} : FdDot{};
    if (c->opts.schur_variant == HP_SCHUR_PCQ2)
        return apply_PQ2(c, q, k, pres_of_full(c, x), pres_of_full(c, y), nrhs, prec,
                         pd ? &qdot : nullptr);
    return apply_PQ1(c, q, k, pres_of_full(c, x), pres_of_full(c, y), nrhs, prec,
                     pd ? &qdot : nullptr);
}

// The V block of P_k (and the velocity part of the dot) on c->stream.
hipError_t pk_v_block(hp_ctx* c, int q, int k, const double* x, double* y, int nrhs,
                      const PkDot* pd) {
    const FdDot vdot = pd ? FdDot{pd->with, pd->vpart} : FdDot{};
    return apply_PV(c, q, k, vel_of_full(c, x), vel_of_full(c, y), nrhs, c->opts.precision,
                    pd ? &vdot : nullptr);
}

// Runs fn() with the Q block's settings: stream s, the second workspace and
// its own Richardson residual slot; restores the context afterwards.
template <typename F>
hipError_t with_q_settings(hp_ctx* c, hipStream_t s, F fn) {
    Extra* ex = extra_of(c);
    hipStream_t s0 = c->stream;
    double* ws0 = c->ws;
    c->stream = s;
    c->ws = ex->ws2;
    ex->pv_slot = 3;
    const hipError_t e = fn();
    c->stream = s0;
    c->ws = ws0;
    ex->pv_slot = 0;
    return e;
}

// P_0, and P_1 of eq. Pcq1, with the two blocks in common launches.  At k = 1
// they run in step: each of the q - 1 updates needs P_{V,0}^{-1} of the V
// block's residual and of the Q block's 2 nu D' s, then the pressure chains of
// A y and of B', and at the end P_0 of all four fields.  Against one stream
// per block this is about half the launches and no fork and join (four event
// calls, about 20 us of host time): a MINRES solve at 32^3, degree 3, 3.76 ->
// 3.20 ms, the quadrature one at 16^3, degree 4, 4.08 -> 3.73.  The gain falls
// as the kernels fill the chip (P_1 alone, us, in common and on two streams:
// 32^3 57.6 and 68 to 86, 48^3 84.0 and 85 to 89, 61^3 95.2 and 97.5).
hipError_t apply_Pk_joint(hp_ctx* c, int q, int k, const double* x, double* y, int nrhs,
                          const PkDot* pd) {
    Extra* ex = extra_of(c);
    const int prec = c->opts.precision;
    const FdDot vdot = pd ? FdDot{pd->with, pd->vpart} : FdDot{};
    const FdDot qdot = pd ? FdDot{pd->with, pd->qpart} : FdDot{};
    const FdDot *vd = pd ? &vdot : nullptr, *qd = pd ? &qdot : nullptr;
    const Fields fx = full_fields(c, x), fy = full_fields(c, y);
    if (k == 0) {
        const P0Set all{fx, fy, c->ws, false, false};
        return launch_P0_sets(c, &all, 1, true, true, prec, nrhs, vd, qd);
    }
    const long long nV = c->nV, R = c->opts.max_rhs;
    const Fields xv = vel_of_full(c, x), yv = vel_of_full(c, y), xq = pres_of_full(c, x);
    const Fields res = vel_fields(c, ex->hv, nV);                 // V block: x - A y
    const Fields b1 = vel_fields(c, ex->hv + nV * R, nV);         // Q block: 2 nu D' s
    const Fields b2 = vel_fields(c, ex->hv + 2 * nV * R, nV);     // P_{V,0}^{-1} b1
    const Fields sa = hq_slot(c, 1, 0), sb = hq_slot(c, 1, 1), t = hq_slot(c, 1, 2);
    const Fields* s = &xq;  // s_1 = x
    hipError_t e;
    for (int i = 1; i < q; ++i) {
        if ((e = launch_operator(c, OP_DT, *s, b1, q0_factor(c), 0.0, nullptr, nrhs)) != hipSuccess)
            return e;
        const P0Set vel[2] = {{i == 1 ? xv : res, yv, c->ws, i > 1, false},
                              {b1, b2, ex->ws2, false, false}};
        if ((e = launch_P0_sets(c, vel, 2, true, false, prec, nrhs)) != hipSuccess) return e;
        if ((e = launch_residual_and_Bt(c, yv, res, xv, b2, t, nrhs)) != hipSuccess) return e;
        if (i == q - 1) break;
        const Fields* sn = (s == &sa) ? &sb : &sa;
        if ((e = pres_axpbypcz(c, 1.0, xq, 1.0, *s, -1.0, t, *sn, nrhs)) != hipSuccess) return e;
        s = sn;
    }
    // y_V += P_{V,0}^{-1} (x - A y), y_Q = P_{Q,0}^{-1} (x + s - t)
    Fields in = res;
    in.f[3] = xq.f[3];
    in.stride[3] = xq.stride[3];
    const FdComb comb{*s, t, 1.0, 1.0, -1.0};
    const P0Set all{in, fy, c->ws, true, false};
    return launch_P0_sets(c, &all, 1, true, true, prec, nrhs, vd, qd, &comb);
}

hipError_t apply_Pk(hp_ctx* c, int q, int k, const double* x, double* y, int nrhs,
                    const PkDot* pd = nullptr) {
    Extra* ex = extra_of(c);
    if (ex->side && (k == 0 || (k == 1 && c->opts.schur_variant == HP_SCHUR_PCQ1)))
        return apply_Pk_joint(c, q, k, x, y, nrhs, pd);
    if (!ex->side) {
        hipError_t e = pk_v_block(c, q, k, x, y, nrhs, pd);
        return e != hipSuccess ? e : pk_q_block(c, q, k, x, y, nrhs, pd);
    }
    hipStream_t main = c->stream;
    hipError_t e = hipEventRecord(ex->fork_ev, main);
    if (e == hipSuccess) e = hipStreamWaitEvent(ex->side, ex->fork_ev, 0);
    if (e != hipSuccess) return e;
    const hipError_t eq =
        with_q_settings(c, ex->side, [&]() { return pk_q_block(c, q, k, x, y, nrhs, pd); });
    // join even after an error, so that a capture on `main` stays well formed
    e = hipEventRecord(ex->join_ev, ex->side);
    const hipError_t ev = pk_v_block(c, q, k, x, y, nrhs, pd);
    if (e == hipSuccess) e = hipStreamWaitEvent(main, ex->join_ev, 0);
    if (eq != hipSuccess) return eq;
    if (ev != hipSuccess) return ev;
    return e;
}

// ---- device memory --------------------------------------------------------------------
hp_status alloc_device(double** p, size_t doubles) {
    if (hipMalloc(reinterpret_cast<void**>(p), std::max<size_t>(doubles, 1) * sizeof(double)) !=
        hipSuccess)
        return HP_ENOMEM;
    return HP_OK;
}

hp_status ensure_krylov(hp_ctx* c, size_t doubles) {
    Extra* ex = extra_of(c);
    if (ex->kv_doubles >= doubles) return HP_OK;
    if (ex->kv) (void)hipFree(ex->kv);
    ex->kv = nullptr;
    ex->kv_doubles = 0;
    hp_status s = alloc_device(&ex->kv, doubles);
    if (s != HP_OK) return s;
    ex->kv_doubles = doubles;
    return HP_OK;
}

hp_status stage_coef(hp_ctx* c, const std::vector<double>& v) {
    Extra* ex = extra_of(c);
    if (v.size() > ex->coef_doubles) return HP_EINVAL;
    std::memcpy(ex->hcoef, v.data(), v.size() * sizeof(double));
    if (hipMemcpyAsync(ex->dcoef, ex->hcoef, v.size() * sizeof(double), hipMemcpyHostToDevice,
                       c->stream) != hipSuccess)
        return HP_EHIP;
    // the pinned staging buffer is reused: wait until the copy has been consumed
    if (hipStreamSynchronize(c->stream) != hipSuccess) return HP_EHIP;
    return HP_OK;
}


// ---- MINRES (preconditioned; Lanczos in the P^{-1} inner product) ------------------
// All recurrence scalars live on the device (k_minres_* kernels), so one
// iteration is a fixed sequence of launches: it is captured once per
// buffer-rotation phase (period 6) as a HIP graph and replayed.  The host
// reads the per-rhs convergence flags one iteration behind the GPU.
struct MinresBufs {
    double *vo, *v, *vn, *z, *zn, *wo, *w, *wn, *Kz, *x;
};

MinresBufs minres_bufs(hp_ctx* c, int phase, int nrhs) {
    const long long V = c->N * (long long)c->opts.max_rhs;
    double* base = extra_of(c)->kv;
    double* vb[3] = {base, base + V, base + 2 * V};
    double* zb[2] = {base + 3 * V, base + 4 * V};
    double* wb[3] = {base + 5 * V, base + 6 * V, base + 7 * V};
    MinresBufs b;
    b.vo = vb[phase % 3];
    b.v = vb[(phase + 1) % 3];
    b.vn = vb[(phase + 2) % 3];
    b.z = zb[phase % 2];
    b.zn = zb[(phase + 1) % 2];
    b.wo = wb[phase % 3];
    b.w = wb[(phase + 1) % 3];
    b.wn = wb[(phase + 2) % 3];
    b.Kz = base + 8 * V;
    b.x = base + 9 * V;
    (void)nrhs;
    return b;
}

// One MINRES iteration; it reads the scalar state msc[cur] and writes the
// next one to msc[cur ^ 1] and to the host mirror `mirror` (device address
// of pinned host memory).  Its pieces: K z and (Kz . z); one update launch
// that finishes the previous iteration (its rotation and w/x update, from the
// partials of (z . v) its P_k left; skipped in the first iteration, pb null)
// and forms v_new; then P_k as the Q block beside the V block, whose launches
// leave the partials of (z_new . v_new) for the next iteration's update (or
// for minres_w_step after the last one).  pb: the previous iteration's
// buffers; polled (may be null): an event recorded after the update launch,
// which marks the point where the previous iteration's flags are final.
PkDot minres_pk_dot(hp_ctx* c, const MinresBufs& b) {
    Extra* ex = extra_of(c);
    return PkDot{b.vn, ex->mfg, ex->mfq};
}
hipError_t minres_w_step(hp_ctx* c, const MinresBufs& b, int nrhs, double tol,
                         MinresScalars* mirror, int cur) {
    Extra* ex = extra_of(c);
    const long long N = c->N;
    const int R = c->opts.max_rhs;
    const PkDot pd = minres_pk_dot(c, b);
    return minres_w(c->stream, N, N, nrhs, b.z, b.wo, b.w, b.wn, b.x, ex->msc + cur * R,
                    ex->msc + (cur ^ 1) * R, Partials{pd.vpart, fd_dot_count(c, true)},
                    Partials{pd.qpart, fd_dot_count(c, false)}, tol, c->opts.breakdown_tol,
                    mirror);
}

hipError_t minres_iteration(hp_ctx* c, const MinresBufs& b, const MinresBufs* pb, int nrhs,
                            double tol, MinresScalars* mirror, int cur, hipEvent_t polled) {
    Extra* ex = extra_of(c);
    const long long N = c->N;
    const int R = c->opts.max_rhs;
    double* p0 = ex->mpart;
    hipError_t e;
    if ((e = launch_forward(c, b.z, b.Kz, nrhs)) != hipSuccess) return e;
    if ((e = vec_dot_partials(c->stream, N, N, b.Kz, b.z, nrhs, p0)) != hipSuccess) return e;
    const MinresBufs& q = pb ? *pb : b;  // the w/x vectors are not touched without pb
    const Partials pa = pb ? Partials{ex->mfg, fd_dot_count(c, true)} : Partials{nullptr, 0};
    const Partials pq = pb ? Partials{ex->mfq, fd_dot_count(c, false)} : Partials{nullptr, 0};
    if ((e = minres_wv(c->stream, N, N, nrhs, b.Kz, b.v, b.vo, b.vn, q.z, q.wo, q.w, q.wn, b.x,
                       ex->msc + cur * R, ex->msc + (cur ^ 1) * R,
                       Partials{p0, vec_dot_partial_count(N)}, pa, pq, tol,
                       c->opts.breakdown_tol, mirror)) != hipSuccess)
        return e;
    if (polled && (e = hipEventRecord(polled, c->stream)) != hipSuccess) return e;
    const PkDot pd = minres_pk_dot(c, b);
    return apply_Pk(c, c->opts.order, c->opts.iters, b.vn, b.zn, nrhs, &pd);
}

void drop_graphs(Extra* ex) {
    for (auto& g : ex->g_exec)
        if (g) {
            (void)hipGraphExecDestroy(g);
            g = nullptr;
        }
    ex->g_valid = false;
}

// Captures fn() on the capture stream and instantiates it into *out.
template <typename F>
hp_status capture_graph(hp_ctx* c, hipGraphExec_t* out, F fn) {
    Extra* ex = extra_of(c);
    hipGraph_t g = nullptr;
    if (hipStreamBeginCapture(ex->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) return HP_EHIP;
    const hipError_t e = fn();
    const hipError_t e2 = hipStreamEndCapture(ex->cap, &g);
    hp_status st = (e != hipSuccess || e2 != hipSuccess) ? HP_EHIP : HP_OK;
    if (st == HP_OK && hipGraphInstantiate(out, g, nullptr, nullptr, 0) != hipSuccess) st = HP_EHIP;
    if (g) (void)hipGraphDestroy(g);
    return st;
}

// Graphs of the MINRES iterations, one per buffer-rotation phase (period 6);
// the Q block of P_k is a parallel branch of each.
hp_status build_graphs(hp_ctx* c, int nrhs, double tol) {
    Extra* ex = extra_of(c);
    const hp_opts& o = c->opts;
    if (ex->g_valid && ex->g_q == o.order && ex->g_k == o.iters && ex->g_nrhs == nrhs &&
        ex->g_var == o.schur_variant && ex->g_sched == o.l_schedule && ex->g_prec == o.precision &&
        ex->g_tol == tol && ex->g_nu == c->nu && ex->g_kv == ex->kv)
        return HP_OK;
    drop_graphs(ex);
    hipStream_t user = c->stream;
    c->stream = ex->cap;
    hp_status st = HP_OK;
    for (int ph = 0; ph < 6 && st == HP_OK; ++ph) {
        // iteration it (phase (it-1) % 6) reads state it & 1 and is polled
        // through mirror it & 1; the graphs serve iterations 2, 3, ... (the
        // first has no previous iteration to finish)
        const MinresBufs bb = minres_bufs(c, ph, nrhs);
        const MinresBufs bp = minres_bufs(c, (ph + 5) % 6, nrhs);
        const int cur = (ph + 1) & 1;
        st = capture_graph(c, &ex->g_exec[ph], [&]() {
            return minres_iteration(c, bb, &bp, nrhs, tol, ex->dmsc[cur], cur, nullptr);
        });
    }
    c->stream = user;
    if (st != HP_OK) {
        drop_graphs(ex);
        return st;
    }
    ex->g_valid = true;
    ex->g_q = o.order;
    ex->g_k = o.iters;
    ex->g_nrhs = nrhs;
    ex->g_var = o.schur_variant;
    ex->g_sched = o.l_schedule;
    ex->g_prec = o.precision;
    ex->g_tol = tol;
    ex->g_nu = c->nu;
    ex->g_kv = ex->kv;
    return HP_OK;
}

hp_status minres(hp_ctx* c, const double* b, double* x, int nrhs, double tol, hp_solve_info* info) {
    Extra* ex = extra_of(c);
    const long long N = c->N;
    const long long V = N * nrhs;
    if (ensure_krylov(c, 10 * N * (size_t)c->opts.max_rhs) != HP_OK) return HP_ENOMEM;
    const bool graphs = c->opts.use_graph != 0;
    if (graphs && build_graphs(c, nrhs, tol) != HP_OK) return HP_EHIP;
    MinresBufs b0 = minres_bufs(c, 0, nrhs);
    const bool warm = c->opts.use_x0 != 0;
    double* ref_part = ex->mpart + vec_partial_doubles(1, c->opts.max_rhs);
    if (warm) {
        // start residual v = b - K x_0 (x is updated in place from x_0), and
        // ||b||_{P^{-1}} for the stopping test (z = P_k^{-1} b)
        HIPCHK(vec_copy(c->stream, V, x, b0.x));
        HIPCHK(launch_forward(c, b0.x, b0.v, nrhs));
        HIPCHK(vec_axpby(c->stream, V, 1.0, b, -1.0, b0.v));
        HIPCHK(apply_Pk(c, c->opts.order, c->opts.iters, b, b0.z, nrhs));
        HIPCHK(vec_dot_partials(c->stream, N, N, b0.z, b, nrhs, ref_part));
    } else {
        HIPCHK(vec_zero(c->stream, V, b0.x));
        HIPCHK(vec_copy(c->stream, V, b, b0.v));
    }
    HIPCHK(vec_zero(c->stream, V, b0.vo));
    HIPCHK(vec_zero(c->stream, V, b0.wo));
    HIPCHK(vec_zero(c->stream, V, b0.w));
    HIPCHK(apply_Pk(c, c->opts.order, c->opts.iters, b0.v, b0.z, nrhs));
    HIPCHK(vec_dot_partials(c->stream, N, N, b0.z, b0.v, nrhs, ex->mpart));
    // iteration it reads the state msc[it & 1]: the first reads msc[1]
    MinresScalars* s1 = ex->msc + c->opts.max_rhs;
    HIPCHK(minres_init(c->stream, s1, ex->mpart, warm ? ref_part : nullptr,
                       (int)vec_dot_partial_count(N), tol, nrhs));
    const size_t sbytes = sizeof(MinresScalars) * nrhs;
    auto all_done = [&](const MinresScalars* h) {
        for (int r = 0; r < nrhs; ++r)
            if (!h[r].done) return false;
        return true;
    };
    HIPCHK(hipMemcpyAsync(ex->hmsc[0], s1, sbytes, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    int it = 0;
    const int lag = c->opts.poll_lag;
    bool finished = all_done(ex->hmsc[0]);
    while (!finished && it < c->opts.maxit) {
        const int ph = it % 6;
        ++it;
        if (graphs && it > 1) {
            HIPCHK(hipGraphLaunch(ex->g_exec[ph], c->stream));
            HIPCHK(hipEventRecord(ex->mev[it & 3], c->stream));
        } else {
            const MinresBufs bp = minres_bufs(c, (ph + 5) % 6, nrhs);
            HIPCHK(minres_iteration(c, minres_bufs(c, ph, nrhs), it > 1 ? &bp : nullptr, nrhs,
                                    tol, ex->dmsc[it & 1], it & 1, ex->mev[it & 3]));
        }
        // the flags of iteration it - lag are final once the update launch of
        // iteration it - lag + 1 has run (its mirror slot may already hold a
        // later state: done is monotone).  Launched directly, that launch is
        // marked by its own event, and the host waits for it with the rest of
        // iteration it - lag + 1 still queued (for lag 1, P_k of iteration it:
        // measured at 32^3, the device does not wait for the host then, and
        // one iteration less runs past convergence); a graph is marked at
        // its end only, so the host waits for iteration it - lag.
        const int pj = graphs ? it - lag : it - lag + 1;
        if (pj >= 1) {
            HIPCHK(hipEventSynchronize(ex->mev[pj & 3]));
            finished = all_done(ex->hmsc[pj & 1]);
        }
    }
    // the last iteration's rotation and w/x update (nothing for a state
    // already done); after it the state is msc[it & 1] (msc[1], from
    // minres_init, when no iteration ran)
    if (it > 0)
        HIPCHK(minres_w_step(c, minres_bufs(c, (it - 1) % 6, nrhs), nrhs, tol, nullptr,
                             (it + 1) & 1));
    HIPCHK(hipStreamSynchronize(c->stream));
    const int fin = it > 0 ? (it & 1) : 1;
    const MinresScalars* h = ex->hmsc[fin];
    HIPCHK(hipMemcpy(ex->hmsc[fin], ex->msc + fin * c->opts.max_rhs, sbytes,
                     hipMemcpyDeviceToHost));
    HIPCHK(vec_copy(c->stream, V, b0.x, x));
    hp_status status = HP_OK;
    bool conv = true;
    if (info) {
        info->iterations = 0;
        info->relres = 0.0;
    }
    for (int r = 0; r < nrhs; ++r) {
        if (h[r].status != 0 && status == HP_OK) status = (hp_status)h[r].status;
        if (!h[r].done) conv = false;
        if (info) {
            info->iterations = std::max(info->iterations, h[r].iters);
            info->relres = std::max(info->relres, h[r].rel);
            if (r < 64) info->iters_per_rhs[r] = h[r].iters;
        }
    }
    if (info) info->converged = conv && status == HP_OK;
    if (status != HP_OK) return status;
    return conv ? HP_OK : HP_ENOCONV;
}

// ---- FGMRES(m), right preconditioned, CGS2 Arnoldi -----------------------------------
// Hessenberg matrix, Givens rotations and the small least-squares solve run
// on the device (k_fg_* kernels); iteration j of a cycle is captured as graph
// j and replayed.  The true residual is checked at the end of every cycle.
constexpr int FG_MMAX = 128;

// One Arnoldi step j of FGMRES(m); the updated scalars are also written to
// the host mirror `mirror` (device address of pinned host memory).  polled (may
// be null) is recorded where they are final, before the new basis vector is
// scaled.
hipError_t fgmres_iteration(hp_ctx* c, int j, int m, int nrhs, double tol, FgScalars* mirror,
                            hipEvent_t polled = nullptr) {
    Extra* ex = extra_of(c);
    const long long N = c->N;
    const long long V = N * (long long)c->opts.max_rhs;
    double* Vb = ex->kv;
    double* Zb = Vb + (long long)(m + 1) * V;
    double* w = Zb + (long long)m * V;
    double* Vj = Vb + (long long)j * V;
    double* Zj = Zb + (long long)j * V;
    const int cnt = (int)vec_dot_partial_count(N);
    hipError_t e;
    if ((e = apply_Pk(c, c->opts.order, c->opts.iters, Vj, Zj, nrhs)) != hipSuccess) return e;
    if ((e = launch_forward(c, Zj, w, nrhs)) != hipSuccess) return e;
    // two passes: w -> w - V h (kept in V_{j+1}) -> w
    double* Vn = Vb + (long long)(j + 1) * V;
    auto coef = [&](int pass) {
        return fg_h(c->stream, ex->fsc, ex->fpart, cnt, ex->fH, ex->fhc, j, pass, m, nrhs);
    };
    if ((e = gs_dots(c->stream, N, N, Vb, V, j + 1, w, nrhs, ex->fpart)) != hipSuccess) return e;
    if ((e = coef(0)) != hipSuccess) return e;
    if ((e = gs_update_dots(c->stream, N, N, Vb, V, j + 1, ex->fhc, m + 1, w, Vn, nrhs, ex->fpart)) !=
        hipSuccess)
        return e;
    if ((e = coef(1)) != hipSuccess) return e;
    if ((e = gs_update_norm(c->stream, N, N, Vb, V, j + 1, ex->fhc, m + 1, Vn, w, nrhs, ex->fpart)) !=
        hipSuccess)
        return e;
    if ((e = fg_rot(c->stream, ex->fsc, ex->fpart, cnt, ex->fH, ex->fcs, ex->fsn, ex->fg, ex->fvs, tol,
                    c->opts.breakdown_tol, j, m, nrhs, mirror)) != hipSuccess)
        return e;
    if (polled && (e = hipEventRecord(polled, c->stream)) != hipSuccess) return e;
    const double* xs[1] = {w};
    return vec_lincomb(c->stream, N, N, nrhs, 1, xs, ex->fvs, Vn);
}

void drop_fg_graphs(Extra* ex) {
    for (auto& g : ex->f_exec)
        if (g) (void)hipGraphExecDestroy(g);
    ex->f_exec.clear();
    ex->f_valid = false;
}

hp_status build_fg_graphs(hp_ctx* c, int m, int nrhs, double tol) {
    Extra* ex = extra_of(c);
    const hp_opts& o = c->opts;
    if (ex->f_valid && ex->f_q == o.order && ex->f_k == o.iters && ex->f_nrhs == nrhs &&
        ex->f_var == o.schur_variant && ex->f_sched == o.l_schedule && ex->f_prec == o.precision &&
        ex->f_m == m && ex->f_tol == tol && ex->f_nu == c->nu && ex->f_kv == ex->kv)
        return HP_OK;
    drop_fg_graphs(ex);
    hipStream_t user = c->stream;
    c->stream = ex->cap;
    hp_status st = HP_OK;
    ex->f_exec.assign(m, nullptr);
    for (int j = 0; j < m && st == HP_OK; ++j) {
        hipGraph_t g = nullptr;
        if (hipStreamBeginCapture(ex->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
            st = HP_EHIP;
            break;
        }
        // step j is polled through mirror (j + 1) & 1
        hipError_t e = fgmres_iteration(c, j, m, nrhs, tol, ex->dfsc[(j + 1) & 1]);
        hipError_t e2 = hipStreamEndCapture(ex->cap, &g);
        if (e != hipSuccess || e2 != hipSuccess) st = HP_EHIP;
        if (st == HP_OK && hipGraphInstantiate(&ex->f_exec[j], g, nullptr, nullptr, 0) != hipSuccess)
            st = HP_EHIP;
        if (g) (void)hipGraphDestroy(g);
    }
    c->stream = user;
    if (st != HP_OK) {
        drop_fg_graphs(ex);
        return st;
    }
    ex->f_valid = true;
    ex->f_q = o.order;
    ex->f_k = o.iters;
    ex->f_nrhs = nrhs;
    ex->f_var = o.schur_variant;
    ex->f_sched = o.l_schedule;
    ex->f_prec = o.precision;
    ex->f_m = m;
    ex->f_tol = tol;
    ex->f_nu = c->nu;
    ex->f_kv = ex->kv;
    return HP_OK;
}

hp_status fgmres(hp_ctx* c, const double* b, double* x, int nrhs, double tol, hp_solve_info* info) {
    Extra* ex = extra_of(c);
    const long long N = c->N;
    const int m = std::max(1, std::min(c->opts.restart, FG_MMAX));
    const long long Vn = N * nrhs;
    const long long V = N * (long long)c->opts.max_rhs;
    if (ensure_krylov(c, (size_t)(2 * m + 2) * V) != HP_OK) return HP_ENOMEM;
    const bool graphs = c->opts.use_graph != 0;
    if (graphs && build_fg_graphs(c, m, nrhs, tol) != HP_OK) return HP_EHIP;
    double* Vb = ex->kv;
    double* Zb = Vb + (long long)(m + 1) * V;
    double* w = Zb + (long long)m * V;
    const size_t sbytes = sizeof(FgScalars) * nrhs;
    // The flags are read one step behind, so that the GPU never waits for the
    // host, at the price of one step past convergence -- unless the scaling of
    // the new vector alone, 2^22 entries in 15 us, covers the host's way back:
    // then the step's own flags are waited for (48^3, degree 2, 32 right-hand
    // sides: 30 steps of 2.2 ms instead of 31).
    const bool wait = !graphs && N * (long long)nrhs >= (1LL << 22);
    HIPCHK(vec_dot_partials(c->stream, N, N, b, b, nrhs, ex->fpart));
    HIPCHK(fg_init(c->stream, ex->fsc, ex->fpart, (int)vec_dot_partial_count(N), nrhs));
    // x_0 = 0, or the x passed in (warm start): every cycle starts from b - K x
    if (!c->opts.use_x0) HIPCHK(vec_zero(c->stream, Vn, x));
    auto all = [&](const FgScalars* h, bool active) {
        for (int r = 0; r < nrhs; ++r)
            if (active ? h[r].active : !h[r].done) return false;
        return true;
    };
    HIPCHK(hipMemcpyAsync(ex->hfsc[0], ex->fsc, sbytes, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(hipStreamSynchronize(c->stream));
    bool done = all(ex->hfsc[0], false);
    int total = 0;
    while (!done && total < c->opts.maxit) {
        // cycle start: w = b - K x, V0 = w / ||w||
        HIPCHK(launch_forward(c, x, w, nrhs));
        HIPCHK(vec_axpby(c->stream, Vn, 1.0, b, -1.0, w));
        HIPCHK(vec_dot_partials(c->stream, N, N, w, w, nrhs, ex->fpart));
        HIPCHK(fg_begin(c->stream, ex->fsc, ex->fpart, (int)vec_dot_partial_count(N), ex->fg,
                        ex->fvs, m, nrhs));
        {
            const double* xs[1] = {w};
            HIPCHK(vec_lincomb(c->stream, N, N, nrhs, 1, xs, ex->fvs, Vb));
        }
        int jl = 0;
        bool stop = false;
        while (jl < m && total < c->opts.maxit && !stop) {
            if (graphs) {
                HIPCHK(hipGraphLaunch(ex->f_exec[jl], c->stream));
            } else {
                HIPCHK(fgmres_iteration(c, jl, m, nrhs, tol, ex->dfsc[(jl + 1) & 1],
                                        ex->mev[(jl + 1) & 1]));
            }
            ++jl;
            ++total;
            if (graphs) HIPCHK(hipEventRecord(ex->mev[jl & 1], c->stream));
            if (wait) {
                HIPCHK(hipEventSynchronize(ex->mev[jl & 1]));
                stop = all(ex->hfsc[jl & 1], true);
            } else if (jl >= 2) {
                HIPCHK(hipEventSynchronize(ex->mev[(jl - 1) & 1]));
                stop = all(ex->hfsc[(jl - 1) & 1], true);
            }
        }
        // x += Z y with H y = g
        HIPCHK(fg_solve(c->stream, ex->fsc, ex->fH, ex->fg, ex->fy, m, jl, nrhs));
        HIPCHK(vec_add_combo(c->stream, N, N, Zb, V, jl, ex->fy, m, nrhs, x));
        // true residual
        HIPCHK(launch_forward(c, x, w, nrhs));
        HIPCHK(vec_axpby(c->stream, Vn, 1.0, b, -1.0, w));
        HIPCHK(vec_dot_partials(c->stream, N, N, w, w, nrhs, ex->fpart));
        HIPCHK(fg_check(c->stream, ex->fsc, ex->fpart, (int)vec_dot_partial_count(N), tol, nrhs));
        HIPCHK(hipMemcpyAsync(ex->hfsc[0], ex->fsc, sbytes, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(hipStreamSynchronize(c->stream));
        done = all(ex->hfsc[0], false);
    }
    const FgScalars* h = ex->hfsc[0];
    hp_status status = HP_OK;
    if (info) {
        info->iterations = 0;
        info->relres = 0.0;
        info->converged = 1;
    }
    for (int r = 0; r < nrhs; ++r) {
        if (h[r].status != 0 && status == HP_OK) status = (hp_status)h[r].status;
        if (info) {
            info->iterations = std::max(info->iterations, h[r].iters);
            info->relres = std::max(info->relres, h[r].rel);
            if (!h[r].done) info->converged = 0;
            if (r < 64) info->iters_per_rhs[r] = h[r].iters;
        }
    }
    if (status != HP_OK) return status;
    return done ? HP_OK : HP_ENOCONV;
}

// ---- right-hand side -------------------------------------------------------------------
hp_status build_rhs(hp_ctx* c, const double* lid, int nmodes, const double* amp, const int* waves,
                    const double* beta, double* b, int nrhs) {
    const Tables1D& T = c->tab;
    const int nN = c->nN, nM = c->nM;
    // per (rhs, component): factors s1, s2, s3 (each nt terms) assembled on the host
    // from 1D quadrature; the 3D sums run on the device.
    const int nt = nmodes + 1;
    const int nmax = std::max(nN, nM);
    std::vector<double> hs((size_t)3 * nt * nmax);
    double* ds = nullptr;
    if (alloc_device(&ds, hs.size()) != HP_OK) return HP_ENOMEM;
    hp_status st = HP_OK;
    HIPCHK(vec_zero(c->stream, c->N * nrhs, b));
    for (int r = 0; r < nrhs && st == HP_OK; ++r) {
        for (int comp = 0; comp < 3; ++comp) {
            int n[3];
            for (int d = 0; d < 3; ++d) n[d] = (int)c->dims[comp][d];
            std::fill(hs.begin(), hs.end(), 0.0);
            int cnt = 0;
            double* s1 = hs.data();
            double* s2 = s1 + (size_t)nt * nmax;
            double* s3 = s2 + (size_t)nt * nmax;
            if (comp == 0 && lid && lid[r] != 0.0) {
                // F_u1 = 2 nu U (int N) (x) (int M) (x) (alpha M(1) - M'(1)/2)
                for (int i = 0; i < nN; ++i) s1[cnt * n[0] + i] = T.int_N[i];
                for (int i = 0; i < nM; ++i) s2[cnt * n[1] + i] = T.int_M[i];
                for (int i = 0; i < nM; ++i) s3[cnt * n[2] + i] = 2.0 * c->nu * lid[r] * T.lid3[i];
                ++cnt;
            }
            for (int mo = 0; mo < nmodes; ++mo) {
                size_t id = ((size_t)r * 3 + comp) * nmodes + mo;
                double a = amp[id];
                if (a == 0.0) continue;
                double* dst[3] = {s1 + (size_t)cnt * n[0], s2 + (size_t)cnt * n[1],
                                  s3 + (size_t)cnt * n[2]};
                for (int d = 0; d < 3; ++d) {
                    std::vector<double> l = sine_load(T, d == comp ? 0 : 1, waves[id * 3 + d]);
                    for (int i = 0; i < n[d]; ++i) dst[d][i] = (d == 2 ? a : 1.0) * l[i];
                }
                ++cnt;
            }
            if (cnt == 0) continue;
            // pack contiguously: s1 (cnt x n0), s2 (cnt x n1), s3 (cnt x n2)
            std::vector<double> pk;
            pk.insert(pk.end(), s1, s1 + (size_t)cnt * n[0]);
            pk.insert(pk.end(), s2, s2 + (size_t)cnt * n[1]);
            pk.insert(pk.end(), s3, s3 + (size_t)cnt * n[2]);
            if (hipMemcpyAsync(ds, pk.data(), pk.size() * sizeof(double), hipMemcpyHostToDevice,
                               c->stream) != hipSuccess) { st = HP_EHIP; break; }
            if (rank1_sum(c->stream, n[0], n[1], n[2], cnt, ds, ds + (size_t)cnt * n[0],
                          ds + (size_t)cnt * (n[0] + n[1]), b + r * c->N + c->off[comp]) !=
                hipSuccess) { st = HP_EHIP; break; }
            if (hipStreamSynchronize(c->stream) != hipSuccess) { st = HP_EHIP; break; }
        }
    }
    // body force with coefficients beta in V_h: b_u += M_V beta
    if (st == HP_OK && beta) {
        const Fields bu = vel_of_full(c, b);
        if (launch_operator(c, OP_MV, vel_fields(c, beta, c->nV), bu, 1.0, 1.0, &bu, nrhs) !=
            hipSuccess)
            st = HP_EHIP;
    }
    (void)hipStreamSynchronize(c->stream);
    (void)hipFree(ds);
    return st;
}

static void upload_band(const std::vector<double>& A, int n, int w, double* dst) {
    const int W = 2 * w + 1;
    std::vector<double> b((size_t)n * W, 0.0);
    for (int i = 0; i < n; ++i)
        for (int t = 0; t < W; ++t) {
            int j = i + t - w;
            if (j >= 0 && j < n) b[(size_t)i * W + t] = A[(size_t)i * n + j];
        }
    (void)hipMemcpy(dst, b.data(), b.size() * sizeof(double), hipMemcpyHostToDevice);
}

// ---- autotuner ----------------------------------------------------------------------
constexpr int TUNE_PASSES = 2;  // passes over the candidate list (fastest kept)
constexpr int TUNE_REPS = 5;    // timed launches per candidate and pass

// Times fn() (reps launches after one warm-up) on the context stream, in us.
template <typename F>
double time_launches(hp_ctx* c, hipEvent_t e0, hipEvent_t e1, int reps, F fn) {
    if (fn() != hipSuccess) return -1.0;
    if (hipEventRecord(e0, c->stream) != hipSuccess) return -1.0;
    for (int i = 0; i < reps; ++i)
        if (fn() != hipSuccess) return -1.0;
    float ms = 0.0f;
    if (hipEventRecord(e1, c->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        return -1.0;
    return 1e3 * ms / reps;
}

// Picks the operator launch shape (for 1 and max_rhs right-hand sides) and
// the P_0 plan (per precision) by timing them on zero vectors.  Only the
// launch configuration changes, never the arithmetic of a point.
hp_status autotune(hp_ctx* c) {
    const long long R = c->opts.max_rhs, N = c->N;
    double *x = nullptr, *y = nullptr;
    if (hipMalloc(reinterpret_cast<void**>(&x), sizeof(double) * N * R) != hipSuccess) return HP_ENOMEM;
    if (hipMalloc(reinterpret_cast<void**>(&y), sizeof(double) * N * R) != hipSuccess) {
        (void)hipFree(x);
        return HP_ENOMEM;
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hp_status st = HP_OK;
    if (hipMemsetAsync(x, 0, sizeof(double) * N * R, c->stream) != hipSuccess ||
        hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        st = HP_EHIP;
    const Fields fx = full_fields(c, x), fy = full_fields(c, y);
    // Each candidate is timed in TUNE_PASSES passes over the whole list and
    // keeps its fastest pass, so that a slow moment (clock changes, other
    // work on the device) does not decide; the device is warmed up first.
    for (int i = 0; i < 20 && st == HP_OK; ++i)
        if (launch_operator(c, OP_K, fx, fy, 1.0, 0.0, nullptr, 1) != hipSuccess) st = HP_EHIP;
    // operator: chunk lengths x the two velocity workgroup orders (x slabs)
    const int nrhs_list[2] = {1, (int)R};
    for (int e = 0; e < (R > 1 ? 2 : 1) && st == HP_OK && c->opts.op_kchunk == 0; ++e) {
        const int nr = nrhs_list[e];
        static const int cand[] = {2, 3, 4, 6, 8, 12, 16, 20, 25, 32, 40, 48, 64};
        std::vector<OpShape> shapes;
        for (int kc : cand) {
            if (kc > c->nM) break;
            for (int order = 0; order <= 1; ++order)
                for (int slabs = 1; slabs <= 4; slabs *= 2)
                    for (int staged = 0; staged <= 1; ++staged)
                        for (int pwide = 0; pwide <= 1; ++pwide) {
                            if (c->opts.op_order >= 0 && order != c->opts.op_order) continue;
                            if (c->opts.op_slabs > 0 ? slabs != c->opts.op_slabs
                                                     : (slabs > 1 && c->nM < 64))
                                continue;
                            if (c->opts.op_staged >= 0 && staged != c->opts.op_staged) continue;
                            if (staged && !op_staged_ok(c->p, kc)) continue;
                            // the 32 x 8 pressure tiles: streaming kernels, 32+ points wide
                            if (pwide && (staged || c->nM < 32)) continue;
                            if (c->opts.op_pres_wide >= 0 && pwide != c->opts.op_pres_wide)
                                continue;
                            OpShape sh{kc, order, slabs, 0, staged};
                            sh.pwide = pwide;
                            sh.dma = c->opts.op_dma != 0;
                            shapes.push_back(sh);
                        }
        }
        std::vector<double> us(shapes.size(), -1.0);
        for (int pass = 0; pass < TUNE_PASSES && st == HP_OK; ++pass)
            for (size_t i = 0; i < shapes.size() && st == HP_OK; ++i) {
                c->op_force = shapes[i];
                const double t = time_launches(c, e0, e1, TUNE_REPS, [&]() {
                    return launch_operator(c, OP_K, fx, fy, 1.0, 0.0, nullptr, nr);
                });
                if (t < 0.0) st = HP_EHIP;
                else if (us[i] < 0.0 || t < us[i]) us[i] = t;
            }
        double best = -1.0;
        OpShape best_sh = op_model_shape(c, nr);
        for (size_t i = 0; i < shapes.size(); ++i)
            if (us[i] >= 0.0 && (best < 0.0 || us[i] < best)) {
                best = us[i];
                best_sh = shapes[i];
            }
        c->op_force = OpShape{0, 1, 1};
        c->op_tuned[e].nrhs = nr;
        c->op_tuned[e].kchunk = best_sh.kchunk;
        c->op_tuned[e].shape = best_sh;
        c->op_tuned_us[e] = best;
    }
    // P_0: every plan that fits, per precision (velocity and pressure blocks)
    for (int prec = 0; prec < 3 && st == HP_OK && c->fd_ok && c->opts.fd_plan < 0; ++prec) {
        double us[FD_PLAN_LAST + 1];
        for (double& u : us) u = -1.0;
        for (int pass = 0; pass < TUNE_PASSES && st == HP_OK; ++pass)
            for (int plan = 0; plan <= FD_PLAN_LAST && st == HP_OK; ++plan) {
                if (!fd_plan_valid(c, prec, plan)) continue;
                // the plane plans alone where they exist: they agree bit for
                // bit, the passes do not, for little or no gain (us, planes and
                // passes: 96^3 123.7 and 122.3, FP32 80.8 and 91.8; 120^3 183.4
                // and 181.2, FP32 105.7 and 118.2)
                if (fd_plan_lines(plan) && fd_plan_valid(c, prec, FD_PLAN_PLANE)) continue;
                c->fd_force = plan;
                const double t = time_launches(c, e0, e1, TUNE_REPS, [&]() {
                    return launch_P0(c, fx, fy, true, true, false, prec, 1);
                });
                if (t < 0.0) st = HP_EHIP;
                else if (us[plan] < 0.0 || t < us[plan]) us[plan] = t;
            }
        double best = -1.0;
        int best_plan = -1;
        for (int plan = 0; plan <= FD_PLAN_LAST; ++plan)
            if (us[plan] >= 0.0 && (best < 0.0 || us[plan] < best)) {
                best = us[plan];
                best_plan = plan;
            }
        c->fd_force = -1;
        c->fd_tuned[prec] = best_plan;
        c->fd_tuned_us[prec] = best;
    }
    c->op_force = OpShape{0, 1, 1};
    c->fd_force = -1;
    if (hipStreamSynchronize(c->stream) != hipSuccess && st == HP_OK) st = HP_EHIP;
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(x);
    (void)hipFree(y);
    return st;
}

// ---- spectra of the preconditioned blocks (Sec. 2, Sec. 5.2) ------------------------
// Number of eigenvalues below x of the symmetric tridiagonal matrix
// tridiag(b; a; b) (Sturm sequence of the LDL' pivots).
int sturm_below(const std::vector<double>& a, const std::vector<double>& b, double x) {
    int cnt = 0;
    double d = 1.0;
    for (size_t i = 0; i < a.size(); ++i) {
        d = (a[i] - x) - (i ? b[i - 1] * b[i - 1] / d : 0.0);
        if (d == 0.0) d = -1e-300;
        if (d < 0.0) ++cnt;
    }
    return cnt;
}

// Smallest (which = 1) or largest (which = m) eigenvalue by bisection inside
// the Gershgorin interval.
double tridiag_eig(const std::vector<double>& a, const std::vector<double>& b, int which) {
    const int m = (int)a.size();
    double lo = a[0], hi = a[0];
    for (int i = 0; i < m; ++i) {
        double r = (i ? std::fabs(b[i - 1]) : 0.0) + (i + 1 < m ? std::fabs(b[i]) : 0.0);
        lo = std::min(lo, a[i] - r);
        hi = std::max(hi, a[i] + r);
    }
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi) break;
        if (sturm_below(a, b, mid) >= which) hi = mid;
        else lo = mid;
    }
    return 0.5 * (lo + hi);
}

// The constant pressure n = n1 (x) n1 (x) n1 (null vector of B; n1 = M^^{-1} 1
// since B = D' M_q and D' annihilates constants), unit Euclidean norm.
std::vector<double> pressure_null(const hp_ctx* c) {
    const int nM = c->nM;
    std::vector<double> n1(nM, 0.0);
    for (int i = 0; i < nM; ++i)
        for (int j = 0; j < nM; ++j) n1[i] += c->tab.Mcinv[(size_t)i * nM + j];
    double s = 0.0;
    for (double v : n1) s += v * v;
    const double inv = 1.0 / std::pow(s, 1.5);
    std::vector<double> n((size_t)nM * nM * nM);
    size_t t = 0;
    for (int i3 = 0; i3 < nM; ++i3)
        for (int i2 = 0; i2 < nM; ++i2)
            for (int i1 = 0; i1 < nM; ++i1) n[t++] = n1[i1] * n1[i2] * n1[i3] * inv;
    return n;
}

struct DevBuf {
    double* p = nullptr;
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
};

// Lanczos in the inner product of the preconditioner (see hp_spectrum).
hp_status spectrum(hp_ctx* c, int block, int q, int k, int sl, int steps, const double* start,
                   std::vector<double>& al, std::vector<double>& be) {
    const bool vel = block == HP_SPEC_VELOCITY;
    const long long n = vel ? c->nV : c->nQ;
    const int prec = c->opts.precision;
    DevBuf mem;
    if (alloc_device(&mem.p, (size_t)6 * n) != HP_OK) return HP_ENOMEM;
    double* v = mem.p;
    double* pv = v + n;       // P v_j = r_j / beta_j
    double* pvp = v + 2 * n;  // P v_{j-1}
    double* r = v + 3 * n;
    double* z = v + 4 * n;
    double* nul = v + 5 * n;
    auto F = [&](double* b) { return vel ? vel_fields(c, b, n) : pres_fields(c, b, n); };
    auto applyM = [&](double* x, double* y) {  // y = A x or S~_l x
        return vel ? launch_operator(c, OP_A, F(x), F(y), 1.0, 0.0, nullptr, 1)
                   : apply_Stilde(c, q, sl, F(x), F(y), 1, prec);
    };
    auto applyPinv = [&](double* x, double* y) {
        if (vel) return apply_PV(c, q, k, F(x), F(y), 1, prec);
        if (c->opts.schur_variant == HP_SCHUR_PCQ2) return apply_PQ2(c, q, k, F(x), F(y), 1, prec);
        return apply_PQ1(c, q, k, F(x), F(y), 1, prec);
    };
    auto dot = [&](const double* x, const double* y, double& out) {
        return vec_dots(c, n, n, x, y, 1, &out) == hipSuccess ? HP_OK : HP_EHIP;
    };
    auto project = [&](double* x) -> hp_status {  // x -= nul (nul' x) (Schur block)
        if (vel) return HP_OK;
        double d = 0.0;
        if (dot(nul, x, d) != HP_OK) return HP_EHIP;
        HIPCHK(vec_axpbypcz(c->stream, n, 1, -d, nul, n, 1.0, x, n, 0.0, nullptr, 0, x, n));
        return HP_OK;
    };
    if (vel) {
        HIPCHK(hipMemcpyAsync(r, start, sizeof(double) * n, hipMemcpyDeviceToDevice, c->stream));
    } else {
        std::vector<double> h = pressure_null(c);
        HIPCHK(hipMemcpyAsync(nul, h.data(), sizeof(double) * n, hipMemcpyHostToDevice, c->stream));
        HIPCHK(hipStreamSynchronize(c->stream));
        HIPCHK(hipMemcpyAsync(z, start, sizeof(double) * n, hipMemcpyDeviceToDevice, c->stream));
        HIPCHK(applyM(z, r));
        hp_status st = project(r);
        if (st != HP_OK) return st;
    }
    HIPCHK(vec_zero(c->stream, n, pvp));
    HIPCHK(applyPinv(r, z));
    double b2 = 0.0;
    if (dot(r, z, b2) != HP_OK) return HP_EHIP;
    if (!std::isfinite(b2)) return HP_ENAN;
    if (b2 < 0.0) return HP_ENOTSPD;
    if (b2 == 0.0) return HP_EINVAL;  // start vector in the null space
    double b = std::sqrt(b2), amax = 0.0;
    for (int j = 0; j < steps; ++j) {
        HIPCHK(vec_axpbypcz(c->stream, n, 1, 1.0 / b, z, n, 0.0, nullptr, 0, 0.0, nullptr, 0, v, n));
        HIPCHK(vec_axpbypcz(c->stream, n, 1, 1.0 / b, r, n, 0.0, nullptr, 0, 0.0, nullptr, 0, pv, n));
        HIPCHK(applyM(v, r));  // r = M v_j
        double a = 0.0;
        if (dot(v, r, a) != HP_OK) return HP_EHIP;
        // r = M v_j - alpha_j P v_j - beta_j P v_{j-1}
        HIPCHK(vec_axpbypcz(c->stream, n, 1, 1.0, r, n, -a, pv, n, -b, pvp, n, r, n));
        hp_status st = project(r);
        if (st != HP_OK) return st;
        HIPCHK(applyPinv(r, z));
        double bn2 = 0.0;
        if (dot(r, z, bn2) != HP_OK) return HP_EHIP;
        if (!std::isfinite(a) || !std::isfinite(bn2)) return HP_ENAN;
        al.push_back(a);
        amax = std::max(amax, std::fabs(a));
        if (bn2 < -1e-12 * amax * amax) return HP_ENOTSPD;
        const double bn = std::sqrt(std::max(bn2, 0.0));
        be.push_back(bn);
        if (bn <= 1e-10 * amax) break;  // invariant subspace
        std::swap(pv, pvp);
        b = bn;
    }
    return HP_OK;
}

// The setup gate (hp_opts.spectrum_gate): `steps` Lanczos steps on each block
// of P_0 -- sigma(P_{V,0}^{-1} A) and sigma(P_{Q,0}^{-1} B' P_{V,0}^{-1} B) --
// from a fixed start vector; HP_ENOTSPD when an estimate leaves (0, 2), the
// interval in which the hyper-power sequence converges and keeps P_k
// positive definite (Sec. 2, Lemma Sk_posdef, Remark rmk:convergence_Pk).
hp_status spectrum_gate(hp_ctx* c, int steps) {
    for (int block = HP_SPEC_VELOCITY; block <= HP_SPEC_SCHUR; ++block) {
        const long long n = block == HP_SPEC_VELOCITY ? c->nV : c->nQ;
        std::vector<double> h((size_t)n);
        for (long long i = 0; i < n; ++i) h[(size_t)i] = std::sin(0.754877666 * (double)(i + 1)) + 0.1;
        DevBuf start;
        if (alloc_device(&start.p, (size_t)n) != HP_OK) return HP_ENOMEM;
        HIPCHK(hipMemcpyAsync(start.p, h.data(), sizeof(double) * n, hipMemcpyHostToDevice,
                              c->stream));
        HIPCHK(hipStreamSynchronize(c->stream));
        std::vector<double> al, be;
        const hp_status st =
            spectrum(c, block, 2, 0, 0, (int)std::min<long long>(steps, n), start.p, al, be);
        if (st != HP_OK) return st;
        std::vector<double> off(be.begin(), be.begin() + (al.size() - 1));
        const double lmin = tridiag_eig(al, off, 1), lmax = tridiag_eig(al, off, (int)al.size());
        if (!(lmin > 0.0) || !(lmax < 2.0)) return HP_ENOTSPD;
    }
    return HP_OK;
}

// ---- the solve without device allocation (hp_solve_noalloc) ----------------------------
// The Krylov vectors of hp_solve_noalloc live in this file-scope device array
// instead of memory the library allocates: each GPU the library runs on holds
// its own copy until the process ends.  In host code `noalloc_scratch` only
// names a host-side stand-in; the device address of each GPU's copy is taken
// once per device with hipGetSymbolAddress (at the first hp_setup on it) and
// used everywhere instead.
constexpr size_t NOALLOC_DOUBLES = (size_t)1 << 22;  // 32 MiB
static __device__ __align__(256) double noalloc_scratch[NOALLOC_DOUBLES];

constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex noalloc_mu;
double* noalloc_ptr[NOALLOC_MAX_DEVICES] = {};

// With `device` current: find its copy of the array (once per device).
hp_status noalloc_init(int device) {
    if (device < 0 || device >= NOALLOC_MAX_DEVICES) return HP_OK;  // the variant then refuses
    std::lock_guard<std::mutex> lock(noalloc_mu);
    if (noalloc_ptr[device]) return HP_OK;
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch)) != hipSuccess || !p) return HP_EHIP;
    noalloc_ptr[device] = static_cast<double*>(p);
    return HP_OK;
}

// Krylov doubles the solve of this context needs (vector slots are laid out
// for max_rhs right-hand sides).
size_t krylov_doubles(const hp_ctx* c) {
    const size_t V = (size_t)c->N * (size_t)c->opts.max_rhs;
    if (c->opts.krylov == HP_MINRES) return 10 * V;
    const int m = std::max(1, std::min(c->opts.restart, FG_MMAX));
    return (size_t)(2 * m + 2) * V;
}

}  // namespace

// =====================================================================================
extern "C" {

void hp_default_opts(hp_opts* o) {
    if (!o) return;
    o->c_pen = 0.0;
    o->schur_variant = HP_SCHUR_PCQ1;
    o->l_schedule = HP_L_LITERAL;
    o->precision = HP_PREC_FP64;
    o->krylov = HP_MINRES;
    o->restart = 50;
    o->maxit = 1000;
    o->order = 2;
    o->iters = 1;
    o->max_rhs = 1;
    o->poll_lag = 1;
    o->use_graph = 0;
    o->autotune = 1;
    o->op_kchunk = 0;
    o->op_order = -1;
    o->fd_plan = -1;
    o->op_slabs = 0;
    o->schur_level = 0;
    o->op_fused = -1;
    o->op_staged = -1;
    o->forward = 0;
    o->schur_pcg_iters = 20;
    o->schur_pcg_tol = 1e-2;
    o->use_x0 = 0;
    o->spectrum_gate = 0;
    o->p0_scale = 1.0;
    o->breakdown_tol = 0.0;
    o->op_dma = -1;
    o->op_pres_wide = -1;
}

const char* hp_status_string(hp_status s) {
    switch (s) {
        case HP_OK: return "ok";
        case HP_EINVAL: return "invalid argument";
        case HP_EHIP: return "HIP runtime error";
        case HP_ENOMEM: return "out of device memory";
        case HP_ENOTSPD: return "preconditioner not positive definite";
        case HP_EBREAKDOWN: return "Krylov breakdown";
        case HP_ENOCONV: return "not converged within maxit";
        case HP_ENAN: return "NaN or Inf encountered";
    }
    return "unknown status";
}

hp_status hp_setup(int elements, int degree, double nu, const hp_opts* opts, void* stream,
                   hp_ctx** out) {
    if (!out) return HP_EINVAL;
    *out = nullptr;
    if (elements < 1 || degree < 2 || degree > 8 || !(nu > 0.0)) return HP_EINVAL;
    hp_opts o;
    hp_default_opts(&o);
    if (opts) o = *opts;
    if (o.max_rhs < 1 || o.order < 2 || o.iters < 0 || o.iters > KMAX || !(o.c_pen >= 0.0) ||
        o.precision < 0 || o.precision > 2 || (o.krylov != HP_MINRES && o.krylov != HP_FGMRES) ||
        o.restart < 1 || o.maxit < 1 || o.op_kchunk < 0 || o.op_order < -1 || o.op_order > 1 ||
        o.fd_plan < -1 || o.fd_plan > FD_PLAN_LAST || o.op_slabs < 0 || o.schur_level < 0 ||
        o.schur_level > KMAX || o.schur_variant < HP_SCHUR_PCQ1 || o.schur_variant > HP_SCHUR_PCG ||
        o.schur_pcg_iters < 1 || o.schur_pcg_iters > 1000 || !(o.schur_pcg_tol >= 0.0) ||
        o.op_fused < -1 || o.op_fused > 1 || o.op_staged < -1 || o.op_staged > 1 ||
        o.op_dma < -1 || o.op_dma > 1 || o.op_pres_wide < -1 || o.op_pres_wide > 1 ||
        o.use_graph < 0 || o.use_graph > 1 || o.poll_lag < 1 || o.poll_lag > 3 ||
        o.forward < 0 || o.forward > 1 || o.use_x0 < 0 || o.use_x0 > 1 || o.spectrum_gate < 0 ||
        !(o.p0_scale >= 0.0) || !std::isfinite(o.p0_scale) || !(o.breakdown_tol >= 0.0))
        return HP_EINVAL;
    if (o.p0_scale == 0.0) o.p0_scale = 1.0;
    const int nM = elements + degree - 1;
    if (nM > 4096) return HP_EINVAL;
    if (ops_init_attributes() != hipSuccess || fd_init_attributes() != hipSuccess) return HP_EHIP;
    CtxExtra* ce = new (std::nothrow) CtxExtra();
    if (!ce) return HP_ENOMEM;
    hp_ctx* c = &ce->ctx;
    // the default penalty grows with the degree like the inverse-inequality
    // constant it must dominate (12.5 up to degree 4)
    if (o.c_pen == 0.0) o.c_pen = std::max(12.5, 2.5 * (degree + 1));
    c->opts = o;
    c->stream = reinterpret_cast<hipStream_t>(stream);
    if (hipGetDevice(&c->device) != hipSuccess) { delete ce; return HP_EHIP; }
    if (noalloc_init(c->device) != HP_OK) { delete ce; return HP_EHIP; }
    c->E = elements;
    c->p = degree;
    c->nu = nu;
    try {
        c->tab = build_tables(elements, degree, o.c_pen);
    } catch (...) {
        delete ce;
        return HP_EINVAL;
    }
    // A is SPD only if the Nitsche-augmented T^ is (Sec. 3.1: the penalty
    // alpha = c_pen / h must dominate the inverse inequality, whose constant
    // grows with the degree); refuse a penalty too small for this mesh
    if (*std::min_element(c->tab.lamT.begin(), c->tab.lamT.end()) <= 0.0 ||
        *std::min_element(c->tab.lamK.begin(), c->tab.lamK.end()) <= 0.0) {
        delete ce;
        return HP_ENOTSPD;
    }
    const int nN = c->tab.nN;
    c->nN = nN;
    c->nM = nM;
    long long d[4][3] = {{nN, nM, nM}, {nM, nN, nM}, {nM, nM, nN}, {nM, nM, nM}};
    std::memcpy(c->dims, d, sizeof(d));
    c->off[0] = 0;
    for (int b = 0; b < 4; ++b) c->off[b + 1] = c->off[b] + d[b][0] * d[b][1] * d[b][2];
    c->nV = c->off[3];
    c->nQ = c->off[4] - c->off[3];
    c->N = c->off[4];
    // ---- tables
    const int p = degree, wN = p, wM = p - 1;
    const int nt = fd_half_tiles(nM);
    const size_t nfrag = (size_t)2 * 256 * nt * nt;  // one fragment table
    size_t nb = (size_t)3 * nN * (2 * wN + 1) + (size_t)2 * nM * (2 * wM + 1);
    // (+32: the dense tables start on a 256-byte boundary, for vector loads)
    size_t nfd = 5 * nfrag + nN + nM + 32;
    if (alloc_device(&c->d_tables, nb + nfd) != HP_OK) { delete ce; return HP_ENOMEM; }
    double* tp = c->d_tables;
    c->band.ptr[BK_N] = tp; upload_band(c->tab.K_int, nN, wN, tp); tp += (size_t)nN * (2 * wN + 1);
    c->band.ptr[BM_N] = tp; upload_band(c->tab.M_int, nN, wN, tp); tp += (size_t)nN * (2 * wN + 1);
    c->band.ptr[BM_C] = tp; upload_band(c->tab.Mc, nM, wM, tp); tp += (size_t)nM * (2 * wM + 1);
    c->band.ptr[BT_C] = tp; upload_band(c->tab.Tc, nM, wM, tp); tp += (size_t)nM * (2 * wM + 1);
    {
        // D^^T M^: row i = M^ row i - M^ row i+1 (D^^T w at i is w_i - w_{i+1}),
        // columns i-p+1 .. i+p, stored with half-width p
        const int W = 2 * wN + 1;
        std::vector<double> dm((size_t)nN * W, 0.0);
        auto mc = [&](int rr, int cc) {
            return (rr >= 0 && rr < nM && cc >= 0 && cc < nM) ? c->tab.Mc[(size_t)rr * nM + cc] : 0.0;
        };
        for (int i = 0; i < nN; ++i)
            for (int t = 0; t < W; ++t) {
                const int col = i - wN + t;
                dm[(size_t)i * W + t] = mc(i, col) - mc(i + 1, col);
            }
        (void)hipMemcpy(tp, dm.data(), dm.size() * sizeof(double), hipMemcpyHostToDevice);
        c->band.ptr[BD_M] = tp;
        tp += (size_t)nN * W;
    }
    c->band.n[BK_N] = c->band.n[BM_N] = c->band.n[BD_M] = nN;
    c->band.n[BM_C] = c->band.n[BT_C] = nM;
    c->band.w[BK_N] = c->band.w[BM_N] = c->band.w[BD_M] = wN;
    c->band.w[BM_C] = c->band.w[BT_C] = wM;
    auto up64 = [&](const std::vector<double>& v) {
        (void)hipMemcpy(tp, v.data(), v.size() * sizeof(double), hipMemcpyHostToDevice);
        const double* r = tp;
        tp += v.size();
        return r;
    };
    // fast diagonalisation: the half-size matrices as MFMA fragments, in FP64
    // and FP32, and the eigenvalues
    c->fd_ok = true;
    {
        tp += (32 - (size_t)(tp - c->d_tables) % 32) % 32;  // 256-byte alignment of the fragments
        if (hipMalloc(reinterpret_cast<void**>(&c->d_tables32), 5 * nfrag * sizeof(float)) !=
            hipSuccess) {
            hp_destroy(c);
            return HP_ENOMEM;
        }
        float* fp = c->d_tables32;
        auto up = [&](const std::vector<double>& A, int n, FdPack kind, const double** p64,
                      const float** p32) {
            std::vector<double> v64;
            std::vector<float> v32;
            fd_pack(A, n, nt, kind, v64);
            fd_pack(A, n, nt, kind, v32);
            (void)hipMemcpy(tp, v64.data(), v64.size() * sizeof(double), hipMemcpyHostToDevice);
            (void)hipMemcpy(fp, v32.data(), v32.size() * sizeof(float), hipMemcpyHostToDevice);
            *p64 = tp;
            *p32 = fp;
            tp += v64.size();
            fp += v32.size();
        };
        up(c->tab.UK, nN, FdPack::forward, &c->fd64.F[0], &c->fd32.F[0]);
        up(c->tab.UK, nN, FdPack::inverse, &c->fd64.V[0], &c->fd32.V[0]);
        up(c->tab.UT, nM, FdPack::forward, &c->fd64.F[1], &c->fd32.F[1]);
        up(c->tab.UT, nM, FdPack::inverse, &c->fd64.V[1], &c->fd32.V[1]);
        up(c->tab.Mcinv, nM, FdPack::symmetric, &c->fd64.Mi, &c->fd32.Mi);
        c->fd64.lam[0] = up64(c->tab.lamK);
        c->fd64.lam[1] = up64(c->tab.lamT);
        for (int i = 0; i < 2; ++i) c->fd32.lam[i] = c->fd64.lam[i];
        c->fd64.nN = c->fd32.nN = nN;
        c->fd64.nM = c->fd32.nM = nM;
        c->fd64.nt = c->fd32.nt = nt;
    }
    // ---- workspace: operator intermediates + FD temporaries
    const long long R = o.max_rhs;
    c->ws_doubles = (size_t)(ops_ws_stride(c) + 2 * c->N) * R;
    if (alloc_device(&c->ws, c->ws_doubles) != HP_OK) { hp_destroy(c); return HP_ENOMEM; }
    Extra* ex = &ce->ex;
    if (alloc_device(&ex->hv, (size_t)4 * c->nV * R) != HP_OK) { hp_destroy(c); return HP_ENOMEM; }
    if (c->fd_ok) {
        if (alloc_device(&ex->ws2, c->ws_doubles) != HP_OK ||
            hipStreamCreateWithFlags(&ex->side, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&ex->fork_ev, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ex->join_ev, hipEventDisableTiming) != hipSuccess) {
            hp_destroy(c);
            return HP_ENOMEM;
        }
    }
    if (alloc_device(&ex->hq, (size_t)3 * c->nQ * R * (KMAX + 1)) != HP_OK) { hp_destroy(c); return HP_ENOMEM; }
    if (o.schur_variant == HP_SCHUR_PCG &&
        (alloc_device(&ex->cgv, (size_t)4 * c->nV * R) != HP_OK ||
         alloc_device(&ex->cgcoef, (size_t)6 * R) != HP_OK ||
         alloc_device(&ex->cgpart, vec_partial_doubles(1, (int)R)) != HP_OK ||
         hipMalloc(reinterpret_cast<void**>(&ex->cgsc), sizeof(CgScalars) * R) != hipSuccess)) {
        hp_destroy(c);
        return HP_ENOMEM;
    }
    ex->coef_doubles = (size_t)std::max(4, 132) * R;
    if (alloc_device(&ex->dcoef, ex->coef_doubles) != HP_OK) { hp_destroy(c); return HP_ENOMEM; }
    if (hipHostMalloc(reinterpret_cast<void**>(&ex->hcoef), ex->coef_doubles * sizeof(double)) != hipSuccess) {
        hp_destroy(c);
        return HP_ENOMEM;
    }
    if (hipMalloc(reinterpret_cast<void**>(&ex->msc), 2 * sizeof(MinresScalars) * R) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void**>(&ex->hmsc[0]), sizeof(MinresScalars) * R,
                      hipHostMallocMapped) != hipSuccess ||
        hipHostMalloc(reinterpret_cast<void**>(&ex->hmsc[1]), sizeof(MinresScalars) * R,
                      hipHostMallocMapped) != hipSuccess ||
        hipHostGetDevicePointer(reinterpret_cast<void**>(&ex->dmsc[0]), ex->hmsc[0], 0) != hipSuccess ||
        hipHostGetDevicePointer(reinterpret_cast<void**>(&ex->dmsc[1]), ex->hmsc[1], 0) != hipSuccess ||
        alloc_device(&ex->mpart, 2 * vec_partial_doubles(1, (int)R)) != HP_OK ||
        alloc_device(&ex->mfg, (size_t)fd_dot_capacity(c, true) * R) != HP_OK ||
        alloc_device(&ex->mfq, (size_t)fd_dot_capacity(c, false) * R) != HP_OK ||
        hipMemset(ex->mfg, 0, sizeof(double) * fd_dot_capacity(c, true) * R) != hipSuccess ||
        hipMemset(ex->mfq, 0, sizeof(double) * fd_dot_capacity(c, false) * R) != hipSuccess ||
        hipEventCreateWithFlags(&ex->mev[0], hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ex->mev[1], hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ex->mev[2], hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ex->mev[3], hipEventDisableTiming) != hipSuccess ||
        hipStreamCreateWithFlags(&ex->cap, hipStreamNonBlocking) != hipSuccess) {
        hp_destroy(c);
        return HP_ENOMEM;
    }
    {
        const size_t M1 = FG_MMAX + 1;
        if (hipMalloc(reinterpret_cast<void**>(&ex->fsc), sizeof(FgScalars) * R) != hipSuccess ||
            hipHostMalloc(reinterpret_cast<void**>(&ex->hfsc[0]), sizeof(FgScalars) * R,
                          hipHostMallocMapped) != hipSuccess ||
            hipHostMalloc(reinterpret_cast<void**>(&ex->hfsc[1]), sizeof(FgScalars) * R,
                          hipHostMallocMapped) != hipSuccess ||
            hipHostGetDevicePointer(reinterpret_cast<void**>(&ex->dfsc[0]), ex->hfsc[0], 0) != hipSuccess ||
            hipHostGetDevicePointer(reinterpret_cast<void**>(&ex->dfsc[1]), ex->hfsc[1], 0) != hipSuccess ||
            alloc_device(&ex->fH, M1 * FG_MMAX * R) != HP_OK ||
            alloc_device(&ex->fcs, FG_MMAX * R) != HP_OK || alloc_device(&ex->fsn, FG_MMAX * R) != HP_OK ||
            alloc_device(&ex->fg, M1 * R) != HP_OK || alloc_device(&ex->fy, FG_MMAX * R) != HP_OK ||
            alloc_device(&ex->fhc, M1 * R) != HP_OK || alloc_device(&ex->fvs, R) != HP_OK ||
            alloc_device(&ex->fpart, vec_partial_doubles((int)M1, (int)R)) != HP_OK) {
            hp_destroy(c);
            return HP_ENOMEM;
        }
    }
    c->red_slots = (int)(vec_partial_doubles(130, (int)R) + 130 * R);
    if (alloc_device(&c->d_red, c->red_slots) != HP_OK) { hp_destroy(c); return HP_ENOMEM; }
    if (hipHostMalloc(reinterpret_cast<void**>(&c->h_red), 130 * R * sizeof(double)) != hipSuccess) {
        hp_destroy(c);
        return HP_ENOMEM;
    }
    if (c->opts.forward == 1) {
        const hipError_t qe = quad_setup(c, &ex->quad);
        if (qe != hipSuccess) {
            hp_destroy(c);
            return qe == hipErrorOutOfMemory ? HP_ENOMEM : HP_EHIP;
        }
    }
    if (hipDeviceSynchronize() != hipSuccess) { hp_destroy(c); return HP_EHIP; }
    if (c->opts.autotune) {
        const hp_status ts = autotune(c);
        if (ts != HP_OK) {
            hp_destroy(c);
            return ts;
        }
    }
    if (c->opts.spectrum_gate > 0 && c->fd_ok) {
        const hp_status gs = spectrum_gate(c, c->opts.spectrum_gate);
        if (gs != HP_OK) {
            hp_destroy(c);
            return gs;
        }
    }
    *out = c;
    return HP_OK;
}

hp_status hp_get_tuning(const hp_ctx* c, int nrhs, hp_tuning* out) {
    if (!c || !out || nrhs < 1 || nrhs > c->opts.max_rhs) return HP_EINVAL;
    const OpShape sh = op_shape(c, nrhs);
    out->op_kchunk = std::max(1, std::min(sh.kchunk, c->nM));
    out->op_order = sh.comp_fast;
    out->op_slabs = std::max(1, std::min(sh.slabs, c->nM));
    out->op_staged = sh.staged && !sh.fused && op_staged_ok(c->p, out->op_kchunk) ? 1 : 0;
    out->op_pres_wide = sh.pwide && !sh.fused && !out->op_staged ? 1 : 0;
    out->op_tuned = 0;
    out->op_us = 0.0;
    for (int e = 0; e < 2; ++e)
        if (c->op_tuned[e].kchunk > 0 && c->op_tuned[e].nrhs == nrhs) {
            out->op_tuned = 1;
            out->op_us = c->op_tuned_us[e];
        }
    for (int prec = 0; prec < 3; ++prec) {
        out->fd_plan[prec] = fd_plan_in_use(c, prec);
        out->fd_us[prec] = c->fd_tuned_us[prec];
    }
    return HP_OK;
}

hp_status hp_set_nu(hp_ctx* c, double nu) {
    if (!c || !(nu > 0.0)) return HP_EINVAL;
    c->nu = nu;
    return HP_OK;
}

hp_status hp_sizes(const hp_ctx* c, int64_t dims[4][3], int64_t offsets[5]) {
    if (!c) return HP_EINVAL;
    for (int b = 0; b < 4; ++b)
        for (int d = 0; d < 3; ++d)
            if (dims) dims[b][d] = c->dims[b][d];
    for (int b = 0; b < 5; ++b)
        if (offsets) offsets[b] = c->off[b];
    return HP_OK;
}

hp_status hp_apply_K(hp_ctx* c, const double* x, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !x || !y || x == y) return HP_EINVAL;
    HIPCHK(launch_operator(c, OP_K, full_fields(c, x), full_fields(c, y), 1.0, 0.0, nullptr, nrhs));
    return HP_OK;
}

hp_status hp_apply_K_quad(hp_ctx* c, const double* x, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !x || !y || x == y) return HP_EINVAL;
    QuadOp* q = &extra_of(c)->quad;
    const hipError_t e = quad_setup(c, q);
    if (e == hipErrorOutOfMemory) return HP_ENOMEM;
    HIPCHK(e);
    HIPCHK(launch_quad_K(c, q, full_fields(c, x), full_fields(c, y), nrhs));
    return HP_OK;
}

hp_status hp_apply_A(hp_ctx* c, const double* u, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !u || !y || u == y) return HP_EINVAL;
    HIPCHK(launch_operator(c, OP_A, vel_fields(c, u, c->nV), vel_fields(c, y, c->nV), 1.0, 0.0,
                           nullptr, nrhs));
    return HP_OK;
}

hp_status hp_apply_B(hp_ctx* c, const double* p, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !p || !y || (const void*)p == (const void*)y) return HP_EINVAL;
    HIPCHK(launch_operator(c, OP_B, pres_fields(c, p, c->nQ), vel_fields(c, y, c->nV), 1.0, 0.0,
                           nullptr, nrhs));
    return HP_OK;
}

hp_status hp_apply_Bt(hp_ctx* c, const double* u, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !u || !y || (const void*)u == (const void*)y) return HP_EINVAL;
    HIPCHK(launch_operator(c, OP_BT, vel_fields(c, u, c->nV), pres_fields(c, y, c->nQ), 1.0, 0.0,
                           nullptr, nrhs));
    return HP_OK;
}

hp_status hp_apply_MV(hp_ctx* c, const double* u, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !u || !y || u == y) return HP_EINVAL;
    HIPCHK(launch_operator(c, OP_MV, vel_fields(c, u, c->nV), vel_fields(c, y, c->nV), 1.0, 0.0,
                           nullptr, nrhs));
    return HP_OK;
}

hp_status hp_apply_P0(hp_ctx* c, const double* x, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !x || !y || x == y || !c->fd_ok) return HP_EINVAL;
    HIPCHK(launch_P0(c, full_fields(c, x), full_fields(c, y), true, true, false, c->opts.precision,
                     nrhs));
    return HP_OK;
}

hp_status hp_apply_hyperpower(hp_ctx* c, int order, int iters, const double* x, double* y,
                              int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !x || !y || x == y || order < 2 || iters < 0 ||
        iters > KMAX || !c->fd_ok)
        return HP_EINVAL;
    HIPCHK(apply_Pk(c, order, iters, x, y, nrhs));
    return HP_OK;
}

hp_status hp_apply_PV(hp_ctx* c, int order, int iters, const double* u, double* y, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !u || !y || order < 2 || iters < 0 || iters > KMAX ||
        !c->fd_ok || (u < y + c->nV * (long long)nrhs && y < u + c->nV * (long long)nrhs))
        return HP_EINVAL;
    HIPCHK(apply_PV(c, order, iters, vel_fields(c, u, c->nV), vel_fields(c, y, c->nV), nrhs,
                    c->opts.precision));
    return HP_OK;
}

hp_status hp_spectrum(hp_ctx* c, int block, int order, int iters, int s_level, int steps,
                      const double* start, double* alpha, double* beta, int* done,
                      double* lmin, double* lmax) {
    if (!c || !start || !done || !lmin || !lmax || !c->fd_ok || order < 2 || iters < 0 ||
        iters > KMAX || s_level < 0 || s_level > KMAX ||
        (block != HP_SPEC_VELOCITY && block != HP_SPEC_SCHUR) || steps < 1 ||
        steps > (block == HP_SPEC_VELOCITY ? c->nV : c->nQ))
        return HP_EINVAL;
    std::vector<double> al, be;
    al.reserve(steps);
    be.reserve(steps);
    hp_status st = spectrum(c, block, order, iters, s_level, steps, start, al, be);
    if (st != HP_OK) return st;
    const int m = (int)al.size();
    *done = m;
    for (int j = 0; j < m; ++j) {
        if (alpha) alpha[j] = al[j];
        if (beta) beta[j] = be[j];
    }
    std::vector<double> off(be.begin(), be.begin() + (m - 1));
    *lmin = tridiag_eig(al, off, 1);
    *lmax = tridiag_eig(al, off, m);
    return HP_OK;
}

}  // extern "C"

namespace {

hp_status solve_checks(hp_ctx* c, const double* b, double* x, int nrhs, double tol) {
    if (check_rhs(c, nrhs) != HP_OK || !b || !x || b == x || !(tol > 0.0) || !c->fd_ok)
        return HP_EINVAL;
    if (c->opts.krylov == HP_MINRES &&
        (c->opts.precision != HP_PREC_FP64 || c->opts.schur_variant == HP_SCHUR_PCG))
        return HP_EINVAL;  // MINRES needs a fixed symmetric preconditioner
    return HP_OK;
}

// The solve and its true residual; the Krylov vectors are whatever ex->kv
// holds (allocated on first use unless the caller has put them in place).
hp_status solve_impl(hp_ctx* c, const double* b, double* x, int nrhs, double tol,
                     hp_solve_info* info, double* rr_host, double* bb_host) {
    auto t0 = std::chrono::steady_clock::now();
    hp_solve_info loc{};
    hp_status s = c->opts.krylov == HP_MINRES ? minres(c, b, x, nrhs, tol, &loc)
                                              : fgmres(c, b, x, nrhs, tol, &loc);
    if (s == HP_EHIP || s == HP_ENOMEM) return s;
    // true residual ||b - K x|| / ||b||
    double* w = c->ws + ops_ws_stride(c) * (long long)c->opts.max_rhs;  // FD scratch, N * nrhs
    if (launch_operator(c, OP_K, full_fields(c, x), full_fields(c, w), 1.0, 0.0, nullptr, nrhs) !=
            hipSuccess ||
        vec_axpby(c->stream, c->N * nrhs, 1.0, b, -1.0, w) != hipSuccess)
        return HP_EHIP;
    if (vec_dots(c, c->N, c->N, w, w, nrhs, rr_host) != hipSuccess ||
        vec_dots(c, c->N, c->N, b, b, nrhs, bb_host) != hipSuccess)
        return HP_EHIP;
    loc.true_relres = 0.0;
    for (int r = 0; r < nrhs; ++r)
        loc.true_relres =
            std::max(loc.true_relres, bb_host[r] > 0 ? std::sqrt(rr_host[r] / bb_host[r]) : 0.0);
    loc.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (info) *info = loc;
    return s;
}

}  // namespace

extern "C" {

hp_status hp_solve(hp_ctx* c, const double* b, double* x, int nrhs, double tol,
                   hp_solve_info* info) {
    const hp_status chk = solve_checks(c, b, x, nrhs, tol);
    if (chk != HP_OK) return chk;
    std::vector<double> rr(nrhs), bb(nrhs);
    return solve_impl(c, b, x, nrhs, tol, info, rr.data(), bb.data());
}

hp_status hp_solve_noalloc(hp_ctx* c, const double* b, double* x, int nrhs, double tol,
                           hp_solve_info* info) {
    const hp_status chk = solve_checks(c, b, x, nrhs, tol);
    if (chk != HP_OK) return chk;
    if (nrhs > 64) return HP_EINVAL;
    if (c->device < 0 || c->device >= NOALLOC_MAX_DEVICES || !noalloc_ptr[c->device])
        return HP_EHIP;
    // the quadrature forward operator allocates its tables on first use
    if (c->opts.forward == 1 && !extra_of(c)->quad.ready) return HP_EINVAL;
    if (krylov_doubles(c) > NOALLOC_DOUBLES) return HP_ENOMEM;
    Extra* ex = extra_of(c);
    double* kv0 = ex->kv;
    const size_t kd0 = ex->kv_doubles;
    const int graph0 = c->opts.use_graph;
    ex->kv = noalloc_ptr[c->device];
    ex->kv_doubles = NOALLOC_DOUBLES;
    c->opts.use_graph = 0;  // capturing and instantiating graphs allocates
    double rr[64], bb[64];
    const hp_status st = solve_impl(c, b, x, nrhs, tol, info, rr, bb);
    ex->kv = kv0;
    ex->kv_doubles = kd0;
    c->opts.use_graph = graph0;
    return st;
}

hp_status hp_build_rhs(hp_ctx* c, const double* lid, int nmodes, const double* amp,
                       const int* waves, const double* beta, double* b, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !b || nmodes < 0 || (nmodes > 0 && (!amp || !waves)))
        return HP_EINVAL;
    // beta (n_V per rhs) must not overlap b (N per rhs)
    if (beta && beta < b + c->N * (long long)nrhs && b < beta + c->nV * (long long)nrhs)
        return HP_EINVAL;
    return build_rhs(c, lid, nmodes, amp, waves, beta, b, nrhs);
}

hp_status hp_grad(hp_ctx* c, const double* x, const double* lambda, const double* lid,
                  double* dL_dbeta, double* dL_dnu, int nrhs) {
    if (check_rhs(c, nrhs) != HP_OK || !x || !lambda || !dL_dbeta || !dL_dnu) return HP_EINVAL;
    // dL/dbeta = M_V lambda_u
    HIPCHK(launch_operator(c, OP_MV, vel_of_full(c, lambda), vel_fields(c, dL_dbeta, c->nV), 1.0,
                           0.0, nullptr, nrhs));
    // dL/dnu = lambda_u . (F_lid - A u) / nu ; F_lid into t (full), A u into its velocity part
    double* t = c->ws + ops_ws_stride(c) * (long long)c->opts.max_rhs;  // N * nrhs scratch
    hp_status s = build_rhs(c, lid, 0, nullptr, nullptr, nullptr, t, nrhs);
    if (s != HP_OK) return s;
    const Fields tv = vel_of_full(c, t);
    HIPCHK(launch_operator(c, OP_A, vel_of_full(c, x), tv, -1.0, 1.0, &tv, nrhs));
    std::vector<double> d(nrhs);
    for (int r = 0; r < nrhs; ++r) {
        double out = 0.0;
        if (vec_dots(c, c->nV, c->N, lambda + r * c->N, t + r * c->N, 1, &out) != hipSuccess)
            return HP_EHIP;
        dL_dnu[r] = out / c->nu;
    }
    return HP_OK;
}

void hp_destroy(hp_ctx* c) {
    if (!c) return;
    CtxExtra* ce = reinterpret_cast<CtxExtra*>(c);
    Extra* ex = &ce->ex;
    (void)hipDeviceSynchronize();
    if (c->d_tables) (void)hipFree(c->d_tables);
    if (c->d_tables32) (void)hipFree(c->d_tables32);
    if (c->ws) (void)hipFree(c->ws);
    if (c->d_red) (void)hipFree(c->d_red);
    if (c->h_red) (void)hipHostFree(c->h_red);
    if (ex->hv) (void)hipFree(ex->hv);
    if (ex->ws2) (void)hipFree(ex->ws2);
    if (ex->side) (void)hipStreamDestroy(ex->side);
    quad_free(&ex->quad);
    if (ex->fork_ev) (void)hipEventDestroy(ex->fork_ev);
    if (ex->join_ev) (void)hipEventDestroy(ex->join_ev);
    if (ex->hq) (void)hipFree(ex->hq);
    if (ex->kv) (void)hipFree(ex->kv);
    if (ex->dcoef) (void)hipFree(ex->dcoef);
    drop_graphs(ex);
    drop_fg_graphs(ex);
    for (double* p : {ex->fH, ex->fcs, ex->fsn, ex->fg, ex->fy, ex->fhc, ex->fvs, ex->fpart})
        if (p) (void)hipFree(p);
    if (ex->fsc) (void)hipFree(ex->fsc);
    if (ex->hfsc[0]) (void)hipHostFree(ex->hfsc[0]);
    if (ex->hfsc[1]) (void)hipHostFree(ex->hfsc[1]);
    if (ex->msc) (void)hipFree(ex->msc);
    if (ex->hmsc[0]) (void)hipHostFree(ex->hmsc[0]);
    if (ex->hmsc[1]) (void)hipHostFree(ex->hmsc[1]);
    if (ex->mpart) (void)hipFree(ex->mpart);
    if (ex->mfg) (void)hipFree(ex->mfg);
    if (ex->mfq) (void)hipFree(ex->mfq);
    if (ex->cgv) (void)hipFree(ex->cgv);
    if (ex->cgcoef) (void)hipFree(ex->cgcoef);
    if (ex->cgpart) (void)hipFree(ex->cgpart);
    if (ex->cgsc) (void)hipFree(ex->cgsc);
    for (hipEvent_t ev : ex->mev)
        if (ev) (void)hipEventDestroy(ev);
    if (ex->cap) (void)hipStreamDestroy(ex->cap);
    if (ex->hcoef) (void)hipHostFree(ex->hcoef);
    delete ce;
}

}  // extern "C"
