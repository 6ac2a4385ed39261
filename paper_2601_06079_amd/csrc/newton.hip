// newton.hip -- backward-Euler step by Newton-Raphson with matrix-free GMRES
// (Eqs. 13-14, Sec. 2.3), and the adjoint solve of that step (Supp. Note 2).
//
// Host loop, device data.  All vectors (residual, correction, the Krylov basis,
// the preconditioner) live in the caller's workspace on the device; every
// matrix-vector product is the matrix-free Jacobian kernel; every dot product
// and norm is an FP64 device reduction.  Per Arnoldi step the host reads back
// one Hessenberg column (<= 2 m + 3 doubles) to apply its Givens rotation and
// test convergence; the (m+1) x m Hessenberg matrix and the small triangular
// solve stay on the host in FP64.  The read is pipelined: the next Arnoldi step
// is queued before the host waits for the current column, so the device never
// idles on the round trip; a step queued past convergence is discarded.
//
// GMRES(m) variant: right preconditioning (it monitors an estimate of the true
// residual), classical Gram-Schmidt with one re-orthogonalisation, x0 = 0, restart
// from the true residual b - J x.  Inexact Newton: the linear tolerance is
// clamp(0.1 ||R_k|| / ||R_0||, lin_rtol_min, lin_rtol_max) relative to ||R_k||.
#include <cmath>
#include <array>
#include <cstring>

#include "api_internal.hpp"
#include "kernels.hpp"
#include "krylov.hpp"

namespace pfapi {
namespace {

constexpr int MAXM = 32;  // largest restart length

inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Workspace layout shared by the forward Newton step and the adjoint solve.
template <typename T>
struct NWS {
    T *R, *x, *w, *z, *b, *V, *pinv;
    long long ld;
    double *part, *dev;  // dev: [h1(MAXM+1) | h2(MAXM+1) | nrm(2) | y(MAXM) | misc(8)]
    long long part_len;  // doubles in part
    double* theta;       // device copy of a host theta_bar (pf_vjp with PF_VJP_THETA_HOST), or a
                         // trajectory's sums (node kernels)
    size_t bytes;
};

template <typename T>
NWS<T> layout(const pf_problem* p, void* base)
{
    const pfk::Geom g = geom_of(p);
    const long long n = ndof(p);
    NWS<T> L{};
    // basis columns 256-byte aligned and 1280 bytes off a power-of-two stride, so that
    // the k streams of a Gram-Schmidt sweep do not start on the same HBM channel
    L.ld = (n + 63) / 64 * 64 + 1280 / (long long)sizeof(T);
    char* c = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t b) {
        char* r = c ? c + off : nullptr;
        off += align256(b);
        return r;
    };
    L.R = (T*)take(n * sizeof(T));
    L.x = (T*)take(n * sizeof(T));
    L.w = (T*)take(n * sizeof(T));
    L.z = (T*)take(n * sizeof(T));
    L.b = (T*)take(n * sizeof(T));
    L.V = (T*)take((size_t)(MAXM + 1) * L.ld * sizeof(T));
    L.pinv = (T*)take((size_t)(p->model == PF_COUPLED ? 9 : p->model == PF_CAHN_HILLIARD ? 4
                               : p->model == PF_GRAIN ? p->nfields : 1) * g.N * sizeof(T));
    const long long nbp = std::max<long long>(pfk::krylov_blocks(n), (g.N + 255) / 256);
    L.part = (double*)take((size_t)(MAXM + 2) * nbp * sizeof(double) + 64);
    L.part_len = (long long)(MAXM + 2) * nbp;
    L.dev = (double*)take(4 * (MAXM + 8) * sizeof(double));
    L.theta = (double*)take(4 * sizeof(double));
    L.bytes = off;
    return L;
}

enum { DEV_H1 = 0, DEV_H2 = MAXM + 1, DEV_NRM = 2 * (MAXM + 1), DEV_Y = 2 * (MAXM + 1) + 2,
       DEV_MISC = 3 * (MAXM + 1) + 2 };

// Pinned host slots for the Hessenberg columns (two, used alternately) and the
// scalars the kernels store directly, with the events that mark each slot's step.
// The memory belongs to the context (made by pf_create); this is a view of it.
// Layout (doubles): [slot 0: DEV_Y | slot 1: DEV_Y | y: MAXM | scalars: 8].
struct ColReadback {
    double* host = nullptr;      // host address of the slots
    double* host_dev = nullptr;  // the same memory as the device addresses it
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};  // slot 0, slot 1, scalars
    double* y() const { return host + 2 * DEV_Y; }
    double* scal() const { return host + 2 * DEV_Y + MAXM; }
    double* scal_dev() const { return host_dev + 2 * DEV_Y + MAXM; }
    // wait for the scalars written by kernels queued so far on s
    int wait_scalars(hipStream_t s) const
    {
        if (hipEventRecord(ev[2], s) != hipSuccess || hipEventSynchronize(ev[2]) != hipSuccess)
            return check_launch("scalar readback");
        return PF_OK;
    }
};
constexpr size_t RB_DOUBLES = 2 * DEV_Y + MAXM + 8;
constexpr int SCAL_SPEC = 6;  // of the scalars: launch_spectrum's two (before them the norms and the CG's)

ColReadback col_readback(const pf_ctx* ctx)
{
    static_assert(MAXM <= pfk::KR_MAXK, "restart length beyond the Gram-Schmidt kernels");
    ColReadback r;
    r.host = ctx->gmres.host;
    r.host_dev = ctx->gmres.dev;
    for (int i = 0; i < 3; ++i) r.ev[i] = ctx->gmres.ev[i];
    return r;
}

struct Opts {
    double rtol, atol, lmin, lmax;
    int max_newton, m, max_its, precond, stagnation, krylov;
};

Opts resolve(const pf_newton_opts* o)
{
    pf_newton_opts d;
    pf_newton_default_opts(&d);
    if (!o) o = &d;
    Opts r{};
    r.rtol = o->rtol;
    r.atol = o->atol;
    r.lmin = o->lin_rtol_min;
    r.lmax = o->lin_rtol_max;
    r.max_newton = o->max_newton;
    r.m = o->gmres_restart;
    r.max_its = o->gmres_max_its;
    r.precond = o->precond;
    r.stagnation = o->stagnation;
    r.krylov = o->krylov;
    return r;
}

int check_opts(const Opts& o)
{
    if (!(o.rtol >= 0.0) || !(o.atol >= 0.0) || !std::isfinite(o.rtol) || !std::isfinite(o.atol))
        return fail(PF_EINVAL, "rtol/atol must be finite and >= 0");
    if (o.max_newton < 0 || o.max_newton > 1000) return fail(PF_EINVAL, "max_newton out of range");
    if (o.m < 1 || o.m > MAXM) return fail(PF_EINVAL, "gmres_restart must be in 1..%d", MAXM);
    if (o.max_its < 1) return fail(PF_EINVAL, "gmres_max_its must be >= 1");
    if (o.precond != PF_PRECOND_NONE && o.precond != PF_PRECOND_JACOBI)
        return fail(PF_EINVAL, "unknown preconditioner");
    if (!(o.lmin > 0.0) || !(o.lmax >= o.lmin) || !(o.lmax < 1.0))
        return fail(PF_EINVAL, "need 0 < lin_rtol_min <= lin_rtol_max < 1");
    if (o.krylov != PF_KRYLOV_GMRES && o.krylov != PF_KRYLOV_CG) return fail(PF_EINVAL, "unknown krylov solver");
    return PF_OK;
}

// CG needs a symmetric positive definite Jacobian.  Allen-Cahn's is
// (m/dt) M + L (N'(eta) + kappa K) with N'(eta) >= -W M_c (f'' >= -W for both
// double wells) and M_c <= the lumped mass, so dt L W < 1 makes it positive
// definite for every eta; the other models are not symmetric (or not definite).
int check_cg(const pf_problem* p, double dt, const Opts& o)
{
    if (o.krylov != PF_KRYLOV_CG) return PF_OK;
    if (p->model != PF_ALLEN_CAHN) return fail(PF_EINVAL, "krylov = CG needs the Allen-Cahn model");
    // positive definiteness below rests on L > 0, kappa >= 0 (K is positive
    // semi-definite) and W >= 0 (f'' >= -W for both double wells)
    if (!(p->mobility > 0.0)) return fail(PF_EINVAL, "krylov = CG needs mobility > 0 (got %g)", p->mobility);
    if (!(p->kappa >= 0.0)) return fail(PF_EINVAL, "krylov = CG needs kappa >= 0 (got %g)", p->kappa);
    if (!(p->W >= 0.0)) return fail(PF_EINVAL, "krylov = CG needs W >= 0 (got %g)", p->W);
    if (!(dt * p->mobility * p->W < 1.0))
        return fail(PF_EINVAL, "krylov = CG needs dt L W < 1 (got %g): the Jacobian may be indefinite",
                    dt * p->mobility * p->W);
    return PF_OK;
}

int d2h(void* dst, const void* src, size_t bytes, hipStream_t s)
{
    if (hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return check_launch("device-to-host read");
    return PF_OK;
}

// The elimination needs a diagonal mass, the point preconditioner (its absence is a
// request for the bare system) and the marching kernels (fields below 2 GiB).
template <typename T>
bool schur_ok(const pf_problem* p, const pfk::Geom& g, const Opts& o)
{
    return p->model == PF_CAHN_HILLIARD && !g.cm && o.precond == PF_PRECOND_JACOBI &&
           (size_t)g.N * sizeof(T) < (size_t(1) << 31);
}

// Allen-Cahn's polynomial needs the same, and GMRES (a CG iteration is already as cheap as
// a product in the polynomial).
template <typename T>
bool poly_ok(const pf_problem* p, const pfk::Geom& g, const Opts& o)
{
    return p->model == PF_ALLEN_CAHN && !g.cm && o.precond == PF_PRECOND_JACOBI && o.krylov == PF_KRYLOV_GMRES &&
           (size_t)g.N * sizeof(T) < (size_t(1) << 31);
}

// Chebyshev polynomial of D^-1 J over [theta - delta, theta + delta] as a preconditioner:
// deg - 1 further products with J per application.
struct Cheb {
    int deg = 1;
    double theta = 1.0, delta = 0.0;
    double rate = 0.0;  // log of the residual reduction an Arnoldi step should give
};

// The linear operator handed to GMRES: J = dR/dU at U (or its transpose), or, for
// Cahn-Hilliard with the lumped mass, the same system with mu eliminated.  Its mu row is
// linear and diagonal in x_mu,
//   ib (inv_dt m x_c + M K x_mu) = b_c,   ib (m x_mu - A x_c) = b_mu,   A = N'(c) + kappa K
// (ib = 1 / 2^b on no-flux rows), so
//   S x_c = ib (inv_dt m x_c + (M / m) K A x_c) = b_c - ib (M / m) K (2^b b_mu),
//   x_mu = (2^b b_mu + A x_c) / m.
// Vectors of N instead of 2N entries, and about half the iterations: block Jacobi couples
// the two planes only through their diagonals.  The residual of S is that of the whole
// system (its mu row is solved exactly), so the stop tests keep their meaning.
// Transposed: S^T l_c = b_c + ib A (2^b b_mu) / m, l_mu = (2^b b_mu - M K l_c) / m.
template <typename T>
struct LinOp {
    const pf_problem* p;
    pfk::Geom g;
    pfk::FreeEnergy f;
    double inv_dt;
    const T* U;
    int trans;
    bool schur = false;
    T* tmp = nullptr;  // N values between the two stencils of S
    Cheb cheb{};       // polynomial preconditioner (deg 1: the diagonal alone)
    const T* pinv = nullptr;
    T* zb = nullptr;   // n values: the second iterate of the polynomial
    double mass() const { return std::pow(g.h, g.dim); }
    void apply(const T* v, T* out, hipStream_t s) const
    {
        if (p->model == PF_COUPLED)
            pfk::launch_cp_jvp<T>(g, p->kappa, p->mobility, p->mobility_eta, inv_dt, U, v, out, s);
        else if (p->model == PF_GRAIN)
            pfk::launch_gg_jvp2d<T>(g, p->nfields, p->mobility, p->kappa, p->gamma, inv_dt, U, v, out, s);
        else if (schur)
            schur_pass(pfk::ME_OUT, v, out, s);
        else
            pfk::launch_jvp<T>(g, p->model, f, p->kappa, p->mobility, inv_dt, U, v, out, s, trans, 0);
    }
    // z = p(J) pinv v by the Chebyshev semi-iteration from z0 = pinv v (which carries
    // 1 / theta); returns the buffer (z0 or zb) that holds the result
    T* poly(const T* v, T* z0, hipStream_t s) const
    {
        T *z = z0, *zp = zb;
        double rho = cheb.delta / cheb.theta;
        for (int k = 1; k < cheb.deg; ++k) {
            const double rn = 1.0 / (2.0 * cheb.theta / cheb.delta - rho);
            pfk::March<T> e;
            e.p0 = v;
            e.p1 = pinv;
            e.p2 = k > 1 ? zp : nullptr;
            e.s1 = rho * rn;
            e.s2 = 2.0 * rn * cheb.theta / cheb.delta;
            if (schur) {
                schur_pass(pfk::ME_CHEB, z, zp, s, e);
            } else {
                e.u = U;
                e.v = z;
                e.out = zp;
                e.nq = p->mobility;
                e.kv = p->mobility * p->kappa;
                e.s0 = inv_dt * mass();
                e.rows = 1;
                pfk::launch_march<T>(g, pfk::MOP_JVP, pfk::ME_CHEB, f, e, s);
            }
            std::swap(z, zp);
            rho = rn;
        }
        return z;
    }
    // The same with several steps a pass (2-D): w = J z if w is given, else z, in the buffer
    // returned; null where it does not apply (nothing is launched then).  Between passes the
    // two iterates stand in z0 and zb or in c and d (needed from the third pass on, and from
    // the second if w is null); the steps are spread evenly over as few passes as hold them.
    bool fuses() const { return g.dim == 2 && !(schur && trans) && g.n[1] > pfk::CHEB_MAXS; }
    // passes of poly_fused with or without the product (0: it does not apply)
    int fused_passes(bool product, bool scratch) const
    {
        if (!fuses() || cheb.deg < 2) return 0;
        const int n = cheb.deg - 1 + (product ? 1 : 0), top = schur ? pfk::CHEB_MAXS / 2 : pfk::CHEB_MAXS;
        const int passes = (n + top - 1) / top;
        return passes > (product ? 2 : 1) && !scratch ? 0 : passes;
    }
    T* poly_fused(const T* v, T* z0, T* w, T* c, T* d, hipStream_t s) const
    {
        const int passes = fused_passes(w != nullptr, c && d), n = cheb.deg - 1 + (w ? 1 : 0);
        if (passes == 0) return nullptr;
        T *in[2] = {nullptr, nullptr}, *nx[2] = {z0, zb};
        double rho = cheb.delta / cheb.theta;
        for (int i = 0, k = 0; i < passes; ++i) {
            const bool last = i == passes - 1;
            const int S = n / passes + (i < n % passes ? 1 : 0);
            pfk::ChebGroup<T> q;
            q.z = in[0];
            q.zm = in[1];
            q.product = last && w;
            for (int j = 0; j < S && ++k < cheb.deg; ++j) {
                const double rn = 1.0 / (2.0 * cheb.theta / cheb.delta - rho);
                q.s1[j] = rho * rn;
                q.s2[j] = 2.0 * rn * cheb.theta / cheb.delta;
                rho = rn;
            }
            pfk::March<T> e;
            e.u = U;
            e.p0 = v;
            e.p1 = pinv;
            e.out = last && w ? w : nx[0];
            q.out2 = last ? nullptr : nx[1];
            e.s0 = inv_dt * mass();
            e.nq = schur ? 1.0 / mass() : p->mobility;
            e.kv = schur ? p->kappa / mass() : p->mobility * p->kappa;
            e.kw = p->mobility;
            if (!pfk::launch_cheb2d<T>(g, schur ? pfk::MOP_SCHUR : pfk::MOP_JVP, f, e, q, S, s)) return nullptr;
            if (last) return e.out;
            in[0] = nx[0];
            in[1] = nx[1];
            nx[0] = in[0] == z0 ? c : z0;
            nx[1] = in[0] == z0 ? d : zb;
        }
        return nullptr;
    }
    // out = S v (epi ME_OUT), or a step of the Chebyshev iteration (ME_CHEB, e: its inputs)
    void schur_pass(int epi, const T* v, T* out, hipStream_t s, pfk::March<T> b = {}) const
    {
        const double m = mass();
        pfk::March<T> a;
        b.out = out;
        b.s0 = inv_dt * m;
        b.rows = 1;
        if (!trans && g.dim == 2) {
            b.u = U;
            b.v = v;
            b.nq = 1.0 / m;
            b.kv = p->kappa / m;
            b.kw = p->mobility;
            if (pfk::launch_march<T>(g, pfk::MOP_SCHUR, epi, f, b, s)) return;
        }
        b.base = v;
        b.v = tmp;
        a.v = v;
        a.out = tmp;
        if (!trans) {
            a.u = U;
            a.nq = 1.0 / m;
            a.kv = p->kappa / m;
            b.kv = p->mobility;
            pfk::launch_march<T>(g, pfk::MOP_JVP, pfk::ME_OUT, f, a, s);
            pfk::launch_march<T>(g, pfk::MOP_STIFF, epi, f, b, s);
        } else {
            a.kv = p->mobility / m;
            b.u = U;
            b.nq = 1.0;
            b.kv = p->kappa;
            pfk::launch_march<T>(g, pfk::MOP_STIFF, pfk::ME_OUT, f, a, s);
            pfk::launch_march<T>(g, pfk::MOP_JVP, epi, f, b, s);
        }
    }
    // out = the right-hand side of S for (b_c, b_mu) = b
    void schur_rhs(const T* b, T* out, hipStream_t s) const
    {
        const double m = mass();
        const T* bm = b + g.N;
        if (g.bc) {
            pfk::launch_unrow<T>(g, 1.0, bm, tmp, s);
            bm = tmp;
        }
        pfk::March<T> a;
        a.v = bm;
        a.base = b;
        a.out = out;
        a.rows = 1;
        if (!trans) {
            a.kv = p->mobility / m;
        } else {
            a.u = U;
            a.nq = -1.0 / m;
            a.kv = -p->kappa / m;
        }
        pfk::launch_march<T>(g, trans ? pfk::MOP_JVP : pfk::MOP_STIFF, pfk::ME_SUB, f, a, s);
    }
    // x_mu (behind x_c in x) from x_c and b
    void schur_back(const T* b, T* x, hipStream_t s) const
    {
        const double m = mass();
        pfk::March<T> a;
        a.v = x;
        a.out = x + g.N;
        a.p0 = b + g.N;
        a.s0 = 1.0 / m;
        a.rows = 1;
        if (!trans) {
            a.u = U;
            a.nq = 1.0 / m;
            a.kv = p->kappa / m;
        } else {
            a.kv = -p->mobility / m;
        }
        pfk::launch_march<T>(g, trans ? pfk::MOP_STIFF : pfk::MOP_JVP, pfk::ME_BACK, f, a, s);
    }
    // out = J v with the per-block partial sums of v . out in part2 (at most max_blocks),
    // their count in *nb; false (nothing launched) where the operator has no such fused
    // form (then apply and a separate sum are needed)
    bool apply_pq(const T* v, T* out, double* part2, int* nb, int max_blocks, hipStream_t s) const
    {
        if (p->model != PF_ALLEN_CAHN) return false;
        return pfk::launch_jvp2d_stream<T>(g, p->model, f, p->kappa, p->mobility, inv_dt, U, v, out, s, part2, nb,
                                           max_blocks);
    }
};

// Solve J x = b (L.x overwritten, starting from 0; n unknowns) to ||b - J x|| <= tol_abs.
// The preconditioner (if any) must already be in L.pinv.  At most max_its Arnoldi steps.
// Returns PF status; *its receives the dimension of the Krylov space in J searched (Arnoldi
// steps, each counting the polynomial's degree), *res the last residual estimate.  A polynomial under
// which ten Arnoldi steps in a row give less than a quarter of the reduction its interval
// promises is dropped: its interval does not hold the spectrum, and the diagonal alone
// (a constant factor in it does not matter to GMRES) goes on from the residual reached.
// verify: the residual of a solution is formed too, and the solver goes on where it is more
// than ten times the tolerance and still falls; *res is that residual.
template <typename T>
int gmres(const ColReadback* rb, LinOp<T> A, NWS<T>& L, const T* b, long long n, int m, int max_its, bool prec,
          double bnorm, double tol_abs, int* its, double* res, hipStream_t s, bool verify = false)
{
    constexpr int JUDGE = 10;
    // grain growth and the eliminated Cahn-Hilliard system: point Jacobi over all n unknowns
    // (the Krylov kernels' point model)
    const bool point = A.p->model == PF_GRAIN || A.schur;
    const int model = point ? 0 : A.p->model;
    const long long Nn = point ? n : A.g.N;
    const T* pinv = prec ? L.pinv : nullptr;
    const int tr = A.trans;
    double* dh1 = L.dev + DEV_H1;
    double* dh2 = L.dev + DEV_H2;
    double* dnrm = L.dev + DEV_NRM;
    double* dy = L.dev + DEV_Y;
    if (hipMemsetAsync(L.x, 0, (size_t)n * sizeof(T), s) != hipSuccess) return check_launch("gmres init");
    std::array<double, (MAXM + 1) * MAXM> H{};
    std::array<double, MAXM> cs{}, sn{}, y{};
    std::array<double, MAXM + 1> gv{};
    int total = 0, products = 0;
    double beta = bnorm;
    bool first = true, claimed = false;
    int judged = 0;           // Arnoldi steps since the polynomial was last judged
    double res_then = bnorm;  // and the residual there
    *res = bnorm;
    if (bnorm <= tol_abs) {
        *its = 0;
        return PF_OK;
    }
    for (;;) {
        // v0 = r / ||r||, z = P^-1 v0 with r = b - J x (= b on the first cycle)
        if (first) {
            pfk::kr_norm2<T>(b, nullptr, n, L.part, dnrm, s);
        } else {
            A.apply(L.x, L.w, s);
            pfk::kr_rsub<T>(b, L.w, n, s);
            pfk::kr_norm2<T>(L.w, nullptr, n, L.part, dnrm, s, rb->scal_dev());
            if (int rc = rb->wait_scalars(s)) return rc;
            const double before = beta;
            beta = std::sqrt(rb->scal()[0]);
            *res = beta;
            if (!std::isfinite(beta)) return fail(PF_ENONFINITE, "GMRES residual is not finite");
            if (beta <= (claimed ? 10.0 : 1.0) * tol_abs || total >= max_its || (claimed && beta > 0.5 * before)) break;
        }
        // (a fused polynomial forms P^-1 v itself)
        auto z_of = [&](int i) { return A.fused_passes(true, i + 2 <= MAXM) ? nullptr : L.z; };
        pfk::kr_normalize_prec<T>(model, first ? b : L.w, dnrm, L.V, z_of(0), pinv, Nn, 1.0, s, tr);
        first = false;
        std::fill(gv.begin(), gv.end(), 0.0);
        gv[0] = beta;
        // Arnoldi step i: w = J z_i, orthogonalise, v_{i+1} and z_{i+1}; its
        // column goes to pinned slot i % 2
        auto enqueue = [&](int i) -> int {
            // (the basis vectors behind v_{i+1} serve as scratch until they are made)
            T *vi = L.V + (long long)i * L.ld, *sc = i + 2 <= MAXM ? vi + L.ld : nullptr;
            if (!A.poly_fused(vi, L.z, L.w, sc, sc ? sc + L.ld : nullptr, s)) A.apply(A.poly(vi, L.z, s), L.w, s);
            double* slot = rb->host_dev + (i & 1) * DEV_Y;
            const pfk::KrOut out{dh1, dh2, dnrm, slot + DEV_H1, slot + DEV_H2, slot + DEV_NRM};
            if (pfk::kr_cgs2<T>(model, L.V, L.ld, i + 1, L.w, L.V + (long long)(i + 1) * L.ld, z_of(i + 1), pinv,
                                Nn, L.part, out, s, tr))
                return fail(PF_EINVAL, "Gram-Schmidt basis of %d vectors", i + 1);
            if (hipEventRecord(rb->ev[i & 1], s) != hipSuccess) return check_launch("GMRES column readback");
            return PF_OK;
        };
        int j = 0;
        bool done = false, stuck = false;
        const int deg = A.cheb.deg;  // products with J per Arnoldi step
        const int steps = std::min(m, max_its - total);
        if (steps > 0)
            if (int rc = enqueue(0)) return rc;
        for (; j < steps; ++j) {
            if (j + 1 < steps)
                if (int rc = enqueue(j + 1)) return rc;
            if (hipEventSynchronize(rb->ev[j & 1]) != hipSuccess) return check_launch("GMRES column wait");
            const double* col = rb->host + (j & 1) * DEV_Y;
            ++total;
            products += deg;
            for (int i = 0; i <= j; ++i) H[i * MAXM + j] = col[DEV_H1 + i] + col[DEV_H2 + i];
            const double hn = std::sqrt(std::max(col[DEV_NRM], 0.0));
            H[(j + 1) * MAXM + j] = hn;
            for (int i = 0; i < j; ++i) {
                const double t = cs[i] * H[i * MAXM + j] + sn[i] * H[(i + 1) * MAXM + j];
                H[(i + 1) * MAXM + j] = -sn[i] * H[i * MAXM + j] + cs[i] * H[(i + 1) * MAXM + j];
                H[i * MAXM + j] = t;
            }
            const double a = H[j * MAXM + j], bb = H[(j + 1) * MAXM + j];
            const double rr = std::hypot(a, bb);
            if (!std::isfinite(rr)) {
                hipStreamSynchronize(s);
                return fail(PF_ENONFINITE, "GMRES Hessenberg is not finite");
            }
            if (rr == 0.0) {  // J maps this direction to nothing new: the residual stays
                *res = std::fabs(gv[j]);
                done = true;
                break;
            }
            cs[j] = a / rr;
            sn[j] = bb / rr;
            H[j * MAXM + j] = rr;
            H[(j + 1) * MAXM + j] = 0.0;
            gv[j + 1] = -sn[j] * gv[j];
            gv[j] = cs[j] * gv[j];
            *res = std::fabs(gv[j + 1]);
            if (*res <= tol_abs || hn == 0.0) {
                ++j;
                done = true;
                break;
            }
            if (deg > 1 && ++judged == JUDGE) {
                stuck = std::log(res_then / *res) < 0.25 * JUDGE * A.cheb.rate;
                judged = 0;
                res_then = *res;
                if (stuck) {
                    ++j;
                    break;
                }
            }
        }
        // y = H^-1 g (upper triangular j x j), x += P^-1 V y
        for (int i = j - 1; i >= 0; --i) {
            double sum = gv[i];
            for (int k = i + 1; k < j; ++k) sum -= H[i * MAXM + k] * y[k];
            y[i] = H[i * MAXM + i] != 0.0 ? sum / H[i * MAXM + i] : 0.0;
        }
        if (j > 0) {
            // pinned source: the copy is asynchronous; the host rewrites y only after
            // waiting on work queued behind it
            std::copy(y.begin(), y.begin() + j, rb->y());
            if (hipMemcpyAsync(dy, rb->y(), (size_t)j * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
                return check_launch("GMRES solution coefficients");
            if (A.cheb.deg > 1) {
                // w = V y, z = pinv w
                pfk::kr_combine<T>(L.V, L.ld, j, dy, pinv, L.w, A.fused_passes(false, true) ? nullptr : L.z, n, s);
                // (the basis is made anew on the next cycle: scratch)
                const T* z = A.poly_fused(L.w, L.z, nullptr, L.V, L.V + L.ld, s);
                pfk::kr_add<T>(L.x, z ? z : A.poly(L.w, L.z, s), n, s);
            } else {
                pfk::kr_update<T>(model, L.V, L.ld, j, dy, pinv, L.x, Nn, s, tr);
            }
        }
        claimed = done;
        if (done ? !verify : total >= max_its) break;
        if (stuck) A.cheb = Cheb{};
    }
    *its = products;
    return check_launch("gmres");
}

// The polynomial for a linear solve to the relative residual lin: the interval and the
// degree.
// Upper end: launch_spectrum's bound at the field (Allen-Cahn 1% added for rounding; S,
// where it is an estimate, 5%): beyond the interval the polynomial grows with the degree's
// power, and f'' has no upper limit of its own.
// Lower end: Allen-Cahn's Jacobian is symmetric and, where f'' >= f, its eigenvalues are at
// least (1/dt + L f) m; S is similar to a symmetric operator whose eigenvalues are at least
// m/dt, less M f^2 m / (4 kappa) if f < 0 (the least value of k (kappa k + f m) M / m over
// the stiffness's eigenvalues k >= 0).  f = -W holds everywhere but is far too low for a
// developed field, in which f'' is 2 W but for walls a few nodes thick, whose own modes lie
// near f = 0, and pockets too small for a mode of their own.  So f is launch_spectrum's
// estimate, less 0.1 W for what a mean hides.  An eigenvalue below the interval does no
// harm: GMRES finds it.
// Degree: the diagonal alone would take about P = sqrt(hi / lo) ln(2 / lin) / 2 products;
// a product in the polynomial costs two to three vectors less than the Gram-Schmidt
// sweeps of one more basis vector, so the basis is kept to about six vectors and the
// degree to 10; with several products a pass they cost a quarter of that: four vectors
// and 20.  A loose solve (the first correction, whose residual is mostly of short waves)
// stops at 2.
// Measured, ms per step, degree 1 against six vectors, one product a pass: 2048^2
// Allen-Cahn 19.1 / 6.1, 500 x 420 Cahn-Hilliard 15.4 / 7.2, 128^3 Cahn-Hilliard 5.8 / 4.1;
// several products a pass, six vectors against four: 2048^2 Allen-Cahn 4.4 / 3.9, 1024^2
// 1.50 / 1.40 (FP64 1.68 / 1.59), 500^2 1.05 / 0.84, 300^2 Cahn-Hilliard 2.18 / 2.12.
struct Interval {
    double lo = 0.0, hi = 0.0;
    double indefinite = HUGE_VAL;  // Cahn-Hilliard: dt M f^2 / (4 kappa), f < 0; lo > 0 below 1
};
// the interval of a field with launch_spectrum's estimate f and the given upper
// bound (0: what every field has at least)
template <typename T>
Interval interval_of(const LinOp<T>& A, double f, double bound)
{
    const pf_problem* p = A.p;
    const pfk::StencilDiag d = pfk::stencil_diag(A.g);
    const double m = A.mass(), hk = A.g.dim == 3 ? A.g.h : 1.0, mob = p->mobility, fp = std::max(f, 0.0);
    if (!(mob > 0.0) || !(p->kappa > 0.0) || !(p->W >= 0.0)) return {};
    if (p->model == PF_CAHN_HILLIARD) {
        const double fm = std::min(f, 0.0), q = mob * fm * fm / (4.0 * p->kappa * A.inv_dt);
        return {(1.0 - q) * A.inv_dt * m /
                    (A.inv_dt * m + mob * p->kappa / m * d.kk * hk * hk + mob * d.km * hk * fp),
                bound > 0.0 ? 1.05 * bound : d.kmax * d.kmax / d.kk, q};
    }
    return {(A.inv_dt + mob * f) * m / (A.inv_dt * m + mob * p->kappa * d.kd * hk + mob * m * d.mm * fp),
            bound > 0.0 ? 1.01 * bound : d.kmax / d.kd, 0.0};
}
template <typename T>
int cheb_degree(const LinOp<T>& A, const Interval& v, double lin)
{
    if (!(v.lo > 0.0) || !(v.lo < v.hi) || !std::isfinite(v.hi)) return 1;
    const double products = 0.5 * std::sqrt(v.hi / v.lo) * std::log(2.0 / lin);
    const int top = A.fuses() ? 20 : 10;
    return (int)std::lround(std::min(products / (A.fuses() ? 4.0 : 6.0), (double)top));
}
template <typename T>
Cheb choose_cheb(const LinOp<T>& A, const Interval& v, double lin)
{
    const int deg = cheb_degree<T>(A, v, lin);
    Cheb c;
    if (deg < 2) return c;
    c.deg = lin > 3e-3 ? 2 : deg;
    c.theta = 0.5 * (v.hi + v.lo);
    c.delta = 0.5 * (v.hi - v.lo);
    c.rate = std::min(0.5, 2.0 * c.deg * std::sqrt(v.lo / v.hi));
    return c;
}

// What the field says of the interval.  It is found once for a Newton step and holds while
// the field moves little: where f'' has changed by at most df, a quotient over the nodes
// grows from q to (q + r) / (1 - r) at most, with r the share of df in the least diagonal.
template <typename T>
struct FieldEnds {
    bool wanted = false, found = false;
    double bound = 0.0, f = 0.0, moved = 0.0;

    // wanted: a solve to lin may take a polynomial, or be eliminated, depending on the field
    FieldEnds(const LinOp<T>& A, bool candidate, double lin) : f(-A.p->W)
    {
        const Interval v = interval_of<T>(A, f, 0.0);
        wanted = candidate && v.hi > 0.0 && (!(v.lo > 0.0) || cheb_degree<T>(A, v, lin) > 1);  // (hi 0: no such system)
    }
    // before a wait for the scalars, and after it
    void queue(const ColReadback* rb, const LinOp<T>& A, const NWS<T>& L, hipStream_t s)
    {
        const pf_problem* p = A.p;
        wanted = pfk::launch_spectrum<T>(A.g, p->model, A.f, p->kappa, p->mobility, A.inv_dt, A.U, L.part, L.part_len,
                                         rb->scal_dev() + SCAL_SPEC, s);
    }
    void take(const ColReadback* rb, const LinOp<T>& A)
    {
        if (!wanted) return;
        bound = rb->scal()[SCAL_SPEC];
        f = std::max(-A.p->W, rb->scal()[SCAL_SPEC + 1] - 0.1 * A.p->W);
        moved = 0.0;
        found = true;
    }
    double drift(const LinOp<T>& A) const
    {
        const pf_problem* p = A.p;
        const pfk::StencilDiag d = pfk::stencil_diag(A.g);
        const double m = A.mass(), hk = A.g.dim == 3 ? A.g.h : 1.0, mob = p->mobility;
        if (p->model == PF_CAHN_HILLIARD)
            return mob * d.kmmax * hk * moved / (A.inv_dt * m + mob / m * p->kappa * d.kk * hk * hk);
        const double least = (A.inv_dt - mob * p->W * d.mm) * m + mob * p->kappa * d.kd * hk;
        return least > 0.0 ? mob * m * moved / least : HUGE_VAL;
    }
    // the interval at A.U; a new pass over the field where it has moved too far
    int interval(const ColReadback* rb, const LinOp<T>& A, const NWS<T>& L, Interval* v, hipStream_t s)
    {
        *v = interval_of<T>(A, f, HUGE_VAL);  // (without an upper end: no polynomial)
        if (!wanted) return PF_OK;
        double r = drift(A);
        if (!found || !(r <= 0.02)) {
            queue(rb, A, L, s);
            if (int rc = rb->wait_scalars(s)) return rc;
            take(rb, A);
            r = 0.0;
        }
        if (wanted) *v = interval_of<T>(A, f, (bound + r) / (1.0 - r));
        return PF_OK;
    }
};

// The system and the polynomial of a solve.  Cahn-Hilliard whose spectrum reaches far below
// zero (large steps from the unstable point) keeps both planes and their 2x2 blocks.  ms a
// step, eliminated / blocks, by dt M f^2 / (4 kappa), kappa / h^2 = 2: noise of 0.05 at 1.06
// 120 / none (256^2), 119 / none (64^3); of 0.05 about 0.3 at 1.03 36 / 103, 30 / 107; of
// 0.7 at 1.25 146 / none (256^2); of 0.05 about 0.3 at 1.38 none / 286, none / 107 (none: no
// convergence in 20 corrections).
template <typename T>
void choose_system(LinOp<T>& A, const Interval& v, bool schur, double lin, const NWS<T>& L)
{
    A.schur = schur && v.indefinite < 1.3;
    A.zb = A.schur ? L.R + A.g.N : L.R;
    A.cheb = !schur || A.schur ? choose_cheb<T>(A, v, lin) : Cheb{};
}

// The whole Cahn-Hilliard correction (or adjoint) J x = L.b through the eliminated
// system: L.x receives both planes.  L.R holds the right-hand side meanwhile (the
// caller evaluates the residual anew afterwards).
template <typename T>
int gmres_schur(const ColReadback* rb, const LinOp<T>& A, NWS<T>& L, int m, int max_its, double tol_abs, int* its,
                double* res, hipStream_t s, bool verify = false)
{
    const long long N = A.g.N;
    A.schur_rhs(L.b, L.R, s);
    pfk::kr_norm2<T>(L.R, nullptr, N, L.part, L.dev + DEV_NRM, s, rb->scal_dev());
    if (int rc = rb->wait_scalars(s)) return rc;
    const double bn = std::sqrt(rb->scal()[0]);
    if (!std::isfinite(bn)) return fail(PF_ENONFINITE, "right-hand side is not finite");
    if (int rc = gmres<T>(rb, A, L, L.R, N, m, max_its, true, bn, tol_abs, its, res, s, verify)) return rc;
    A.schur_back(L.b, L.x, s);
    return check_launch("eliminated system");
}

// Preconditioned CG on J x = b (x overwritten, starting from 0) to
// ||b - J x|| <= tol_abs, for a symmetric positive definite J (check_cg).  The
// scalars stay on the device; the host reads the pinned mirror one iteration
// behind the GPU.  Returns PF status; *its: iterations, *res: ||r||.
template <typename T>
int pcg(const ColReadback* rb, const LinOp<T>& A, NWS<T>& L, long long n, int max_its, bool prec, double bnorm,
        double tol_abs, int* its, double* res, hipStream_t s)
{
    *its = 0;
    *res = bnorm;
    const T* pinv = prec ? L.pinv : nullptr;
    T* r = L.V;
    T* pdir = L.V + L.ld;
    T* q = L.V + 2 * L.ld;
    double* part = L.part;
    double* part2 = L.part + 2 * pfk::cg_blocks(n);
    // room for part2 in the workspace's partial-sum area (MAXM + 2 rows of nbp)
    const int pq_max = (int)std::min<long long>(INT_MAX, L.part_len - 2 * pfk::cg_blocks(n));
    double* st = L.dev + DEV_MISC;
    double* hdev = rb->scal_dev();
    const double* h = rb->scal();
    pfk::cg_start<T>(L.b, pinv, r, L.z, pdir, L.x, n, part, st, hdev, tol_abs * tol_abs, max_its, s);
    if (bnorm <= tol_abs) return check_launch("CG start");
    int enq = 0, slot = 0;
    bool pending = false;
    for (;;) {
        pfk::cg_dir<T>(L.z, pdir, n, part, st, hdev, s);
        int nb2 = 0;  // the Jacobian product may leave the p . q partials itself
        if (!A.apply_pq(pdir, q, part2, &nb2, pq_max, s)) {
            A.apply(pdir, q, s);
            pfk::cg_pq<T>(pdir, q, n, part2, st, s);
            nb2 = 0;
        }
        pfk::cg_alpha<T>(L.x, r, L.z, pdir, q, pinv, n, part2, part, st, hdev, s, nb2);
        ++enq;
        if (int rc = check_launch("CG iteration")) return rc;
        if (hipEventRecord(rb->ev[slot], s) != hipSuccess) return check_launch("CG event");
        if (pending) {
            if (hipEventSynchronize(rb->ev[slot ^ 1]) != hipSuccess) return check_launch("CG wait");
            if (*(volatile const double*)&h[pfk::CG_H_DONE] != 0.0) break;
        }
        pending = true;
        slot ^= 1;
        if (enq > max_its) break;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return check_launch("CG sync");
    const double done = *(volatile const double*)&h[pfk::CG_H_DONE];
    *its = (int)*(volatile const double*)&h[pfk::CG_H_ITS];
    *res = std::sqrt(std::max((double)*(volatile const double*)&h[pfk::CG_H_RR], 0.0));
    if (done == pfk::CG_NONFINITE) return fail(PF_ENONFINITE, "CG met a non-finite value");
    if (done == pfk::CG_BREAKDOWN)
        return fail(PF_ENOCONV, "CG breakdown after %d iterations (Jacobian not positive definite)", *its);
    return PF_OK;  // converged, or the iteration limit (an inexact correction, as GMRES)
}

template <typename T>
double eps_of()
{
    return sizeof(T) == 4 ? 1.1920928955078125e-07 : 2.220446049250313e-16;
}

template <typename T>
int newton_t(const pf_ctx* ctx, const pf_problem* p, double dt, const T* Uold, T* U, const Opts& o,
             pf_newton_report* rep, void* ws, hipStream_t s)
{
    const pfk::Geom g = geom_of(p);
    const pfk::FreeEnergy f = pfk::make_free_energy(p->fe, p->W);
    const long long n = ndof(p);
    NWS<T> L = layout<T>(p, ws);
    const double inv_dt = 1.0 / dt;
    double* dnrm = L.dev + DEV_NRM;
    double* dmisc = L.dev + DEV_MISC;
    pf_newton_report R{};
    const ColReadback rbv = col_readback(ctx);
    const ColReadback* rb = &rbv;
    LinOp<T> A{p, g, f, inv_dt, U, 0};
    A.pinv = L.pinv;
    A.tmp = L.z + g.N;  // (with mu eliminated the solver's vectors fill half their space)
    const bool schur = schur_ok<T>(p, g, o), poly = schur || poly_ok<T>(p, g, o);
    FieldEnds<T> ends(A, poly, o.lmin);
    bool blocks = false;  // an unsolved eliminated correction did harm: no more of them
    const auto copy_field = [&](T* to, const T* from) -> int {
        return hipMemcpyAsync(to, from, (size_t)n * sizeof(T), hipMemcpyDeviceToDevice, s) == hipSuccess
                   ? PF_OK
                   : check_launch("Newton field copy");
    };
    // ||R(U)||, read back together with whatever scalars were queued before it
    auto residual_norm = [&](double* out) -> int {
        if (p->model == PF_COUPLED)
            pfk::launch_cp_residual<T>(g, p->kappa, p->mobility, p->mobility_eta, U, L.R, s, Uold, inv_dt);
        else if (p->model == PF_GRAIN)
            pfk::launch_gg_tile2d<T>(g, p->nfields, p->mobility, p->kappa, p->gamma, 0.0, U, L.R, 1, s, Uold,
                                     inv_dt);
        else
            pfk::launch_residual<T>(g, p->model, f, p->kappa, p->mobility, U, L.R, s, Uold, inv_dt);
        const bool first = ends.wanted && !ends.found;
        if (first) ends.queue(rb, A, L, s);
        pfk::kr_norm2<T>(L.R, nullptr, n, L.part, dnrm, s, rb->scal_dev());
        if (int rc = rb->wait_scalars(s)) return rc;
        if (first) ends.take(rb, A);
        *out = std::sqrt(rb->scal()[0]);
        return PF_OK;
    };
    double r0;
    if (int rc = residual_norm(&r0)) return rc;
    R.res_norm[0] = r0;
    R.reason = -1;
    int status = PF_OK;
    double rk = r0, rprev = r0;
    if (!std::isfinite(r0)) {
        R.reason = -2;
        status = fail(PF_ENONFINITE, "initial residual is not finite");
    }
    int k = 0;
    double dmax = 0.0, umax = 0.0;
    while (status == PF_OK) {
        if (rk <= o.rtol * r0) { R.converged = 1; R.reason = 0; break; }
        if (rk <= o.atol) { R.converged = 1; R.reason = 1; break; }
        // rounding floor: the residual stopped falling, and either the last correction
        // was within a few units in the last place of the field, or it left the
        // residual where it was (within 10%) although it was too small (at most
        // sqrt(eps) of the field) for the nonlinearity to undo a converged linear
        // solve -- the residual was rounding noise, whose correction can stay well
        // above the field's last place
        if (o.stagnation && k >= 2 && rk > 0.5 * rprev &&
            (dmax <= 8.0 * eps_of<T>() * umax ||
             (rk > 0.9 * rprev && dmax <= std::sqrt(eps_of<T>()) * umax))) {
            R.converged = 1;
            R.reason = 2;  // rounding floor of the field precision reached
            break;
        }
        if (k >= o.max_newton) break;
        const double lin = std::min(o.lmax, std::max(o.lmin, 0.1 * rk / r0));
        if (poly) {
            Interval v;  // (as it stands: blocks)
            if (!blocks)
                if (int rc = ends.interval(rb, A, L, &v, s)) return rc;
            choose_system<T>(A, v, schur, lin, L);
        }
        if (o.precond == PF_PRECOND_JACOBI) {
            if (p->model == PF_COUPLED)
                pfk::launch_cp_prec<T>(g, p->kappa, p->mobility, p->mobility_eta, inv_dt, U, L.pinv, s);
            else if (p->model == PF_GRAIN)
                pfk::launch_gg_tile2d<T>(g, p->nfields, p->mobility, p->kappa, p->gamma, 0.0, U, L.pinv, 2, s,
                                         nullptr, inv_dt);
            else if (A.schur)
                pfk::launch_prec_schur<T>(g, f, p->kappa, p->mobility, inv_dt, A.cheb.theta, U, L.pinv, s);
            else
                pfk::launch_prec<T>(g, p->model, f, p->kappa, p->mobility, inv_dt, U, L.pinv, s, A.cheb.theta);
        }
        pfk::kr_scale<T>(L.R, L.b, -1.0, n, s);  // b = -R
        int its = 0;
        double lres = 0.0;
        const bool jac = o.precond == PF_PRECOND_JACOBI;
        if (int rc = o.krylov == PF_KRYLOV_CG ? pcg<T>(rb, A, L, n, o.max_its, jac, rk, lin * rk, &its, &lres, s)
                     : A.schur ? gmres_schur<T>(rb, A, L, o.m, o.max_its, lin * rk, &its, &lres, s)
                               : gmres<T>(rb, A, L, L.b, n, o.m, o.max_its, jac, rk, lin * rk, &its, &lres, s)) {
            status = rc;
            R.reason = -2;
            break;
        }
        R.gmres_its += its;
        // An eliminated correction that its solve left above the tolerance is taken back where
        // the residual grew, and the blocks carry on: Cahn-Hilliard fields far from a root have
        // steps that only their corrections, solved or not, bring there.  256^2, 30 time units
        // after noise, kappa / h^2 = 1, dt M W^2 / (4 kappa) = 2 and 5: no convergence in 20
        // corrections without this; 19 and 8, as with blocks alone.
        const bool missed = A.schur && lres > lin * rk;
        if (missed)  // (the basis holds the field meanwhile)
            if (int rc = copy_field(L.V, U)) return rc;
        pfk::kr_add_maxabs<T>(U, L.x, n, L.part, dmisc, s, rb->scal_dev() + 1);
        double r;
        if (int rc = residual_norm(&r)) return rc;
        if (missed && !(r <= 1.1 * rk)) {  // (within 10%: may be rounding, as above)
            blocks = true;
            if (int rc = copy_field(U, L.V)) return rc;
            if (int rc = residual_norm(&rk)) return rc;
            continue;
        }
        rprev = rk;
        rk = r;
        dmax = rb->scal()[1];
        umax = rb->scal()[2];
        ends.moved += dmax * (std::fabs(f.b1) + std::fabs(f.b2) * (2.0 * umax + dmax));
        ++k;
        if (k <= 32) R.res_norm[k] = rk;
        if (!std::isfinite(rk)) {
            R.reason = -2;
            status = fail(PF_ENONFINITE, "Newton residual is not finite");
        }
    }
    R.newton_its = k;
    if (rep) *rep = R;
    if (status != PF_OK) return status;
    if (!R.converged)
        return fail(PF_ENOCONV, "Newton stopped after %d corrections at ||R|| = %.3e (||R0|| = %.3e)",
                    k, rk, r0);
    return check_launch("pf_newton_step");
}

}  // namespace

size_t newton_workspace_bytes(const pf_problem* p, int)
{
    return p->dtype == PF_F64 ? layout<double>(p, nullptr).bytes : layout<float>(p, nullptr).bytes;
}

size_t vjp_workspace_bytes(const pf_problem* p) { return newton_workspace_bytes(p, MAXM); }

template <typename T>
int vjp_simple_t(const pf_problem* p, int kind, double dt, bool be, const T* U, const T* vbar, T* Ubar,
                 double* theta_bar, void* ws, hipStream_t s)
{
    const pfk::Geom g = geom_of(p);
    const pfk::FreeEnergy f = pfk::make_free_energy(p->fe, p->W);
    NWS<T> L = layout<T>(p, ws);
    if (kind == PF_VJP_RESIDUAL) {
        // Ubar += (dr/dU)^T vbar : the transpose Jacobian product with no time term
        pfk::launch_jvp<T>(g, p->model, f, p->kappa, p->mobility, 0.0, U, vbar, Ubar, s, 1, 1);
        // backward-Euler residual R = M (U - U_old)/dt + r (Eq. 14): M is symmetric,
        // so its transposed time term adds (M/dt) vbar on the mass rows
        if (be) pfk::launch_mass_axpy<T>(g, 1.0 / dt, vbar, Ubar, s);
        pfk::launch_dtheta<T>(g, p->model, f, p->kappa, p->mobility, U, vbar, 1.0, L.part,
                              theta_bar, s);
    } else {
        pfk::launch_vjp_explicit<T>(g, p->model, f, p->kappa, p->mobility, dt, U, vbar, Ubar, L.V,
                                    L.part, L.part_len, theta_bar, s);
    }
    return check_launch("pf_vjp");
}

// Adjoint of nsteps explicit steps along stored states (see pf_vjp_explicit_trajectory)
template <typename T>
int vjp_trajectory_t(const pf_problem* p, double dt, int64_t nsteps, const T* states, T* lam, double* theta_bar,
                     int flags, void* ws, hipStream_t s)
{
    const pfk::Geom g = geom_of(p);
    const pfk::FreeEnergy f = pfk::make_free_energy(p->fe, p->W);
    NWS<T> L = layout<T>(p, ws);
    const long long nd = ndof(p);
    const bool ch = p->model == PF_CAHN_HILLIARD;
    // the sums of a trajectory stay in part (marched, one or two a wave) or theta (node kernels)
    const bool marched = pfk::adjoint_marches<T>(g, p->model, L.part_len);
    T* other = L.V;       // lam's second buffer (marched Cahn-Hilliard: in place)
    T* t = L.V + L.ld;    // Cahn-Hilliard
    T* cur = lam;
    int fresh = flags & PF_VJP_BEGIN ? 1 : 0;
    if (fresh && !marched) pfk::launch_zero<double>(L.theta, 3, s);
    if (fresh && marched && nsteps == 0) pfk::launch_zero<double>(L.part, L.part_len, s);  // (else the first step sets them)
    for (int64_t k = nsteps - 1; k >= 0; --k) {
        const T* U = states + k * nd;
        const T* mu = U + (ch ? g.N : 0);
        T* out = ch && marched ? cur : (cur == lam ? other : lam);
        if (marched) {
            pfk::launch_adjoint_step<T>(g, p->model, f, p->kappa, p->mobility, dt, U, mu, cur, out, nullptr, t, L.part,
                                        L.part_len, fresh, s);
        } else {
            pfk::launch_zero<T>(out, g.N, s);
            pfk::launch_adjoint_nodes<T>(g, p->model, f, p->kappa, p->mobility, dt, U, mu, cur, out, t, L.part, L.theta,
                                         s);
        }
        cur = out;
        fresh = 0;
    }
    if (cur != lam && hipMemcpyAsync(lam, cur, (size_t)g.N * sizeof(T), hipMemcpyDeviceToDevice, s) != hipSuccess)
        return check_launch("adjoint copy-back");
    if (flags & PF_VJP_END) {
        if (marched)
            pfk::launch_adjoint_theta<T>(g, p->model, f, p->kappa, p->mobility, dt, L.part, L.part_len, theta_bar, s);
        else
            pfk::launch_add3(L.theta, theta_bar, s);
    }
    return check_launch("pf_vjp_explicit_trajectory");
}

// Adjoint of one backward-Euler step at its root U (II.5-II.6):
// solve (dR/dU)^T lambda = vbar, then Uold_bar += (M/dt) lambda on the mass
// rows and theta_bar -= (dr/dtheta)^T lambda.  lambda is left in the
// workspace's x vector.
template <typename T>
int newton_adjoint_t(const pf_ctx* ctx, const pf_problem* p, double dt, const T* U, const T* vbar, T* Ubar,
                     double* theta_bar, const Opts& o, void* ws, hipStream_t s)
{
    const ColReadback rbv = col_readback(ctx);
    const pfk::Geom g = geom_of(p);
    const pfk::FreeEnergy f = pfk::make_free_energy(p->fe, p->W);
    const long long n = ndof(p);
    NWS<T> L = layout<T>(p, ws);
    const double inv_dt = 1.0 / dt;
    LinOp<T> At{p, g, f, inv_dt, U, 1};
    At.tmp = L.z + g.N;
    At.pinv = L.pinv;
    const bool schur = schur_ok<T>(p, g, o);
    // the adjoint solve is taken to the field-precision floor, not an inexact-Newton tolerance
    const double lin = sizeof(T) == 4 ? 1e-6 : 1e-12;
    if (schur || poly_ok<T>(p, g, o)) {
        Interval v;
        if (int rc = FieldEnds<T>(At, true, lin).interval(&rbv, At, L, &v, s)) return rc;
        choose_system<T>(At, v, schur, lin, L);
    }
    if (At.schur)
        pfk::launch_prec_schur<T>(g, f, p->kappa, p->mobility, inv_dt, At.cheb.theta, U, L.pinv, s);
    else if (o.precond == PF_PRECOND_JACOBI)
        pfk::launch_prec<T>(g, p->model, f, p->kappa, p->mobility, inv_dt, U, L.pinv, s, At.cheb.theta);
    if (hipMemcpyAsync(L.b, vbar, (size_t)n * sizeof(T), hipMemcpyDeviceToDevice, s) != hipSuccess)
        return check_launch("adjoint rhs copy");
    pfk::kr_norm2<T>(L.b, nullptr, n, L.part, L.dev + DEV_NRM, s);
    double nn;
    if (int rc = d2h(&nn, L.dev + DEV_NRM, sizeof(double), s)) return rc;
    const double bn = std::sqrt(nn);
    if (!std::isfinite(bn)) return fail(PF_ENONFINITE, "adjoint right-hand side is not finite");
    int its = 0;
    double res = 0.0;
    const double tol = lin * bn;
    const bool jac = o.precond == PF_PRECOND_JACOBI;
    // (Allen-Cahn's Jacobian is symmetric: CG solves the transposed system as well)
    if (int rc = o.krylov == PF_KRYLOV_CG ? pcg<T>(&rbv, At, L, n, o.max_its * 4, jac, bn, tol, &its, &res, s)
                 : At.schur ? gmres_schur<T>(&rbv, At, L, o.m, o.max_its * 4, tol, &its, &res, s, true)
                            : gmres<T>(&rbv, At, L, L.b, n, o.m, o.max_its * 4, jac, bn, tol, &its, &res, s, true))
        return rc;
    // a residual at the rounding floor, above the tolerance, is the best there is; one the
    // solver did not bring down is no solution
    if (!(res <= std::sqrt(lin) * bn))
        return fail(PF_ENOCONV, "adjoint solve stopped after %d products at a relative residual of %.1e", its, res / bn);
    // Ubar (mass rows) += (m/dt) lambda ; theta_bar -= (dr/dtheta)^T lambda
    pfk::launch_mass_axpy<T>(g, inv_dt, L.x, Ubar, s);
    pfk::launch_dtheta<T>(g, p->model, f, p->kappa, p->mobility, U, L.x, -1.0, L.part, theta_bar, s);
    return check_launch("newton adjoint");
}

int newton_adjoint(const pf_ctx* ctx, const pf_problem* p, double dt, const void* U, const void* vbar, void* Ubar,
                   double* theta_bar, void* ws, hipStream_t s)
{
    const Opts o = resolve(nullptr);
    if (p->dtype == PF_F32)
        return newton_adjoint_t<float>(ctx, p, dt, (const float*)U, (const float*)vbar, (float*)Ubar,
                                       theta_bar, o, ws, s);
    return newton_adjoint_t<double>(ctx, p, dt, (const double*)U, (const double*)vbar, (double*)Ubar,
                                    theta_bar, o, ws, s);
}

size_t newton_pinned_doubles() { return RB_DOUBLES; }

}  // namespace pfapi

using namespace pfapi;

extern "C" {

void pf_newton_default_opts(pf_newton_opts* o)
{
    if (!o) return;
    *o = pf_newton_opts{};
    o->rtol = 1e-8;
    o->atol = 0.0;
    o->max_newton = 20;
    o->gmres_restart = 30;
    o->gmres_max_its = 600;
    o->precond = PF_PRECOND_JACOBI;
    o->lin_rtol_max = 1e-2;
    o->lin_rtol_min = 1e-6;
    o->stagnation = 1;
}

int pf_newton_step(pf_ctx* ctx, const pf_problem* p, double dt, const void* U_old, void* U,
                   const pf_newton_opts* opts, pf_newton_report* rep, void* ws, void* stream)
{
    return guarded("pf_newton_step", [&]() -> int {
        if (int rc = check_ctx(ctx)) return rc;
        if (int rc = validate(p)) return rc;
        if (p->model == PF_GRAIN)
            if (int rc = grain_implicit_ok(p)) return rc;
        if (!(dt > 0.0) || !std::isfinite(dt)) return fail(PF_EINVAL, "dt must be finite and > 0");
        if (int rc = check_ptr(U_old, p, "U_old")) return rc;
        if (int rc = check_ptr(U, p, "U")) return rc;
        if (U == U_old) return fail(PF_EINVAL, "U and U_old must not alias");
        if (!ws || reinterpret_cast<uintptr_t>(ws) % 256) return fail(PF_EINVAL, "ws must be 256-byte aligned");
        const Opts o = resolve(opts);
        if (int rc = check_opts(o)) return rc;
        if (int rc = check_cg(p, dt, o)) return rc;
        if (int rc = require_device(ctx)) return rc;
        hipStream_t s = (hipStream_t)stream;
        if (p->dtype == PF_F32)
            return newton_t<float>(ctx, p, dt, (const float*)U_old, (float*)U, o, rep, ws, s);
        return newton_t<double>(ctx, p, dt, (const double*)U_old, (double*)U, o, rep, ws, s);
    });
}

int pf_vjp(pf_ctx* ctx, const pf_problem* p, int kind, double dt, const void* U, const void* U_old,
           const void* vbar, void* Ubar, double* theta_bar, int flags, void* ws, void* stream)
{
    return guarded("pf_vjp", [&]() -> int {
        if (int rc = check_ctx(ctx)) return rc;
        if (int rc = validate(p)) return rc;
        if (p->model == PF_COUPLED) return fail(PF_EUNSUPPORTED, "pf_vjp: coupled model not implemented");
        if (p->model == PF_GRAIN) return fail(PF_EUNSUPPORTED, "pf_vjp: grain growth not implemented");
        if (p->quad != PF_QUAD_GAUSS) return fail(PF_EUNSUPPORTED, "pf_vjp: Gauss-Lobatto quadrature not implemented");
        if (kind != PF_VJP_RESIDUAL && kind != PF_VJP_EXPLICIT_STEP && kind != PF_VJP_NEWTON_STEP)
            return fail(PF_EINVAL, "unknown vjp kind %d", kind);
        if (flags & ~PF_VJP_THETA_HOST) return fail(PF_EINVAL, "unknown flags 0x%x", flags);
        const bool be = kind == PF_VJP_RESIDUAL && U_old != nullptr;
        if ((kind != PF_VJP_RESIDUAL || be) && (!(dt > 0.0) || !std::isfinite(dt)))
            return fail(PF_EINVAL, "dt must be finite and > 0");
        if (kind == PF_VJP_EXPLICIT_STEP && p->mass != PF_MASS_LUMPED)
            return fail(PF_EUNSUPPORTED, "explicit steps need the lumped mass");
        if (int rc = check_ptr(U, p, "U")) return rc;
        if (U_old)
            if (int rc = check_ptr(U_old, p, "U_old")) return rc;
        if (int rc = check_ptr(vbar, p, "vbar")) return rc;
        if (int rc = check_ptr(Ubar, p, "Ubar")) return rc;
        if (Ubar == U || Ubar == vbar) return fail(PF_EINVAL, "Ubar must not alias U or vbar");
        if (!theta_bar || reinterpret_cast<uintptr_t>(theta_bar) % 8)
            return fail(PF_EINVAL, "theta_bar is NULL or misaligned");
        if (!ws || reinterpret_cast<uintptr_t>(ws) % 256) return fail(PF_EINVAL, "ws must be 256-byte aligned");
        if (int rc = require_device(ctx)) return rc;
        hipStream_t s = (hipStream_t)stream;
        const bool host_theta = (flags & PF_VJP_THETA_HOST) != 0;
        double* tb = theta_bar;
        if (host_theta) {  // accumulate into a device copy, then return it to the host
            tb = p->dtype == PF_F32 ? layout<float>(p, ws).theta : layout<double>(p, ws).theta;
            if (hipMemcpyAsync(tb, theta_bar, 3 * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
                return check_launch("theta_bar upload");
        }
        int rc;
        if (kind == PF_VJP_NEWTON_STEP)
            rc = newton_adjoint(ctx, p, dt, U, vbar, Ubar, tb, ws, s);
        else if (p->dtype == PF_F32)
            rc = vjp_simple_t<float>(p, kind, dt, be, (const float*)U, (const float*)vbar, (float*)Ubar, tb, ws, s);
        else
            rc = vjp_simple_t<double>(p, kind, dt, be, (const double*)U, (const double*)vbar, (double*)Ubar, tb,
                                      ws, s);
        if (rc != PF_OK || !host_theta) return rc;
        if (hipMemcpyAsync(theta_bar, tb, 3 * sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return check_launch("theta_bar download");
        return PF_OK;
    });
}

int pf_vjp_explicit_trajectory(pf_ctx* ctx, const pf_problem* p, double dt, int64_t nsteps, const void* states,
                               void* lam, double* theta_bar, int flags, void* ws, void* stream)
{
    return guarded("pf_vjp_explicit_trajectory", [&]() -> int {
        if (int rc = check_ctx(ctx)) return rc;
        if (int rc = validate(p)) return rc;
        if (int rc = explicit_trajectory_ok(p, dt, nsteps)) return rc;
        if (p->quad != PF_QUAD_GAUSS) return fail(PF_EUNSUPPORTED, "pf_vjp: Gauss-Lobatto quadrature not implemented");
        if (flags & ~(PF_VJP_BEGIN | PF_VJP_END)) return fail(PF_EINVAL, "unknown flags 0x%x", flags);
        if (int rc = check_ptr(states, p, "states")) return rc;
        if (int rc = check_ptr(lam, p, "lam")) return rc;
        if (!theta_bar || reinterpret_cast<uintptr_t>(theta_bar) % 8)
            return fail(PF_EINVAL, "theta_bar is NULL or misaligned");
        if (!ws || reinterpret_cast<uintptr_t>(ws) % 256) return fail(PF_EINVAL, "ws must be 256-byte aligned");
        if (int rc = require_device(ctx)) return rc;
        if (p->dtype == PF_F32)
            return vjp_trajectory_t<float>(p, dt, nsteps, (const float*)states, (float*)lam, theta_bar, flags, ws,
                                           (hipStream_t)stream);
        return vjp_trajectory_t<double>(p, dt, nsteps, (const double*)states, (double*)lam, theta_bar, flags, ws,
                                        (hipStream_t)stream);
    });
}

}  // extern "C"
