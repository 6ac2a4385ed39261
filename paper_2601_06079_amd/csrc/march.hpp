// march.hpp -- what the marching stencil kernels (2-D row streams, 3-D plane
// streams) share: the operator applied at a node and what is done with it there.
//
// With N(u)_a = sum_e sum_q |J| f'(u_q) phi_a(q), N'(u) v its linearisation and K the
// Q1 stiffness, a kernel forms one of
//   MOP_GRAD:  o = [N(u) + kappa K u]     (scaled by the coefficients)
//   MOP_JVP:   o = [N'(u) v + kappa K v]
//   MOP_STIFF: o = K v
//   MOP_SCHUR: o = K [N'(u) v + kappa K v]   (2-D)
// and, with c the value of the operator's argument at the node (or base[idx] when that
// pointer is given), ib = 1 / 2^b on the rows of a node on b no-flux faces (rows = 1):
//   ME_OUT:   out = (o + s0 (c - p1)) ib               p1 may be null (0)
//   ME_SUB:   out = c - o ib
//   ME_MU:    out = (s0 p0 - o) ib
//   ME_BACK:  out = s0 p0 / ib + o
//   ME_CHRES: (GRAD with v, 2-D) the Cahn-Hilliard residual rows: out2 = (s0 v - o) ib,
//             out = (kw K v + s1 (c - p1)) ib    p1 may be null (0)
//   ME_CHEB:  out = c + s1 (c - p2) + s2 p1 (p0 - (o + s0 c) ib)   p2 may be null (0)
//   ME_ADJ:   (JVP) out = c - o ib + p1                 p1 may be null (0)
//   ME_ADJK:  (STIFF) out = o
// The last two belong to the adjoint of the explicit step: the operator acts on 2^b v, and
// each wave also leaves FP64 sums over its nodes and elements in part (added to what is
// there unless fresh): ME_ADJ part[2 w] = sum_e sum_q f1'(u_q) v_q (f1 the free energy at
// W = 1, real elements only), part[2 w + 1] = sum u ib K v; ME_ADJK part[w] = sum p0 ib K v
// (K v without kv, times 3 in 2-D and 12 / h in 3-D).  scale: v carries the factor 2^b.
// ME_CHEB is one step of the Chebyshev semi-iteration for the operator (o + s0 c) ib
// with right-hand side p0 and diagonal preconditioner p1; out may be p2's buffer (each
// lane reads its own node of p2 before it writes it).
#pragma once
#include <hip/hip_runtime.h>

namespace pfk {

enum { MOP_GRAD = 0, MOP_JVP = 1, MOP_STIFF = 2, MOP_SCHUR = 3 };
enum { ME_OUT = 0, ME_SUB = 1, ME_MU = 2, ME_BACK = 3, ME_CHEB = 4, ME_CHRES = 5, ME_ADJ = 6,
       ME_ADJK = 7 };

// Coefficients are doubles here (rounded once to the field type by the launcher).
// f: cubic (GRAD) or quadratic (JVP, SCHUR) of the local energy without |J|; nq
// multiplies the quadrature sum's |J| (2-D (h/2)^2 and so on are applied by the
// launcher), kv multiplies K v; kw multiplies
// the outer K of SCHUR and the K v of ME_CHRES.
template <typename T>
struct March {
    const T* u = nullptr;     // GRAD, JVP, SCHUR: the state
    const T* v = nullptr;     // JVP, STIFF, SCHUR: the direction
    T *out = nullptr, *out2 = nullptr;
    const T* base = nullptr;  // c from memory instead of the operator's argument
    const T *p0 = nullptr, *p1 = nullptr, *p2 = nullptr;
    double nq = 1.0, kv = 0.0, kw = 0.0;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    double* part = nullptr;   // ME_ADJ, ME_ADJK: the waves' sums, at most part_max doubles (null:
                              // nothing is launched, only the number of waves reported)
    long long part_max = 0;
    int fresh = 0;
    int scale = 0;            // ME_ADJ, ME_ADJK: v is multiplied by 2^b as it is read
    int rows = 0;             // divide the rows of boundary nodes by 2^b (no-flux)
};

// s + kv K v (lap: K v without its coefficient).  The coefficient folds kappa, dt and the
// like into one number, whose rounding (up to 6e-8 in FP32) would act on every step of a run
// alike; what it leaves is applied too, one operation a node.
template <typename T, typename Coefs>
__device__ __forceinline__ T add_stiffness(const Coefs& k, T lap, T s)
{
    if constexpr (sizeof(T) == 4)
        return __builtin_fmaf(k.kv, lap, __builtin_fmaf(k.kl, lap, s));
    else
        return __builtin_fma(k.kv, lap, s);
}

}  // namespace pfk
