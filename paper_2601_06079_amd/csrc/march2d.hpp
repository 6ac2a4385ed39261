// march2d.hpp -- the row-streamed 2-D stencils: the pieces of k_march2d.hip (one
// operator per pass) and k_cheb2d.hip (several steps of an iteration per pass).
#pragma once
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "kernels.hpp"
#include "march.hpp"
#include "stream2d.hpp"

namespace pfk {

template <typename T>
struct MC2 {
    T a, b, c;  // GRAD: q (a + q (b + c q)); JVP, SCHUR: (a + q (b + c q)) v  (|J| folded in)
    T kv;       // times (9 v - box v), nodal: (4 v - nbrs)
    T kl;       // what the rounding of kv leaves (add_stiffness)
    T kw;       // SCHUR: the outer stencil
    T s0, s1, s2;
    T g1, g2, g3;  // ME_ADJ: f' at W = 1
};

// 9 v - box3x3 v of row r - 1 (nodal: 4 v - axis neighbours) as rows are pushed, from
// differences of neighbouring values (which FP32 forms exactly where the field is smooth:
// with 9 v - box v the rounding floor of the residual was 6 times higher at 2048^2, and
// Newton took one more correction): with e = 2 v - v(x-1) - v(x+1),
//   3 (2 v - v(y-1) - v(y+1)) + e(y-1) + e + e(y+1)
template <typename T, bool NODAL>
struct Lap2 {
    T v1 = 0, d1 = 0, e1 = 0, e2 = 0;  // v at row r-1; v(r-1) - v(r-2); e of rows r-1, r-2
    __device__ __forceinline__ T push(T v)
    {
        const T e = (v - from_left(v)) + (v - from_right(v));
        const T d = v - v1;
        T lap;
        if constexpr (NODAL)
            lap = e1 + (d1 - d);
        else
            lap = fmaT((T)3, d1 - d, (e2 + e1) + e);
        e2 = e1;
        e1 = e;
        d1 = d;
        v1 = v;
        return lap;
    }
};

// quadrature sum of node row r - 1 as rows of u (and v) are pushed
// (SUM: asum receives sum_q f1'(u_q) v_q of the element row (r-1, r) above it)
template <typename T, bool WITHV, bool NODAL, bool SUM = false>
struct Quad2 {
    T xlu = 0, xru = 0, xlv = 0, xrv = 0;  // x-interpolants of row r-1 (nodal: u, v of row r-1 in xlu, xlv)
    T guL = 0, guR = 0;                    // upward scatter of element row (r-2, r-1)

    T asum = 0;

    __device__ __forceinline__ T push(T u, T v, const MC2<T>& k)
    {
        const T gp = (T)GP, gm = (T)GM;
        if constexpr (SUM) asum = 0;
        auto F = [&](T q, T p) {
            if constexpr (SUM) asum = fmaT(cubic(q, k.g1, k.g2, k.g3), p, asum);
            return fmaT(fmaT(k.c, q, k.b), q, k.a) * (WITHV ? p : q);
        };
        if constexpr (NODAL) {
            const T r = F(xlu, xlv);
            xlu = u;
            xlv = v;
            return r;
        } else {
            const T du = from_right(u) - u;
            const T xlu0 = fmaT(gm, du, u), xru0 = fmaT(gp, du, u);
            const T eu0 = xlu0 - xlu, eu1 = xru0 - xru;
            T xlv0 = 0, xrv0 = 0, ev0 = 0, ev1 = 0;
            if constexpr (WITHV) {
                const T dv = from_right(v) - v;
                xlv0 = fmaT(gm, dv, v);
                xrv0 = fmaT(gp, dv, v);
                ev0 = xlv0 - xlv;
                ev1 = xrv0 - xrv;
            }
            const T PL0 = F(fmaT(gm, eu0, xlu), fmaT(gm, ev0, xlv));
            const T PL1 = F(fmaT(gp, eu0, xlu), fmaT(gp, ev0, xlv));
            const T PR0 = F(fmaT(gm, eu1, xru), fmaT(gm, ev1, xrv));
            const T PR1 = F(fmaT(gp, eu1, xru), fmaT(gp, ev1, xrv));
            const T dL = PL0 - PL1, dR = PR0 - PR1;
            const T HL = guL + fmaT(gp, dL, PL1), HR = guR + fmaT(gp, dR, PR1);
            guL = fmaT(gm, dL, PL1);
            guR = fmaT(gm, dR, PR1);
            const T dH = HL - HR;
            xlu = xlu0;
            xru = xru0;
            xlv = xlv0;
            xrv = xrv0;
            return fmaT(gp, dH, HR) + from_left(fmaT(gm, dH, HR));
        }
    }
};

constexpr int MPF = 4;  // rows in flight per field

// the kernels' coefficients of an operator (epilogue coefficients s0 .. s2 apart)
template <typename T>
MC2<T> march2_coef(const Geom& g, int op, const FreeEnergy& f, double nq, double kv, double kw)
{
    const double mm = g.h * g.h, w = nq * (g.quad ? mm : 0.25 * mm), ks = g.quad ? 1.0 : 1.0 / 3.0;
    MC2<T> k{};
    if (op == MOP_GRAD) {
        k.a = (T)(w * f.a1); k.b = (T)(w * f.a2); k.c = (T)(w * f.a3);
    } else {
        k.a = (T)(w * f.b0); k.b = (T)(w * f.b1); k.c = (T)(w * f.b2);
    }
    k.kv = (T)(kv * ks);
    k.kl = (T)(kv * ks - (double)k.kv);
    k.kw = (T)(kw * ks);
    return k;
}

}  // namespace pfk
