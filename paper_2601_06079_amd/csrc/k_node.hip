// k_node.hip -- node-centric kernels for 2-D and 3-D periodic Q1 grids:
// residual (Eq. 11) and backward-Euler residual (Eq. 14), Jacobian products,
// preconditioner, chemical potential, node-centric explicit updates, energy.
// The shared device helpers and the quadrature scheme are in node_common.hpp.
// g.quad selects Gauss-Lobatto (nodal) quadrature: N(u)_a = m f'(u_a), the 5/7-point
// stiffness stencil and the lumped mass (the branch is uniform over the grid).
#include <algorithm>
#include <cmath>

#include "node_common.hpp"

namespace pfk {

namespace {

// r(U): Allen-Cahn  r = L [N + kappa K u];  Cahn-Hilliard r_c = M K mu, r_mu = m mu - [N(c) + kappa K c]
// With Uold != nullptr the time term inv_dt m (U - Uold) of Eq. 14 is added to
// the rows that carry mass (Allen-Cahn eta, Cahn-Hilliard c).  g.cm: the
// consistent mass (3^d stencil) replaces m in the time term and the mu-row.
template <typename T, int D, int MODEL>
__global__ __launch_bounds__(256) void k_residual(const T* __restrict__ U, const T* __restrict__ Uold,
                                                  T* __restrict__ r, Geom g, Cub<T> F, T detJ,
                                                  T kappa, T mob, T m, T inv_dt)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T u[NB<D>::K];
    gather<T, D>(U, g, i, j, k, u);
    const T h = (T)g.h;
    const T Nn = g.quad ? m * F(u[NB<D>::K / 2], (T)0) : detJ * quad_sum<T, D, false>(u, u, F);
    const T Ku = stiff_q<T, D>(g, u, h);
    T tt = (T)0;
    if (Uold) {
        if (g.cm) {
            T uo[NB<D>::K];
            gather<T, D>(Uold, g, i, j, k, uo);
#pragma unroll
            for (int q = 0; q < NB<D>::K; ++q) uo[q] = u[q] - uo[q];
            tt = inv_dt * cmass<T, D>(uo, h);
        } else {
            tt = inv_dt * m * (u[NB<D>::K / 2] - Uold[idx]);
        }
    }
    const T ib = (T)1 / (T)bfactor<D>(g, i, j, k);  // no-flux rows (1 on periodic grids)
    if constexpr (MODEL == 0) {
        r[idx] = (mob * (Nn + kappa * Ku) + tt) * ib;
    } else {
        T w[NB<D>::K];
        gather<T, D>(U + g.N, g, i, j, k, w);
        r[idx] = (mob * stiff_q<T, D>(g, w, h) + tt) * ib;
        const T mw = g.cm ? cmass<T, D>(w, h) : m * w[NB<D>::K / 2];
        r[g.N + idx] = (mw - (Nn + kappa * Ku)) * ib;
    }
}

// (Block-)Jacobi preconditioner of dR/dU at U:
//   Allen-Cahn:    pinv[a] = 1 / (theta (inv_dt m + L (N'_aa + kappa K_aa)))
//   Cahn-Hilliard: pinv[4a..4a+3] = inverse of [[inv_dt m, M K_aa], [-(N'_aa + kappa K_aa), m]]
// (row-major), with N'_aa = sum_e sum_q |J| f''(u_q) phi_a(q)^2.
template <typename T, int D, int MODEL>
__global__ __launch_bounds__(256) void k_prec(const T* __restrict__ U, T* __restrict__ pinv, Geom g,
                                              Lin<T> F, T detJ, T kappa, T mob, T m, T inv_dt, double theta)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T u[NB<D>::K];
    gather<T, D>(U, g, i, j, k, u);
    const double nd = g.quad ? (double)(m * F(u[NB<D>::K / 2], (T)1)) : (double)(detJ * quad_sum_sq<T, D>(u, F));
    const double kd = g.quad ? (double)stiff_lob_diag<T, D>((T)g.h) : (double)stiff_diag<T, D>((T)g.h);
    const double ib = 1.0 / bfactor<D>(g, i, j, k);  // no-flux rows (1 on periodic grids)
    if constexpr (MODEL == 0) {
        pinv[idx] = (T)(1.0 / (theta * ib * ((double)inv_dt * m + (double)mob * (nd + (double)kappa * kd))));
    } else {
        const double a = ib * (double)inv_dt * m, b = ib * (double)mob * kd;
        const double c = -ib * (nd + (double)kappa * kd), d = ib * (double)m;
        const double det = a * d - b * c;
        T* P = pinv + 4 * idx;
        P[0] = (T)(d / det);
        P[1] = (T)(-b / det);
        P[2] = (T)(-c / det);
        P[3] = (T)(a / det);
    }
}

// Point preconditioner of the Cahn-Hilliard Newton system with mu eliminated (see
// newton.hip), S = inv_dt m + (mob / m) K [N'(c) + kappa K], rows / 2^b on no-flux grids:
//   pinv = 1 / (theta diag S),
// with the diagonal of K N'(c) taken as if f'' were constant around the node (cn f''(c))
// and that of K K (ck); a preconditioner may be approximate.  Where f'' < 0 outweighs
// the rest the diagonal is held at a tenth of its positive part.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_prec_schur(const T* __restrict__ U, T* __restrict__ pinv, Geom g, Lin<T> F,
                                                    T d0, T cn, T theta)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    const T d = max(fmaT(cn, F(U[idx], (T)1), d0), (T)0.1 * d0);
    pinv[idx] = (T)bfactor<D>(g, i, j, k) / (theta * d);
}

// What the Chebyshev polynomial needs to know of the field: an upper bound of the
// preconditioned operator's spectrum (see launch_spectrum), one maximum per block, and the
// mean of f'' over the block's tile of nodes.  Bound by its Gauss points, as k_prec is.
struct SpecCoef {
    double a;           // inv_dt m
    double jn;          // |J| times the mobility (nodal: m)
    double kd, km;      // the stiffness: diagonal, and the diagonal that bounds it from above
    double cn, cm;      // Cahn-Hilliard: of f'' in the diagonal, and in the bound
};
template <int D>
struct SpecTile {
    static constexpr int S = D == 2 ? 16 : 8, THREADS = D == 2 ? 256 : 512;  // S^D nodes
};

template <typename T, int D, int MODEL>
__global__ __launch_bounds__(SpecTile<D>::THREADS) void k_spectrum(const T* __restrict__ U,
                                                                   double* __restrict__ part, Geom g, Lin<T> F,
                                                                   SpecCoef c, int tx, int ty)
{
    constexpr int S = SpecTile<D>::S, NW = SpecTile<D>::THREADS / WAVE;
    const int t = blockIdx.x, th = threadIdx.x;
    const int i = t % tx * S + th % S, j = t / tx % ty * S + th / S % S, k = D == 2 ? 0 : t / tx / ty * S + th / (S * S);
    double hi = 0.0, fs = 0.0, cnt = 0.0;
    if (i < g.n[0] && j < g.n[1] && (D == 2 || k < g.n[2])) {
        T u[NB<D>::K];
        gather<T, D>(U, g, i, j, k, u);
        const T fc = F(u[NB<D>::K / 2], (T)1);
        double top, diag;
        if constexpr (MODEL == 0) {
            T np = fc, nd = fc;
            if (!g.quad) nd = quad_sum_sq_pos<T, D>(u, F, np);
            top = c.a + c.jn * (double)np + c.km;
            diag = c.a + c.jn * (double)nd + c.kd;
        } else {
            T f = (T)0;
#pragma unroll
            for (int q = 0; q < NB<D>::K; ++q) f = max(f, F(u[q], (T)1));
            const double d0 = c.a + c.kd;
            top = c.a + c.km + c.cm * (double)f;
            diag = max(d0 + c.cn * (double)fc, 0.1 * d0);
        }
        hi = diag > 0.0 ? top / diag : (double)INFINITY;
        fs = (double)fc;
        cnt = 1.0;
    }
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        hi = max(hi, __shfl_down(hi, o, WAVE));
        fs += __shfl_down(fs, o, WAVE);
        cnt += __shfl_down(cnt, o, WAVE);
    }
    __shared__ double sh[3][NW];
    if (th % WAVE == 0) {
        sh[0][th / WAVE] = hi;
        sh[1][th / WAVE] = fs;
        sh[2][th / WAVE] = cnt;
    }
    __syncthreads();
    if (th == 0) {
        for (int w = 1; w < NW; ++w) {
            hi = max(hi, sh[0][w]);
            fs += sh[1][w];
            cnt += sh[2][w];
        }
        part[2 * t] = hi;
        part[2 * t + 1] = fs / cnt;
    }
}

// The largest of the tiles' bounds, and the least of (mean of f'' + the stiffness energy of a
// mode that lives there) over windows of one tile and of 2, 4, ... tiles a side (means of
// the windows below, kept behind the tiles' pairs): kh (pi / side)^2 for every axis longer
// than the window.  (kh 0: the least tile.)  One block, bound by the latency of the levels:
// 2048^2 (16384 tiles) 20 us.
struct SpecWindows {
    int d[3], n[3];  // tiles and nodes of each axis
    double kh;       // kappa / h^2, or 0
};
__global__ __launch_bounds__(1024) void k_spectrum_ends(double* part, int nb, SpecWindows w, int side, int dim,
                                                        double* __restrict__ out)
{
    __shared__ double sh[2][1024];
    auto energy = [&](int len) {
        double e = 0.0;
        for (int a = 0; a < dim; ++a) e += w.n[a] > len ? 9.869604401089358 / ((double)len * len) : 0.0;
        return w.kh * e;
    };
    double hi = 0.0, f = (double)INFINITY, e = energy(side);
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += 1024) {
        hi = max(hi, part[2 * i]);
        f = min(f, part[2 * i + 1] + e);
    }
    const double* src = part + 1;
    double* dst = part + 2 * (long long)nb;
    int stride = 2, d0 = w.d[0], d1 = w.d[1], d2 = w.d[2];
    while (w.kh > 0.0 && (d0 > 1 || d1 > 1 || d2 > 1)) {
        const int e0 = (d0 + 1) / 2, e1 = (d1 + 1) / 2, e2 = (d2 + 1) / 2;
        side *= 2;
        e = energy(side);
        for (int i = threadIdx.x; i < e0 * e1 * e2; i += 1024) {
            const int x = i % e0 * 2, y = i / e0 % e1 * 2, z = i / e0 / e1 * 2;
            double sum = 0.0, cnt = 0.0;
            for (int c = 0; c < 8; ++c) {
                const int cx = x + (c & 1), cy = y + (c >> 1 & 1), cz = z + (c >> 2);
                if (cx >= d0 || cy >= d1 || cz >= d2) continue;
                sum += src[(long long)stride * (cx + (long long)d0 * (cy + (long long)d1 * cz))];
                cnt += 1.0;
            }
            dst[i] = sum / cnt;
            f = min(f, sum / cnt + e);
        }
        __syncthreads();
        src = dst;
        dst += e0 * e1 * e2;
        stride = 1;
        d0 = e0;
        d1 = e1;
        d2 = e2;
    }
    sh[0][threadIdx.x] = hi;
    sh[1][threadIdx.x] = f;
    __syncthreads();
    for (int st = 512; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            sh[0][threadIdx.x] = max(sh[0][threadIdx.x], sh[0][threadIdx.x + st]);
            sh[1][threadIdx.x] = min(sh[1][threadIdx.x], sh[1][threadIdx.x + st]);
        }
        __syncthreads();
    }
    if (threadIdx.x < 2)
        __hip_atomic_store(out + threadIdx.x, sh[threadIdx.x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// y = scale 2^b x (2^b: the boundary factor of the node's rows)
template <typename T, int D>
__global__ __launch_bounds__(256) void k_unrow(const T* __restrict__ x, T* __restrict__ y, Geom g, T scale)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    y[idx] = scale * (T)bfactor<D>(g, i, j, k) * x[idx];
}

// Jv for R = inv_dt M (U - U_old) + r(U)
// TRANS = 1 gives the transpose product w^T dR/dU (differs from J only for
// Cahn-Hilliard):  [inv_dt m w_c - (N'(c) + kappa K) w_mu ;  M K w_c + m w_mu].
// ACC = 1 adds the result into Jv instead of overwriting it.  g.cm: the
// (symmetric) consistent mass replaces m.  The preconditioner keeps the lumped
// mass as its approximation of the mass blocks.
template <typename T, int D, int MODEL, int TRANS, int ACC>
__global__ __launch_bounds__(256) void k_jvp(const T* __restrict__ U, const T* __restrict__ V,
                                             T* __restrict__ Jv, Geom g, Lin<T> F, T detJ, T kappa,
                                             T mob, T m, T inv_dt)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T u[NB<D>::K], v[NB<D>::K];
    gather<T, D>(U, g, i, j, k, u);
    const T h = (T)g.h;
    const T ib = (T)1 / (T)bfactor<D>(g, i, j, k);  // no-flux rows (1 on periodic grids)
    if constexpr (MODEL == 0) {
        gather<T, D>(V, g, i, j, k, v);
        const T Nv = g.quad ? m * F(u[NB<D>::K / 2], v[NB<D>::K / 2]) : detJ * quad_sum<T, D, true>(u, v, F);
        const T Kv = stiff_q<T, D>(g, v, h);
        const T mv = g.cm ? cmass<T, D>(v, h) : m * v[NB<D>::K / 2];
        const T out = (inv_dt * mv + mob * (Nv + kappa * Kv)) * ib;
        Jv[idx] = ACC ? Jv[idx] + out : out;
    } else {
        T w[NB<D>::K];
        gather<T, D>(V, g, i, j, k, v);         // c-plane of the direction
        gather<T, D>(V + g.N, g, i, j, k, w);   // mu-plane of the direction
        T oc, om;
        const T mv = g.cm ? cmass<T, D>(v, h) : m * v[NB<D>::K / 2];
        const T mw = g.cm ? cmass<T, D>(w, h) : m * w[NB<D>::K / 2];
        const T uc = u[NB<D>::K / 2];
        if constexpr (TRANS == 0) {
            const T Nv = g.quad ? m * F(uc, v[NB<D>::K / 2]) : detJ * quad_sum<T, D, true>(u, v, F);
            oc = inv_dt * mv + mob * stiff_q<T, D>(g, w, h);
            om = mw - (Nv + kappa * stiff_q<T, D>(g, v, h));
        } else {
            const T Nw = g.quad ? m * F(uc, w[NB<D>::K / 2]) : detJ * quad_sum<T, D, true>(u, w, F);
            oc = inv_dt * mv - (Nw + kappa * stiff_q<T, D>(g, w, h));
            om = mob * stiff_q<T, D>(g, v, h) + mw;
        }
        oc *= ib;
        om *= ib;
        Jv[idx] = ACC ? Jv[idx] + oc : oc;
        Jv[g.N + idx] = ACC ? Jv[g.N + idx] + om : om;
    }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void k_chem(const T* __restrict__ c, T* __restrict__ mu, Geom g,
                                              Cub<T> F, T detJ, T kappa, T inv_m)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T u[NB<D>::K];
    gather<T, D>(c, g, i, j, k, u);
    const T h = (T)g.h, m = D == 2 ? h * h : h * h * h;  // interior nodal mass h^D
    const T Nn = g.quad ? m * F(u[NB<D>::K / 2], (T)0) : detJ * quad_sum<T, D, false>(u, u, F);
    mu[idx] = (Nn + kappa * stiff_q<T, D>(g, u, h)) * inv_m;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void k_ch_update(const T* c, const T* __restrict__ mu, T* cout, Geom g,
                                                   T dtM_over_m)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T w[NB<D>::K];
    gather<T, D>(mu, g, i, j, k, w);
    cout[idx] = c[idx] - dtM_over_m * stiff_q<T, D>(g, w, (T)g.h);
}

template <typename T, int D>
__global__ __launch_bounds__(256) void k_ac_step(const T* __restrict__ eta, T* __restrict__ out,
                                                 Geom g, Cub<T> F, T detJ, T kappa, T dtL_over_m)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    int i, j, k;
    if (!node_of<D>(g, idx, i, j, k)) return;
    T u[NB<D>::K];
    gather<T, D>(eta, g, i, j, k, u);
    const T h = (T)g.h, m = D == 2 ? h * h : h * h * h;  // interior nodal mass h^D
    const T Nn = g.quad ? m * F(u[NB<D>::K / 2], (T)0) : detJ * quad_sum<T, D, false>(u, u, F);
    const T r = Nn + kappa * stiff_q<T, D>(g, u, h);
    out[idx] = u[NB<D>::K / 2] - dtL_over_m * r;
}

// ---- energy and mass ---------------------------------------------------------
// Each thread owns the element whose lower corner is its node (none past the upper
// boundary of a no-flux grid) and the mass term of its node.
__device__ __forceinline__ double f_local(int fe, double W, double q)
{
    if (fe == 0) {
        const double t = q * q - 1.0;
        return 0.25 * W * t * t;
    }
    const double t = q * (1.0 - q);
    return W * t * t;
}

constexpr int EBLK = 256;
// blocks of the energy sum: enough waves to cover its latency (two blocks a CU in FP64), few
// enough that the one block that adds their sums reads 8 pairs a thread at most
constexpr int EMAX = 2048;

// Element energy from its corner values.  A gradient component is constant along its own
// axis, so the 2^D points share 2^(D-1) values of it, and the values at the points are
// interpolated axis by axis: 50 FP64 operations an element in 2-D (150 point by point, with
// divisions by h).  With the sum of the block sums, FP64 no-flux: 1001 x 777 11.6 -> 8.2
// us, 2048^2 44 -> 20, 130 x 121 x 117 35 -> 21.
template <int D>
__device__ __forceinline__ double element_energy(const double (&u)[1 << D], const double (&B)[2][2], int fe, double W,
                                                 double kih2)
{
    constexpr int NC = 1 << D;
    double f = 0.0, grad = 0.0;
    // values at the points, one axis after the other
    double q[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) q[i] = u[i];
#pragma unroll
    for (int ax = 0; ax < D; ++ax)
#pragma unroll
        for (int i = 0; i < NC; ++i)
            if (!(i >> ax & 1)) {
                const double lo = q[i], hi = q[i | 1 << ax];
                q[i] = B[0][0] * lo + B[0][1] * hi;
                q[i | 1 << ax] = B[1][0] * lo + B[1][1] * hi;
            }
#pragma unroll
    for (int i = 0; i < NC; ++i) f += f_local(fe, W, q[i]);
    // squared differences along each axis, interpolated along the others
#pragma unroll
    for (int ax = 0; ax < D; ++ax) {
        double d[NC / 2];
#pragma unroll
        for (int i = 0; i < NC / 2; ++i) {
            const int lo = (i & ((1 << ax) - 1)) | (i >> ax) << (ax + 1);  // i with a 0 inserted at bit ax
            d[i] = u[lo | 1 << ax] - u[lo];
        }
#pragma unroll
        for (int o = 0; o < D - 1; ++o)
#pragma unroll
            for (int i = 0; i < NC / 2; ++i)
                if (!(i >> o & 1)) {
                    const double lo = d[i], hi = d[i | 1 << o];
                    d[i] = B[0][0] * lo + B[0][1] * hi;
                    d[i | 1 << o] = B[1][0] * lo + B[1][1] * hi;
                }
#pragma unroll
        for (int i = 0; i < NC / 2; ++i) grad += d[i] * d[i];
    }
    return f + kih2 * grad;  // (kappa / 2) / h^2, twice
}

template <typename T, int D>
__global__ __launch_bounds__(EBLK) void k_energy(const T* __restrict__ c, double* __restrict__ part,
                                                 Geom g, int fe, double W, double kih2)
{
    double e = 0.0, ms = 0.0;
    const double h = g.h, detJ = D == 2 ? 0.25 * h * h : 0.125 * h * h * h, m = D == 2 ? h * h : h * h * h;
    // 1-D shape functions at the quadrature points: Gauss (GP, GM), or
    // Gauss-Lobatto (the points are the nodes: the identity)
    const double bp = g.quad ? 1.0 : GP, bm = g.quad ? 0.0 : GM;
    const double B[2][2] = {{bp, bm}, {bm, bp}};
    for (long long idx = (long long)blockIdx.x * EBLK + threadIdx.x; idx < g.N; idx += (long long)gridDim.x * EBLK) {
        int i, j, k;
        node_of<D>(g, idx, i, j, k);
        const int ii[2] = {i, wrap(i + 1, g.n[0])}, jj[2] = {j, wrap(j + 1, g.n[1])};
        const int kk[2] = {k, D == 3 ? wrap(k + 1, g.n[2]) : 0};
        double u[1 << D];
#pragma unroll
        for (int a = 0; a < 1 << D; ++a)
            u[a] = c[((D == 3 ? (long long)kk[a >> 2] * g.n[1] : 0) + jj[a >> 1 & 1]) * g.n[0] + ii[a & 1]];
        double en = detJ * element_energy<D>(u, B, fe, W, kih2), mn = m * u[0];
        // no-flux: the element exists only below the upper boundary; lumped mass h^d / 2^b
        if (g.bc) {
            const bool elem = i + 1 < g.n[0] && j + 1 < g.n[1] && (D == 2 || k + 1 < g.n[2]);
            if (!elem) en = 0.0;
            if (edge_count(i, g.n[0])) mn *= 0.5;
            if (edge_count(j, g.n[1])) mn *= 0.5;
            if (D == 3 && edge_count(k, g.n[2])) mn *= 0.5;
        }
        e += en;
        ms += mn;
    }
    // block reduction, fixed order: wave shuffle tree, then waves in order
    __shared__ double se[EBLK / WAVE], sm[EBLK / WAVE];
    for (int off = WAVE / 2; off > 0; off >>= 1) {
        e += __shfl_down(e, off, WAVE);
        ms += __shfl_down(ms, off, WAVE);
    }
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    if (lane == 0) {
        se[wv] = e;
        sm[wv] = ms;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < EBLK / WAVE; ++w) {
            a += se[w];
            b += sm[w];
        }
        part[2 * blockIdx.x] = a;
        part[2 * blockIdx.x + 1] = b;
    }
}

// single block sums the per-block partials in a fixed order
__global__ __launch_bounds__(256) void k_reduce_pairs(const double* __restrict__ part, int nb,
                                                      double* __restrict__ out)
{
    __shared__ double se[256], sm[256];
    double a = 0.0, b = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < nb; i += 256) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    se[threadIdx.x] = a;
    sm[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            se[threadIdx.x] += se[threadIdx.x + s];
            sm[threadIdx.x] += sm[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = se[0];
        out[1] = sm[0];
    }
}

inline dim3 grid_for(const Geom& g) { return dim3((unsigned)((g.N + 255) / 256)); }

template <typename T>
Cub<T> cub_of(const FreeEnergy& f, double scale)
{
    return Cub<T>{(T)(scale * f.a1), (T)(scale * f.a2), (T)(scale * f.a3)};
}

}  // namespace

int energy_blocks(const Geom& g) { return (int)((g.N + EBLK - 1) / EBLK); }

void launch_reduce_pairs(const double* part, int nb, double* out, hipStream_t s)
{
    k_reduce_pairs<<<1, 256, 0, s>>>(part, nb, out);
}

#define DIM_SWITCH(g, ...)         \
    if ((g).dim == 2) {            \
        constexpr int D = 2;       \
        __VA_ARGS__;               \
    } else {                       \
        constexpr int D = 3;       \
        __VA_ARGS__;               \
    }

// Where the marching kernels beat one thread per node for the weak forms without a
// direction.  A march is a serial chain of rows or planes (5 us a pass in 2-D, 4-6 in 3-D
// however small the grid), the node kernels evaluate every Gauss point 4 or 8 times in
// parallel.  Measured, march / nodes, us, Gauss, no-flux:
//   3-D step    64^3 FP32 Allen-Cahn 6.2 / 5.4, Cahn-Hilliard 11.4 / 9.5, FP64 15.7 / 15.4;
//               72 x 65 x 60 6.2 / 6.7, 11.4 / 11.9, FP64 15.5 / 20.5
//   3-D Cahn-Hilliard residual (two passes for one) FP32 72 x 65 x 60 9.1 / 7.7,
//               80^3 11.2 / 11.2, 96^3 13.9 / 17.9; FP64 72 x 65 x 60 11.7 / 13.1
//   2-D residual FP32 1001 x 777 Allen-Cahn 5.4 / 5.1, Cahn-Hilliard 6.3 / 6.5, 1400^2
//               7.4 / 9.8, 8.7 / 12.9; FP64 500^2 5.2 / 3.9, 6.5 / 5.2, 1001 x 777 6.5 / 7.3,
//               8.3 / 10.3
// so: 2-D fields of at least 4 MiB, 3-D more than 64^3 nodes (2^19 where two FP32 passes
// stand against one).
bool march_pays(const Geom& g, size_t esz, bool two_passes)
{
    if (g.dim == 2) return (size_t)g.N * esz >= (size_t(4) << 20);
    return g.N > (two_passes && esz == 4 ? 1ll << 19 : 1ll << 18);
}

template <typename T>
void launch_residual(const Geom& g, int model, const FreeEnergy& f, double kappa, double mob,
                     const T* U, T* r, hipStream_t s, const T* Uold, double inv_dt)
{
    const double detJ = std::pow(0.5 * g.h, g.dim), m = std::pow(g.h, g.dim);
    if (!g.cm && march_pays(g, sizeof(T), g.dim == 3 && model == 1)) {
        // marching kernels: every Gauss point once.  In 3-D the Cahn-Hilliard rows take two
        // passes (they share no quadrature); both fit or neither does.
        March<T> a;
        a.u = U;
        a.rows = 1;
        if (model == 0) {
            a.out = r;
            a.nq = mob;
            a.kv = mob * kappa;
            a.s0 = Uold ? inv_dt * m : 0.0;
            a.p1 = Uold;
            if (launch_march<T>(g, MOP_GRAD, ME_OUT, f, a, s)) return;
        } else if (g.dim == 2) {
            a.v = U + g.N;
            a.out = r;
            a.out2 = r + g.N;
            a.kv = kappa;
            a.kw = mob;
            a.s0 = m;
            a.s1 = Uold ? inv_dt * m : 0.0;
            a.p1 = Uold;
            if (launch_march2d<T>(g, MOP_GRAD, ME_CHRES, f, a, s)) return;
        } else {
            a.out = r + g.N;
            a.p0 = U + g.N;
            a.kv = kappa;
            a.s0 = m;
            March<T> b;
            b.v = U + g.N;
            b.base = U;
            b.p1 = Uold;
            b.out = r;
            b.kv = mob;
            b.s0 = Uold ? inv_dt * m : 0.0;
            b.rows = 1;
            if (launch_march<T>(g, MOP_GRAD, ME_MU, f, a, s) && launch_march<T>(g, MOP_STIFF, ME_OUT, f, b, s)) return;
        }
    }
    DIM_SWITCH(g, {
        if (model == 0)
            k_residual<T, D, 0><<<grid_for(g), 256, 0, s>>>(U, Uold, r, g, cub_of<T>(f, 1.0),
                                                             (T)detJ, (T)kappa, (T)mob, (T)m,
                                                             (T)inv_dt);
        else
            k_residual<T, D, 1><<<grid_for(g), 256, 0, s>>>(U, Uold, r, g, cub_of<T>(f, 1.0),
                                                             (T)detJ, (T)kappa, (T)mob, (T)m,
                                                             (T)inv_dt);
    });
}

template <typename T>
void launch_jvp(const Geom& g, int model, const FreeEnergy& f, double kappa, double mob,
                double inv_dt, const T* U, const T* v, T* Jv, hipStream_t s, int trans, int acc)
{
    if (g.dim == 3 && model == 0 && !acc) {
        March<T> a;
        a.u = U;
        a.v = v;
        a.out = Jv;
        a.nq = mob;
        a.kv = mob * kappa;
        a.s0 = inv_dt * std::pow(g.h, 3);
        a.rows = 1;
        if (launch_march3d<T>(g, MOP_JVP, ME_OUT, f, a, s)) return;
    }
    if (g.dim == 3 && !acc && !g.cm && !g.quad) {
        launch_jvp3d<T>(g, model, f, kappa, mob, inv_dt, U, v, Jv, s, trans);
        return;
    }
    // Allen-Cahn's Jacobian is symmetric, so its transpose product is the product
    if (!acc && (model == 0 || !trans) && launch_jvp2d_stream<T>(g, model, f, kappa, mob, inv_dt, U, v, Jv, s))
        return;
    const double detJ = std::pow(0.5 * g.h, g.dim), m = std::pow(g.h, g.dim);
    Lin<T> F{(T)f.b0, (T)f.b1, (T)f.b2};
#define JVP_L(MODEL, TR, AC)                                                                    \
    k_jvp<T, D, MODEL, TR, AC><<<grid_for(g), 256, 0, s>>>(U, v, Jv, g, F, (T)detJ, (T)kappa,  \
                                                           (T)mob, (T)m, (T)inv_dt)
    DIM_SWITCH(g, {
        if (model == 0) {
            if (acc) JVP_L(0, 0, 1); else JVP_L(0, 0, 0);
        } else if (!trans) {
            if (acc) JVP_L(1, 0, 1); else JVP_L(1, 0, 0);
        } else {
            if (acc) JVP_L(1, 1, 1); else JVP_L(1, 1, 0);
        }
    });
#undef JVP_L
}

template <typename T>
void launch_prec(const Geom& g, int model, const FreeEnergy& f, double kappa, double mob,
                 double inv_dt, const T* U, T* pinv, hipStream_t s, double theta)
{
    const double detJ = std::pow(0.5 * g.h, g.dim), m = std::pow(g.h, g.dim);
    Lin<T> F{(T)f.b0, (T)f.b1, (T)f.b2};
    DIM_SWITCH(g, {
        if (model == 0)
            k_prec<T, D, 0><<<grid_for(g), 256, 0, s>>>(U, pinv, g, F, (T)detJ, (T)kappa, (T)mob,
                                                         (T)m, (T)inv_dt, theta);
        else
            k_prec<T, D, 1><<<grid_for(g), 256, 0, s>>>(U, pinv, g, F, (T)detJ, (T)kappa, (T)mob,
                                                         (T)m, (T)inv_dt, 1.0);
    });
}

template <typename T>
void launch_prec_schur(const Geom& g, const FreeEnergy& f, double kappa, double mob, double inv_dt, double theta,
                       const T* U, T* pinv, hipStream_t s)
{
    const double m = std::pow(g.h, g.dim), hk = g.dim == 3 ? g.h : 1.0;
    const StencilDiag d = stencil_diag(g);
    const Lin<T> F{(T)f.b0, (T)f.b1, (T)f.b2};
    const double d0 = inv_dt * m + mob / m * kappa * d.kk * hk * hk, cn = mob * d.km * hk;
    DIM_SWITCH(g, { k_prec_schur<T, D><<<grid_for(g), 256, 0, s>>>(U, pinv, g, F, (T)d0, (T)cn, (T)theta); });
}

template <typename T>
bool launch_spectrum(const Geom& g, int model, const FreeEnergy& f, double kappa, double mob, double inv_dt,
                     const T* U, double* part, long long part_max, double* out, hipStream_t s)
{
    const int ts = g.dim == 2 ? SpecTile<2>::S : SpecTile<3>::S;
    const long long tx = (g.n[0] + ts - 1) / ts, ty = (g.n[1] + ts - 1) / ts;
    const long long tz = g.dim == 3 ? (g.n[2] + ts - 1) / ts : 1, nb = tx * ty * tz;
    long long room = 2 * nb;  // and the windows of every size
    for (long long a = tx, b = ty, c = tz; a > 1 || b > 1 || c > 1;) {
        a = (a + 1) / 2;
        b = (b + 1) / 2;
        c = (c + 1) / 2;
        room += a * b * c;
    }
    if (room > part_max || nb > (1ll << 30)) return false;
    const double m = std::pow(g.h, g.dim), hk = g.dim == 3 ? g.h : 1.0;
    const StencilDiag d = stencil_diag(g);
    const Lin<T> F{(T)f.b0, (T)f.b1, (T)f.b2};
    SpecCoef c{};
    c.a = inv_dt * m;
    if (model == 0) {
        c.jn = mob * (g.quad ? m : std::pow(0.5 * g.h, g.dim));
        c.kd = mob * kappa * d.kd * hk;
        c.km = mob * kappa * d.kmax * hk;
    } else {
        c.kd = mob / m * kappa * d.kk * hk * hk;
        c.km = mob / m * kappa * d.kmax * d.kmax * hk * hk;
        c.cn = mob * d.km * hk;
        c.cm = mob * d.kmmax * hk;
    }
    DIM_SWITCH(g, {
        if (model == 0)
            k_spectrum<T, D, 0><<<(unsigned)nb, SpecTile<D>::THREADS, 0, s>>>(U, part, g, F, c, (int)tx, (int)ty);
        else
            k_spectrum<T, D, 1><<<(unsigned)nb, SpecTile<D>::THREADS, 0, s>>>(U, part, g, F, c, (int)tx, (int)ty);
    });
    const SpecWindows w{{(int)tx, (int)ty, (int)tz},
                        {g.n[0], g.n[1], g.dim == 3 ? g.n[2] : 1},
                        model == 0 ? kappa / (g.h * g.h) : 0.0};
    k_spectrum_ends<<<1, 1024, 0, s>>>(part, (int)nb, w, ts, g.dim, out);
    return true;
}

template <typename T>
void launch_unrow(const Geom& g, double scale, const T* x, T* y, hipStream_t s)
{
    DIM_SWITCH(g, { k_unrow<T, D><<<grid_for(g), 256, 0, s>>>(x, y, g, (T)scale); });
}

template <typename T>
void launch_chem(const Geom& g, const FreeEnergy& f, double kappa, const T* c, T* mu,
                 hipStream_t s)
{
    const double detJ = std::pow(0.5 * g.h, g.dim), m = std::pow(g.h, g.dim);
    March<T> a;
    a.u = c;
    a.out = mu;
    a.nq = 1.0 / m;
    a.kv = kappa / m;
    if (march_pays(g, sizeof(T), false) && launch_march<T>(g, MOP_GRAD, ME_OUT, f, a, s)) return;
    DIM_SWITCH(g, {
        k_chem<T, D><<<grid_for(g), 256, 0, s>>>(c, mu, g, cub_of<T>(f, 1.0), (T)detJ, (T)kappa,
                                                  (T)(1.0 / m));
    });
}

template <typename T>
void launch_ch_update(const Geom& g, double dtM, const T* c, const T* mu, T* c_out, hipStream_t s)
{
    const double m = std::pow(g.h, g.dim);
    March<T> a;
    a.v = mu;
    a.base = c;
    a.out = c_out;
    a.kv = dtM / m;
    if (march_pays(g, sizeof(T), false) && launch_march<T>(g, MOP_STIFF, ME_SUB, FreeEnergy{}, a, s)) return;
    DIM_SWITCH(g, { k_ch_update<T, D><<<grid_for(g), 256, 0, s>>>(c, mu, c_out, g, (T)(dtM / m)); });
}

template <typename T>
void launch_ac_step(const Geom& g, const FreeEnergy& f, double kappa, double dtL, const T* eta,
                    T* eta_out, hipStream_t s)
{
    const double detJ = std::pow(0.5 * g.h, g.dim), m = std::pow(g.h, g.dim);
    March<T> a;
    a.u = eta;
    a.out = eta_out;
    a.nq = dtL / m;
    a.kv = dtL * kappa / m;
    if (march_pays(g, sizeof(T), false) && launch_march<T>(g, MOP_GRAD, ME_SUB, f, a, s)) return;
    DIM_SWITCH(g, {
        k_ac_step<T, D><<<grid_for(g), 256, 0, s>>>(eta, eta_out, g, cub_of<T>(f, 1.0), (T)detJ,
                                                     (T)kappa, (T)(dtL / m));
    });
}

template <typename T>
void launch_energy(const Geom& g, const FreeEnergy& f, double kappa, const T* c, double* partials,
                   double* out, hipStream_t s)
{
    const int nb = std::min(energy_blocks(g), EMAX);
    DIM_SWITCH(g, { k_energy<T, D><<<nb, EBLK, 0, s>>>(c, partials, g, f.fe, f.W, kappa / (g.h * g.h)); });
    k_reduce_pairs<<<1, 256, 0, s>>>(partials, nb, out);
}

#define INST(T)                                                                                   \
    template void launch_residual<T>(const Geom&, int, const FreeEnergy&, double, double, const T*, \
                                     T*, hipStream_t, const T*, double);                          \
    template void launch_jvp<T>(const Geom&, int, const FreeEnergy&, double, double, double,       \
                                const T*, const T*, T*, hipStream_t, int, int);                   \
    template void launch_prec<T>(const Geom&, int, const FreeEnergy&, double, double, double,      \
                                 const T*, T*, hipStream_t, double);                              \
    template void launch_prec_schur<T>(const Geom&, const FreeEnergy&, double, double, double, double, const T*, \
                                       T*, hipStream_t);                                          \
    template bool launch_spectrum<T>(const Geom&, int, const FreeEnergy&, double, double, double, const T*, \
                                     double*, long long, double*, hipStream_t);                    \
    template void launch_unrow<T>(const Geom&, double, const T*, T*, hipStream_t);                 \
    template void launch_chem<T>(const Geom&, const FreeEnergy&, double, const T*, T*, hipStream_t); \
    template void launch_ch_update<T>(const Geom&, double, const T*, const T*, T*, hipStream_t);   \
    template void launch_ac_step<T>(const Geom&, const FreeEnergy&, double, double, const T*, T*,  \
                                    hipStream_t);                                                 \
    template void launch_energy<T>(const Geom&, const FreeEnergy&, double, const T*, double*,      \
                                   double*, hipStream_t);
INST(float)
INST(double)

}  // namespace pfk
