// k_march3d.hip -- node operators of the 3-D weak forms, marched along z in registers.
//
// See march.hpp for the operators and what is done with them.  A 64-lane wave is cut into
// G groups of W = 64 / G lanes; a group owns W - 2 output columns (one halo lane per
// side) of R rows and marches through a chunk of planes.  Per plane a lane loads its
// R + 2 rows (the next plane's loads in flight), takes x-neighbours from the adjacent
// lanes by DPP, and evaluates each element of the slab between two planes once:
// x- and y-interpolants of the new plane, the z-interpolation with the kept ones of the
// plane below to the 8 Gauss points, f' (or f'' v), and the transposed passes back; the
// upper plane's half of the scatter is kept for the next slab.  The stiffness uses the
// closed Q1 stencil (centre 8/3, edges -1/6, corners -1/12, faces 0, times h), split
// into what each plane contributes.  No LDS, no barriers, no atomics.
//
// Why this split: the node-centric kernels evaluate every Gauss point 8 times (about
// 900 VALU per node), the LDS tile kernel once but with 2 barriers per plane and 30
// staged words per element (261 VALU per wave and plane).  Here a plane costs about 90
// VALU per node row (110 with a direction) and R + 1 element rows serve R node rows.
// Halo lanes cost W / (W - 2) and the two warm-up planes of a chunk (pz + 2) / pz; the
// launcher picks G in 1..4 for the fewest waves, and R and pz by shape_gauss or
// shape_light.  Measured, explicit Cahn-Hilliard step (chemical potential, then update):
// FP32 130 x 121 x 117 40.5 -> 23.7 us, 256 x 200 x 180 66 us; the potential alone there
// takes 36 us of about 29 us VALU issue.
#include <algorithm>
#include <cmath>

#include "device.hpp"
#include "kernels.hpp"
#include "march.hpp"
#include "stream2d.hpp"

namespace pfk {
namespace {

template <typename T>
struct MC3 {           // coefficients in the field type
    T a, b, c;         // GRAD: q (a + q (b + c q)); JVP: (a + q (b + c q)) v  (|J| folded in)
    T kv, kl;          // times Lap3 (h / 12 folded in), nodal: times LapN3 (h folded in); its rest
    T s0, s1, s2;
    T g1, g2, g3;      // ME_ADJ: f' at W = 1
};

struct ML3 {           // launch geometry
    int nx, ny, nz, W, G, nstrips, items, wpc, pz, nwaves;
    unsigned bytes;    // one field
};

// 12 / h times the Q1 stiffness row of plane z - 1, as planes are pushed, from differences
// of neighbouring values (which FP32 forms exactly where the field is smooth; the
// residual's rounding floor is theirs).  With e = 2 a - a(x-1) - a(x+1), f the same along
// y and E = e(y-1) + e(y+1), a plane contributes P = 4 f + 2 E to its own row and
// Q = 4 f + 2 e + E to the rows of the planes beside it:
//   12 (2 a - a(z-1) - a(z+1)) + P + Q(z-1) + Q(z+1)
template <typename T, int R>
struct Lap3 {
    T acc[R], qp[R], ap[R], dp[R];  // P + Q(z-1) of the last plane; its Q and a; a - a(z-1) there

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int j = 0; j < R; ++j) acc[j] = qp[j] = ap[j] = dp[j] = (T)0;
    }
    __device__ __forceinline__ void push(const T (&a)[R + 2], T (&lap)[R])
    {
        T e[R + 2], d[R + 1];
#pragma unroll
        for (int j = 0; j < R + 2; ++j) e[j] = (a[j] - from_left(a[j])) + (a[j] - from_right(a[j]));
#pragma unroll
        for (int j = 0; j < R + 1; ++j) d[j] = a[j + 1] - a[j];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T f4 = (T)4 * (d[j] - d[j + 1]);
            const T E = e[j] + e[j + 2];
            const T q = fmaT((T)2, e[j + 1], f4 + E);
            const T dz = a[j + 1] - ap[j];
            lap[j] = fmaT((T)12, dp[j] - dz, acc[j] + q);
            acc[j] = fmaT((T)2, E, f4 + qp[j]);
            qp[j] = q;
            ap[j] = a[j + 1];
            dp[j] = dz;
        }
    }
};

// nodal quadrature: 6 a - (x-, y- and z-neighbours), again from differences
template <typename T, int R>
struct LapN3 {
    T acc[R], ap[R];

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int j = 0; j < R; ++j) acc[j] = ap[j] = (T)0;
    }
    __device__ __forceinline__ void push(const T (&a)[R + 2], T (&lap)[R])
    {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T c = a[j + 1], dz = c - ap[j];
            lap[j] = acc[j] - dz;
            acc[j] = ((c - from_left(c)) + (c - from_right(c))) + ((c - a[j]) + (c - a[j + 2])) + dz;
            ap[j] = c;
        }
    }
};

// x- and y-interpolants of one plane at the 4 in-plane Gauss abscissae of the R + 1
// element rows: q[e] = {left lower, left upper, right lower, right upper}
template <typename T, int R>
__device__ __forceinline__ void interp_plane(const T (&a)[R + 2], T (&q)[R + 1][4])
{
    const T gp = (T)GP, gm = (T)GM;
    T l[R + 2], r[R + 2];
#pragma unroll
    for (int j = 0; j < R + 2; ++j) {
        const T d = from_right(a[j]) - a[j];
        l[j] = fmaT(gm, d, a[j]);
        r[j] = fmaT(gp, d, a[j]);
    }
#pragma unroll
    for (int e = 0; e < R + 1; ++e) {
        const T dl = l[e + 1] - l[e], dr = r[e + 1] - r[e];
        q[e][0] = fmaT(gm, dl, l[e]);
        q[e][1] = fmaT(gp, dl, l[e]);
        q[e][2] = fmaT(gm, dr, r[e]);
        q[e][3] = fmaT(gp, dr, r[e]);
    }
}

// The quadrature pipeline: push the newest plane z of u (and v) and get the sums of
// plane z - 1.
// (SUM: asum[j] receives sum_q f1'(u_q) v_q of the element above node row j, planes z-1..z)
template <typename T, int R, int OP, bool SUM = false>
struct Quad3 {
    T asum[SUM ? R : 1];
    T qu[R + 1][4], up[R + 1][4], qv[OP == MOP_JVP ? R + 1 : 1][4];

    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int e = 0; e < R + 1; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                qu[e][i] = up[e][i] = (T)0;
                if constexpr (OP == MOP_JVP) qv[e][i] = (T)0;
            }
    }
    __device__ __forceinline__ void prime(const T (&u)[R + 2], const T (&v)[R + 2])
    {
        interp_plane<T, R>(u, qu);
        if constexpr (OP == MOP_JVP) interp_plane<T, R>(v, qv);
    }
    __device__ __forceinline__ void push(const T (&u)[R + 2], const T (&v)[R + 2], const MC3<T>& k, T (&s)[R])
    {
        const T gp = (T)GP, gm = (T)GM;
        T nu[R + 1][4], nv[R + 1][4];
        interp_plane<T, R>(u, nu);
        if constexpr (OP == MOP_JVP) interp_plane<T, R>(v, nv);
        T dn[R + 1][2], hi[R + 1][2];  // y-scatter of plane z - 1: to the lower / upper node row (left, right)
#pragma unroll
        for (int e = 0; e < R + 1; ++e) {
            T h[4], as = (T)0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T du = nu[e][i] - qu[e][i];
                const T u0 = fmaT(gm, du, qu[e][i]), u1 = fmaT(gp, du, qu[e][i]);
                T f0 = fmaT(fmaT(k.c, u0, k.b), u0, k.a), f1 = fmaT(fmaT(k.c, u1, k.b), u1, k.a);
                if constexpr (OP == MOP_GRAD) {
                    f0 *= u0;
                    f1 *= u1;
                } else {
                    const T dv = nv[e][i] - qv[e][i];
                    const T v0 = fmaT(gm, dv, qv[e][i]), v1 = fmaT(gp, dv, qv[e][i]);
                    f0 *= v0;
                    f1 *= v1;
                    if constexpr (SUM)
                        as = fmaT(cubic(u1, k.g1, k.g2, k.g3), v1, fmaT(cubic(u0, k.g1, k.g2, k.g3), v0, as));
                    qv[e][i] = nv[e][i];
                }
                qu[e][i] = nu[e][i];
                const T d = f0 - f1;
                h[i] = up[e][i] + fmaT(gp, d, f1);  // plane z - 1 complete
                up[e][i] = fmaT(gm, d, f1);         // plane z, lower slab
            }
            if constexpr (SUM)
                if (e >= 1) asum[e - 1] = as;  // lower corner at node row e - 1 of the block
            const T dl = h[0] - h[1], dr = h[2] - h[3];
            dn[e][0] = fmaT(gp, dl, h[1]);
            hi[e][0] = fmaT(gm, dl, h[1]);
            dn[e][1] = fmaT(gp, dr, h[3]);
            hi[e][1] = fmaT(gm, dr, h[3]);
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T l = hi[j][0] + dn[j + 1][0], r = hi[j][1] + dn[j + 1][1];
            const T d = l - r;
            s[j] = fmaT(gp, d, r) + from_left(fmaT(gm, d, r));
        }
    }
};

// wave -> (plane chunk, wave of the chunk); group g of the wave -> item (strip, row block)
template <typename T, int R, int OP, int EPI, bool MIRROR, bool NODAL>
__global__ __launch_bounds__(256) void k_march3d(March<T> p, ML3 L, MC3<T> k)
{
    const int wave = uniform_wave();
    if (wave >= L.nwaves) return;  // uniform per wave
    const int zc = wave / L.wpc;
    const int z0 = zc * L.pz, z1 = min(L.nz, z0 + L.pz);
    const int lane = threadIdx.x & (WAVE - 1);
    const int grp = min((lane >= L.W) + (lane >= 2 * L.W) + (lane >= 3 * L.W), L.G - 1);
    const int col = lane - grp * L.W;  // col >= W past the last group
    const int item = (wave - zc * L.wpc) * L.G + grp;
    const bool live = item < L.items && col >= 1 && col < L.W - 1;
    const int it = min(item, L.items - 1);
    const int strip = it % L.nstrips, yb = it / L.nstrips;
    const int xl = strip * (L.W - 2) - 1 + col, y0 = yb * R;
    const int x = near_index<MIRROR>(xl, L.nx);
    constexpr int ES = (int)sizeof(T);
    int vo[R + 2];  // byte offset of each row inside a plane
#pragma unroll
    for (int j = 0; j < R + 2; ++j) vo[j] = (near_index<MIRROR>(y0 - 1 + j, L.ny) * L.nx + x) * ES;
    const bool colok = live && xl < L.nx;
    T xs = (T)1;  // no-flux: 1 / 2^b of the columns and rows
    if (MIRROR && p.rows) xs = edge_count(x, L.nx) ? (T)0.5 : (T)1;
    const int planeb = L.nx * L.ny * ES;
    auto plane_off = [&](int z) {
        if constexpr (MIRROR) {
            z = z < 0 ? -z : (z >= L.nz ? 2 * (L.nz - 1) - z : z);
        } else {
            z = z < 0 ? z + L.nz : (z >= L.nz ? z - L.nz : z);
        }
        return z * planeb;
    };
    constexpr bool HASU = OP != MOP_STIFF, HASV = OP != MOP_GRAD;
    constexpr bool ADJ = EPI == ME_ADJ || EPI == ME_ADJK;
    T vf[ADJ && MIRROR ? R + 2 : 1];  // 2^b of the lane's column and rows
    if constexpr (ADJ && MIRROR) {
#pragma unroll
        for (int j = 0; j < R + 2; ++j)
            vf[j] = p.scale ? (T)(1 << (edge_count(x, L.nx) + edge_count(near_index<true>(y0 - 1 + j, L.ny), L.ny))) : (T)1;
    }
    double sA = 0.0, sB = 0.0;
    const auto ru = make_rsrc(HASU ? p.u : p.v, L.bytes);
    const auto rv = make_rsrc(HASV ? p.v : p.u, L.bytes);
    const auto ro = make_rsrc(p.out, L.bytes);
    const auto rb = make_rsrc(p.base ? p.base : p.out, L.bytes);
    const auto r0 = make_rsrc(p.p0 ? p.p0 : p.out, L.bytes);
    const auto r1 = make_rsrc(p.p1 ? p.p1 : p.out, L.bytes);
    const auto r2 = make_rsrc(p.p2 ? p.p2 : p.out, L.bytes);

    Quad3<T, R, NODAL ? MOP_STIFF : OP, EPI == ME_ADJ> qd;
    using LapT = std::conditional_t<NODAL, LapN3<T, R>, Lap3<T, R>>;
    LapT lp;
    if constexpr (HASU && !NODAL) qd.init();
    lp.init();
    T uc[R], vc[R];  // centre values of plane z - 1
#pragma unroll
    for (int j = 0; j < R; ++j) uc[j] = vc[j] = (T)0;

    T nu[R + 2], nv[R + 2];
    auto fetch = [&](int z) {
        const int so = plane_off(z);
#pragma unroll
        for (int j = 0; j < R + 2; ++j) {
            if constexpr (HASU) nu[j] = bload<T>(ru, vo[j], so);
            if constexpr (HASV) nv[j] = bload<T>(rv, vo[j], so);
        }
    };
    fetch(z0 - 1);
    for (int z = z0 - 1; z <= z1; ++z) {
        T u[R + 2], v[R + 2];
#pragma unroll
        for (int j = 0; j < R + 2; ++j) {
            u[j] = HASU ? nu[j] : (T)0;
            v[j] = HASV ? nv[j] : (T)0;
        }
        if constexpr (ADJ && MIRROR) {
            const int zr = z < 0 ? -z : (z >= L.nz ? 2 * (L.nz - 1) - z : z);
            const T zf = p.scale && edge_count(zr, L.nz) ? (T)2 : (T)1;
#pragma unroll
            for (int j = 0; j < R + 2; ++j) v[j] *= vf[j] * zf;
        }
        fetch(min(z + 1, z1));  // past the chunk the last plane is read again (a cache hit)
        // what the epilogue reads of plane z - 1, in flight during the compute
        const bool emit = z > z0;
        const int so = (emit ? z - 1 : z0) * planeb;
        T eb[R], e0[R], e1[R], e2[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            eb[j] = p.base ? bload<T>(rb, vo[j + 1], so) : (T)0;
            e0[j] = (EPI == ME_MU || EPI == ME_BACK || EPI == ME_CHEB || EPI == ME_ADJK) ? bload<T>(r0, vo[j + 1], so) : (T)0;
            e1[j] = (EPI == ME_CHEB || ((EPI == ME_OUT || EPI == ME_ADJ) && p.p1)) ? bload<T>(r1, vo[j + 1], so) : (T)0;
            e2[j] = EPI == ME_CHEB && p.p2 ? bload<T>(r2, vo[j + 1], so) : (T)0;
        }
        T s[R], lap[R];
        if (HASU && !NODAL && R <= 2 && z < z0) {
            // the plane below the chunk: its interpolants only (at 4 rows the branch costs 30
            // VGPRs and more than it saves)
            qd.prime(u, v);
        } else if constexpr (NODAL) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if constexpr (OP == MOP_GRAD) s[j] = cubic(uc[j], k.a, k.b, k.c);
                else if constexpr (OP == MOP_JVP) s[j] = fmaT(fmaT(k.c, uc[j], k.b), uc[j], k.a) * vc[j];
                else s[j] = (T)0;
            }
        } else if constexpr (HASU) {
            qd.push(u, v, k, s);
        }
        lp.push(HASV ? v : u, lap);
        if (emit && colok) {
            T zs = xs;
            if (MIRROR && p.rows) zs = (z - 1 == 0 || z - 1 == L.nz - 1) ? xs * (T)0.5 : xs;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (y0 + j >= L.ny) break;
                T ib = zs;
                if (MIRROR && p.rows) ib = edge_count(y0 + j, L.ny) ? zs * (T)0.5 : zs;
                const T o = add_stiffness(k, lap[j], HASU ? s[j] : (T)0);
                const T c = p.base ? eb[j] : (HASV ? vc[j] : uc[j]);
                T r;
                if constexpr (EPI == ME_OUT) r = (k.s0 != (T)0 ? fmaT(k.s0, c - e1[j], o) : o) * ib;
                else if constexpr (EPI == ME_SUB) r = c - o * ib;
                else if constexpr (EPI == ME_ADJ) {
                    r = (c - o * ib) + e1[j];
                    if (!MIRROR || (x < L.nx - 1 && y0 + j < L.ny - 1 && z - 1 < L.nz - 1)) sA += (double)qd.asum[j];
                    sB += (double)uc[j] * (double)(lap[j] * ib);
                } else if constexpr (EPI == ME_ADJK) {
                    r = o;
                    sB += (double)e0[j] * (double)(lap[j] * ib);
                }
                else if constexpr (EPI == ME_MU) r = fmaT(k.s0, e0[j], -o) * ib;
                else if constexpr (EPI == ME_BACK) r = fmaT(k.s0 / ib, e0[j], o);
                else r = fmaT(k.s1, c - e2[j], c) + k.s2 * e1[j] * (e0[j] - fmaT(k.s0, c, o) * ib);
                bstore(r, ro, vo[j + 1], so);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            uc[j] = u[j + 1];
            vc[j] = v[j + 1];
        }
    }
    if constexpr (ADJ) {
        for (int off = WAVE / 2; off > 0; off >>= 1) {
            sA += __shfl_down(sA, off, WAVE);
            sB += __shfl_down(sB, off, WAVE);
        }
        if (lane == 0) {
            if constexpr (EPI == ME_ADJ) {
                p.part[2 * wave] = p.fresh ? sA : p.part[2 * wave] + sA;
                p.part[2 * wave + 1] = p.fresh ? sB : p.part[2 * wave + 1] + sB;
            } else {
                p.part[wave] = p.fresh ? sB : p.part[wave] + sB;
            }
        }
    }
}

// rows per lane of ME_ADJ, whose pipeline holds two fields and two polynomials (4 rows: 236
// VGPRs in FP32, spills in FP64)
template <typename T>
constexpr int ADJ_ROWS = sizeof(T) == 4 ? 2 : 1;

}  // namespace

// How a grid is split: R rows per lane, G lane groups, pz planes per chunk.
struct Shape3 {
    int R, G, pz;
};

// G with the fewest waves per plane for R rows per lane; returns that number
static long long plane_waves(const Geom& g, int R, int* G)
{
    long long best = -1;
    for (int q = 1; q <= 4; ++q) {
        const int w = WAVE / q;
        const long long items = (long long)((g.n[0] + w - 3) / (w - 2)) * ((g.n[1] + R - 1) / R);
        const long long waves = (items + q - 1) / q;
        if (best < 0 || waves < best) {
            best = waves;
            *G = q;
        }
    }
    return best;
}

// Kernels bound by memory or latency (K v, nodal quadrature) and the adjoint: R given, the
// pz with the least time on the busiest SIMD, taken as max(3, waves per SIMD) pushes of
// pz + 2 planes: below three waves per SIMD the plane loads' latency shows.
static Shape3 shape_light(const Geom& g, int R)
{
    Shape3 p{R, 1, 1};
    const long long bw = plane_waves(g, R, &p.G), simds = 4ll * device_cus();
    double bt = -1.0;
    for (int q = 1; q <= std::min(g.n[2], 64); ++q) {
        const long long per = (bw * ((g.n[2] + q - 1) / q) + simds - 1) / simds;
        const double t = (double)std::max(3ll, per) * (q + 2);
        if (bt < 0.0 || t <= bt) {
            bt = t;
            p.pz = q;
        }
    }
    return p;
}

// Gauss quadrature, bound by issue: a wave pushes pz + 2 planes (with 2 rows and JVP the
// first one is cheaper), 2 rows per lane costing 0.6 (JVP 0.65) of 4, and a SIMD takes its
// waves in turn, idling a share of one wave's time (idle), a last round that is not full
// counting as part of one (part).  Fitted to 32 splits of 12 grids from 72 x 65 x 60 to 256
// x 200 x 180: 0.3% off the best on average, where 4 rows from 2^20 nodes and the rule
// above are 10% (FP32) to 20% (FP64) off.  us before and after: Allen-Cahn step 128^3 FP32
// 17.1 / 14.7, FP64 23.4 / 18.4; product 128^3 21.5 / 18.4, FP64 28.1 / 24.8; 72 x 65 x 60
// 7.4 / 6.5, FP64 9.8 / 7.5.  (Two fields in FP64 leave one wave per SIMD at 4 rows.)
static Shape3 shape_gauss(const Geom& g, bool jvp, bool f64)
{
    static const int planes[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16, 20, 24};
    const double idle = jvp ? (f64 ? 0.2 : 0.8) : (f64 ? 0.4 : 1.0), part = jvp == f64 ? 0.5 : 1.0;
    const double simds = 4.0 * device_cus();
    Shape3 best{2, 1, 1};
    double bt = -1.0;
    for (int R = 2; R <= (jvp && f64 ? 2 : 4); R += 2) {
        int G = 1;
        const long long bw = plane_waves(g, R, &G);
        const double push = R == 4 ? 1.0 : jvp ? 0.65 : 0.6, first = jvp && R == 2 ? 0.4 : 0.0;
        for (int q : planes) {
            if (q > g.n[2]) break;
            const double w = (double)(bw * ((g.n[2] + q - 1) / q)) / simds;
            const double t = push * (std::max(1.0, w + part * (std::ceil(w) - w)) + idle) * (q + 2 - first);
            if (bt < 0.0 || t < bt) {
                bt = t;
                best = {R, G, q};
            }
        }
    }
    return best;
}

template <typename T, int R>
bool launch_r(const Geom& g, const Shape3& shape, int op, int epi, const FreeEnergy& f, const March<T>& m,
              hipStream_t s, int* waves_out)
{
    ML3 L{};
    L.nx = g.n[0];
    L.ny = g.n[1];
    L.nz = g.n[2];
    L.G = shape.G;
    L.pz = shape.pz;
    L.W = WAVE / L.G;
    L.nstrips = (L.nx + L.W - 3) / (L.W - 2);
    const long long items = (long long)L.nstrips * ((L.ny + R - 1) / R);
    const long long wpc = (items + L.G - 1) / L.G, waves = wpc * ((L.nz + L.pz - 1) / L.pz);
    if (waves > (1ll << 30)) return false;
    if (epi == ME_ADJ || epi == ME_ADJK) {
        if (g.quad || (epi == ME_ADJ ? 2 : 1) * waves > m.part_max) return false;
        if (waves_out) *waves_out = (int)waves;
        if (!m.part) return true;
    }
    L.items = (int)items;
    L.wpc = (int)wpc;
    L.nwaves = (int)waves;
    L.bytes = (unsigned)((size_t)g.N * sizeof(T));
    const double detJ = std::pow(0.5 * g.h, 3), mm = std::pow(g.h, 3);
    const double w = m.nq * (g.quad ? mm : detJ);
    MC3<T> k{};
    if (op == MOP_GRAD) {
        k.a = (T)(w * f.a1); k.b = (T)(w * f.a2); k.c = (T)(w * f.a3);
    } else {
        k.a = (T)(w * f.b0); k.b = (T)(w * f.b1); k.c = (T)(w * f.b2);
    }
    const double kv = m.kv * (g.quad ? g.h : g.h / 12.0);
    k.kv = (T)kv;
    k.kl = (T)(kv - (double)k.kv);
    k.s0 = (T)m.s0;
    k.s1 = (T)m.s1;
    k.s2 = (T)m.s2;
    const FreeEnergy f1 = make_free_energy(f.fe, 1.0);
    k.g1 = (T)f1.a1;
    k.g2 = (T)f1.a2;
    k.g3 = (T)f1.a3;
    const unsigned blocks = (unsigned)((waves + 3) / 4);
#define M3Q(OP, EPI, MIR)                                                                  \
    do {                                                                                   \
        if (g.quad) k_march3d<T, R, OP, EPI, MIR, true><<<blocks, 256, 0, s>>>(m, L, k);   \
        else k_march3d<T, R, OP, EPI, MIR, false><<<blocks, 256, 0, s>>>(m, L, k);         \
    } while (0)
#define M3(OP, EPI)                                                                        \
    do {                                                                                   \
        if (g.bc) M3Q(OP, EPI, true); else M3Q(OP, EPI, false);                            \
    } while (0)
#define M3A(OP, EPI)                                                                       \
    do {                                                                                   \
        if (g.bc) k_march3d<T, R, OP, EPI, true, false><<<blocks, 256, 0, s>>>(m, L, k);   \
        else k_march3d<T, R, OP, EPI, false, false><<<blocks, 256, 0, s>>>(m, L, k);       \
    } while (0)
    if constexpr (R == ADJ_ROWS<T>) {
        if (op == MOP_JVP && epi == ME_ADJ) {
            M3A(MOP_JVP, ME_ADJ);
            return true;
        }
    }
    if constexpr (R == 1) return false;
    else switch (op * 8 + epi) {
        case MOP_STIFF * 8 + ME_ADJK: M3A(MOP_STIFF, ME_ADJK); return true;
        case MOP_GRAD * 8 + ME_OUT: M3(MOP_GRAD, ME_OUT); return true;
        case MOP_GRAD * 8 + ME_SUB: M3(MOP_GRAD, ME_SUB); return true;
        case MOP_GRAD * 8 + ME_MU: M3(MOP_GRAD, ME_MU); return true;
        case MOP_JVP * 8 + ME_OUT: M3(MOP_JVP, ME_OUT); return true;
        case MOP_JVP * 8 + ME_SUB: M3(MOP_JVP, ME_SUB); return true;
        case MOP_JVP * 8 + ME_BACK: M3(MOP_JVP, ME_BACK); return true;
        case MOP_JVP * 8 + ME_CHEB: M3(MOP_JVP, ME_CHEB); return true;
        case MOP_STIFF * 8 + ME_OUT: M3(MOP_STIFF, ME_OUT); return true;
        case MOP_STIFF * 8 + ME_SUB: M3(MOP_STIFF, ME_SUB); return true;
        case MOP_STIFF * 8 + ME_BACK: M3(MOP_STIFF, ME_BACK); return true;
        case MOP_STIFF * 8 + ME_CHEB: M3(MOP_STIFF, ME_CHEB); return true;
        default: return false;
    }
#undef M3A
#undef M3
#undef M3Q
}

template <typename T>
bool launch_march3d(const Geom& g, int op, int epi, const FreeEnergy& f, const March<T>& m, hipStream_t s,
                    int* waves_out)
{
    // 32-bit buffer offsets, and the Gauss-integrated mass has no marching form
    if (g.dim != 3 || g.cm || (size_t)g.N * sizeof(T) >= (size_t(1) << 31)) return false;
    if (epi == ME_ADJ)
        return launch_r<T, ADJ_ROWS<T>>(g, shape_light(g, ADJ_ROWS<T>), op, epi, f, m, s, waves_out);
    // rows per lane of the light kernels: 4 element rows' redundancy is 5/4 against 3/2 for
    // 2, which pays once the grid fills the chip; below about a million nodes more waves matter
    const bool f64 = sizeof(T) == 8, two = g.N < (1ll << 20) || (op == MOP_JVP && f64);
    const Shape3 p = op != MOP_STIFF && !g.quad ? shape_gauss(g, op == MOP_JVP, f64) : shape_light(g, two ? 2 : 4);
    return p.R == 4 ? launch_r<T, 4>(g, p, op, epi, f, m, s, waves_out)
                    : launch_r<T, 2>(g, p, op, epi, f, m, s, waves_out);
}

template bool launch_march3d<float>(const Geom&, int, int, const FreeEnergy&, const March<float>&, hipStream_t, int*);
template bool launch_march3d<double>(const Geom&, int, int, const FreeEnergy&, const March<double>&, hipStream_t, int*);

}  // namespace pfk
