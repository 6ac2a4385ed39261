// k_march2d.hip -- node operators of the 2-D weak forms, streamed row by row.
//
// The strip-and-row layout of k_jvp2d.hip (one 64-lane wave per strip of columns and
// chunk of rows, x-neighbours by DPP, rows in registers, four rows in flight) for the
// operators and epilogues of march.hpp: each element row's Gauss points are evaluated
// once, where the node-centric kernels evaluate each four times.  The pointwise inputs
// of an epilogue are prefetched with the rows.  MOP_SCHUR chains two stencils (two halo
// lanes per side): the inner product never reaches memory.
#include <algorithm>
#include <cmath>

#include "march2d.hpp"

namespace pfk {
namespace {

template <typename T, int OP, int EPI, bool MIRROR, bool NODAL>
__global__ __launch_bounds__(256) void k_march2d(March<T> p, int nx, int ny, int nstrips, int nwaves, int ty,
                                                 unsigned bytes, MC2<T> k)
{
    constexpr int H = OP == MOP_SCHUR ? 2 : 1;
    constexpr int OUTW = WAVE - 2 * H;
    constexpr bool HASU = OP != MOP_STIFF, HASV = OP != MOP_GRAD || EPI == ME_CHRES;
    constexpr bool ADJ = EPI == ME_ADJ || EPI == ME_ADJK;
    constexpr bool USE0 = EPI == ME_MU || EPI == ME_BACK || EPI == ME_CHEB || EPI == ME_ADJK;
    constexpr bool USE1 = EPI == ME_CHEB || EPI == ME_OUT || EPI == ME_CHRES || EPI == ME_ADJ, USE2 = EPI == ME_CHEB;
    const int wid = uniform_wave();
    if (wid >= nwaves) return;  // uniform per wave
    const int strip = wid % nstrips, chunk = wid / nstrips;
    const int y0 = chunk * ty, y1 = min(ny, y0 + ty);
    const int lane = threadIdx.x & (WAVE - 1);
    const int xl = strip * OUTW - H + lane;
    int x;
    if constexpr (MIRROR) {
        x = reflect(xl, nx);
    } else {
        x = xl % nx;
        if (x < 0) x += nx;
    }
    const bool out_lane = lane >= H && lane < WAVE - H && xl < nx;
    T xs = (T)1;
    if (MIRROR && p.rows) xs = edge_count(x, nx) ? (T)0.5 : (T)1;
    const int iters = (y1 - y0) + 2 * H;  // rows y0 - H .. y1 + H - 1
    const int rowb = nx * (int)sizeof(T);
    const int vx = x * (int)sizeof(T);
    const auto ru = make_rsrc(HASU ? p.u : p.v, bytes);
    const auto rv = make_rsrc(HASV ? p.v : p.u, bytes);
    const auto ro = make_rsrc(p.out, bytes);
    const auto ro2 = make_rsrc(EPI == ME_CHRES ? p.out2 : p.out, bytes);
    const auto rb = make_rsrc(p.base ? p.base : p.out, bytes);
    const auto r0 = make_rsrc(p.p0 ? p.p0 : p.out, bytes);
    const auto r1 = make_rsrc(p.p1 ? p.p1 : p.out, bytes);
    const auto r2 = make_rsrc(p.p2 ? p.p2 : p.out, bytes);
    // rows read lie in [-H, ny + H - 1] and are wrapped or reflected once (the launcher
    // keeps ny >= 2 H)
    auto row_of = [&](int t) {
        int r = min(y0 - H + t, y1 + H - 1);  // past the chunk the last row is read again (a cache hit)
        if constexpr (MIRROR) {
            r = r < 0 ? -r : (r >= ny ? 2 * (ny - 1) - r : r);
        } else {
            r = r < 0 ? r + ny : (r >= ny ? r - ny : r);
        }
        return r;
    };
    auto row_off = [&](int t) { return row_of(t) * rowb; };
    const T vf = ADJ && MIRROR && p.scale && edge_count(x, nx) ? (T)2 : (T)1;  // 2^b of the lane's column
    double sA = 0.0, sB = 0.0;
    // output row of iteration t: y0 - 2 H + t
    auto out_off = [&](int t) { return min(max(y0 - 2 * H + t, y0), y1 - 1) * rowb; };
    T fu[MPF], fv[MPF], fb[MPF], f0[MPF], f1[MPF], f2[MPF];
    auto fetch = [&](int t, int i) {
        const int off = row_off(t);
        fu[i] = HASU ? bload<T>(ru, vx, off) : (T)0;
        fv[i] = HASV ? bload<T>(rv, vx, off) : (T)0;
        const int oo = out_off(t);
        fb[i] = p.base ? bload<T>(rb, vx, oo) : (T)0;
        f0[i] = USE0 ? bload<T>(r0, vx, oo) : (T)0;
        f1[i] = USE1 && p.p1 ? bload<T>(r1, vx, oo) : (T)0;
        f2[i] = USE2 && p.p2 ? bload<T>(r2, vx, oo) : (T)0;
    };
#pragma unroll
    for (int i = 0; i < MPF; ++i) fetch(i, i);
    constexpr bool VARG = OP != MOP_GRAD;  // the operator's argument is v
    Quad2<T, VARG, NODAL, EPI == ME_ADJ> qd;
    Lap2<T, NODAL> lp, lw;
    T c1 = 0, c2 = 0;  // the operator's argument at rows r-1, r-2
    T u1 = 0;
    // whole groups of MPF rows: the pushes past the chunk compute rows nobody stores
    for (int t0 = 0; t0 < iters; t0 += MPF) {
#pragma unroll
        for (int i = 0; i < MPF; ++i) {
            const int t = t0 + i;
            const T u = fu[i], eb = fb[i], e0 = f0[i], e1 = f1[i], e2 = f2[i];
            T v = fv[i];
            if constexpr (ADJ && MIRROR) {
                const int r = row_of(t);
                if (p.scale) v *= (r == 0 || r == ny - 1) ? vf * (T)2 : vf;
            }
            const T ucen = u1;  // u at the output row (H = 1)
            u1 = u;
            fetch(t + MPF, i);
            T s = 0;
            if constexpr (HASU) s = qd.push(u, v, k);
            const T lap = lp.push(VARG ? v : u);
            const T v1 = lw.v1;  // ME_CHRES: v at the output row
            T lapv = 0;
            if constexpr (EPI == ME_CHRES) lapv = lw.push(v);
            T o = add_stiffness(k, lap, s);
            if constexpr (OP == MOP_SCHUR) o = k.kw * lw.push(o);
            const T cc = H == 2 ? c2 : c1;
            c2 = c1;
            c1 = VARG ? v : u;
            if (t >= 2 * H && t < iters && out_lane) {
                const int yo = y0 - 2 * H + t;
                T ib = xs;
                if (MIRROR && p.rows) ib = (yo == 0 || yo == ny - 1) ? xs * (T)0.5 : xs;
                const T c = p.base ? eb : cc;
                T r;
                if constexpr (EPI == ME_OUT) r = (k.s0 != (T)0 ? fmaT(k.s0, c - e1, o) : o) * ib;
                else if constexpr (EPI == ME_SUB) r = c - o * ib;
                else if constexpr (EPI == ME_ADJ) {
                    r = (c - o * ib) + e1;
                    if (!MIRROR || (x < nx - 1 && yo < ny - 1)) sA += (double)qd.asum;
                    sB += (double)ucen * (double)(lap * ib);
                } else if constexpr (EPI == ME_ADJK) {
                    r = o;
                    sB += (double)e0 * (double)(lap * ib);
                }
                else if constexpr (EPI == ME_MU) r = fmaT(k.s0, e0, -o) * ib;
                else if constexpr (EPI == ME_CHRES) {
                    bstore(fmaT(k.s0, v1, -o) * ib, ro2, vx, yo * rowb);
                    r = (k.s1 != (T)0 ? fmaT(k.kw, lapv, k.s1 * (c - e1)) : k.kw * lapv) * ib;
                } else if constexpr (EPI == ME_BACK) r = fmaT(k.s0 / ib, e0, o);
                else r = fmaT(k.s1, c - e2, c) + k.s2 * e1 * (e0 - fmaT(k.s0, c, o) * ib);
                bstore(r, ro, vx, yo * rowb);
            }
        }
    }
    if constexpr (ADJ) {
        for (int off = WAVE / 2; off > 0; off >>= 1) {
            sA += __shfl_down(sA, off, WAVE);
            sB += __shfl_down(sB, off, WAVE);
        }
        if (lane == 0) {
            if constexpr (EPI == ME_ADJ) {
                p.part[2 * wid] = p.fresh ? sA : p.part[2 * wid] + sA;
                p.part[2 * wid + 1] = p.fresh ? sB : p.part[2 * wid + 1] + sB;
            } else {
                p.part[wid] = p.fresh ? sB : p.part[wid] + sB;
            }
        }
    }
}

}  // namespace

template <typename T>
bool launch_march2d(const Geom& g, int op, int epi, const FreeEnergy& f, const March<T>& m, hipStream_t s,
                    int* waves_out)
{
    // 32-bit buffer offsets; the Gauss-integrated mass has no streaming form
    if (g.dim != 2 || g.cm || (size_t)g.N * sizeof(T) >= (size_t(1) << 31)) return false;
    const int H = op == MOP_SCHUR ? 2 : 1;
    const int nx = g.n[0], ny = g.n[1], outw = WAVE - 2 * H;
    if (ny < 2 * H) return false;
    const int nstrips = (nx + outw - 1) / outw;
    // (the adjoint's waves are the same in every call of a trajectory, whose sums they keep)
    const int tov = epi < ME_ADJ ? tune_stream2d_rows() : 0;
    const int ty = tov > 0 ? std::min(tov, ny) : pass_rows(ny, nstrips, H, device_cus(), epi < ME_ADJ);
    const long long nwaves = (long long)nstrips * ((ny + ty - 1) / ty);
    if (nwaves > (1ll << 30)) return false;
    if (epi == ME_ADJ || epi == ME_ADJK) {
        if (g.quad || (epi == ME_ADJ ? 2 : 1) * nwaves > m.part_max) return false;
        if (waves_out) *waves_out = (int)nwaves;
        if (!m.part) return true;
    }
    MC2<T> k = march2_coef<T>(g, op, f, m.nq, m.kv, m.kw);
    k.s0 = (T)m.s0;
    k.s1 = (T)m.s1;
    k.s2 = (T)m.s2;
    const FreeEnergy f1 = make_free_energy(f.fe, 1.0);
    k.g1 = (T)f1.a1;
    k.g2 = (T)f1.a2;
    k.g3 = (T)f1.a3;
    const unsigned blocks = (unsigned)((nwaves + 3) / 4), bytes = (unsigned)((size_t)g.N * sizeof(T));
#define M2Q(OP, EPI, MIR)                                                                                        \
    do {                                                                                                         \
        if (g.quad)                                                                                              \
            k_march2d<T, OP, EPI, MIR, true><<<blocks, 256, 0, s>>>(m, nx, ny, nstrips, (int)nwaves, ty, bytes, k);  \
        else                                                                                                     \
            k_march2d<T, OP, EPI, MIR, false><<<blocks, 256, 0, s>>>(m, nx, ny, nstrips, (int)nwaves, ty, bytes, k); \
    } while (0)
#define M2(OP, EPI)                                                                                              \
    do {                                                                                                         \
        if (g.bc) M2Q(OP, EPI, true); else M2Q(OP, EPI, false);                                                  \
    } while (0)
    // (the adjoint of a step: Gauss quadrature only)
#define M2A(OP, EPI)                                                                                             \
    do {                                                                                                         \
        if (g.bc)                                                                                                \
            k_march2d<T, OP, EPI, true, false><<<blocks, 256, 0, s>>>(m, nx, ny, nstrips, (int)nwaves, ty, bytes, k);  \
        else                                                                                                     \
            k_march2d<T, OP, EPI, false, false><<<blocks, 256, 0, s>>>(m, nx, ny, nstrips, (int)nwaves, ty, bytes, k); \
    } while (0)
    switch (op * 8 + epi) {
        case MOP_GRAD * 8 + ME_OUT: M2(MOP_GRAD, ME_OUT); return true;
        case MOP_GRAD * 8 + ME_CHRES: M2(MOP_GRAD, ME_CHRES); return true;
        case MOP_JVP * 8 + ME_OUT: M2(MOP_JVP, ME_OUT); return true;
        case MOP_JVP * 8 + ME_SUB: M2(MOP_JVP, ME_SUB); return true;
        case MOP_JVP * 8 + ME_BACK: M2(MOP_JVP, ME_BACK); return true;
        case MOP_JVP * 8 + ME_CHEB: M2(MOP_JVP, ME_CHEB); return true;
        case MOP_JVP * 8 + ME_ADJ: M2A(MOP_JVP, ME_ADJ); return true;
        case MOP_STIFF * 8 + ME_ADJK: M2A(MOP_STIFF, ME_ADJK); return true;
        case MOP_STIFF * 8 + ME_OUT: M2(MOP_STIFF, ME_OUT); return true;
        case MOP_STIFF * 8 + ME_SUB: M2(MOP_STIFF, ME_SUB); return true;
        case MOP_STIFF * 8 + ME_BACK: M2(MOP_STIFF, ME_BACK); return true;
        case MOP_STIFF * 8 + ME_CHEB: M2(MOP_STIFF, ME_CHEB); return true;
        case MOP_SCHUR * 8 + ME_OUT: M2(MOP_SCHUR, ME_OUT); return true;
        case MOP_SCHUR * 8 + ME_CHEB: M2(MOP_SCHUR, ME_CHEB); return true;
        default: return false;
    }
#undef M2A
#undef M2
#undef M2Q
}

template bool launch_march2d<float>(const Geom&, int, int, const FreeEnergy&, const March<float>&, hipStream_t, int*);
template bool launch_march2d<double>(const Geom&, int, int, const FreeEnergy&, const March<double>&, hipStream_t, int*);

}  // namespace pfk
