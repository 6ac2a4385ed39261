// k_cheb2d.hip -- several products of the polynomial preconditioner in one pass (2-D).
//
// A step of the Chebyshev semi-iteration (ME_CHEB of march.hpp) reads five fields and
// writes one for about 60 operations a node: 20 us at 2048^2 FP32, bound by memory.  Here
// a wave marches S steps at once, each stage taking the rows of the one before as they
// are formed (Dl rows behind it: one stencil deep, two for MOP_SCHUR), so a pass reads
// five fields and writes two for S products.  The first pass forms its iterate pinv b
// while it reads (it reads no iterate), the last one ends with the product w = J z itself.
// 2048^2 FP32: 2, 3, 4 steps 20 / 30 / 37 us a pass, now bound by issue (44 operations a
// node and step, and 2 S Dl rows and lanes computed twice, which is why S stays at 4
// stencils).
#include <algorithm>
#include <cmath>

#include "march2d.hpp"

namespace pfk {
namespace {

template <typename T>
struct ChebP {
    const T *u, *b, *pinv;   // the state, the right-hand side, the diagonal preconditioner
    const T *z, *zm;         // the iterate and the one before (null: pinv b and 0)
    T *out, *out2;           // the last stage's result; the iterate before it (null: not kept)
    T s1[CHEB_MAXS], s2[CHEB_MAXS];
    int product;             // the last stage is w = J z
};

// f''(u) at the Gauss points of element row (r-1, r) as rows r of u are pushed (nodal: at
// the nodes of row r - 1), |J| folded in: it is the same for every stage, which takes it
// from a ring (17 of a stage's 60 operations)
template <typename T, bool NODAL>
struct Curv2 {
    static constexpr int NW = NODAL ? 1 : 4;
    T xl = 0, xr = 0;
    __device__ __forceinline__ void push(T u, const MC2<T>& k, T* w)
    {
        auto F = [&](T q) { return fmaT(fmaT(k.c, q, k.b), q, k.a); };
        if constexpr (NODAL) {
            w[0] = F(xl);
            xl = u;
        } else {
            const T gp = (T)GP, gm = (T)GM;
            const T du = from_right(u) - u;
            const T l = fmaT(gm, du, u), r = fmaT(gp, du, u);
            const T e0 = l - xl, e1 = r - xr;
            w[0] = F(fmaT(gm, e0, xl));
            w[1] = F(fmaT(gp, e0, xl));
            w[2] = F(fmaT(gm, e1, xr));
            w[3] = F(fmaT(gp, e1, xr));
            xl = l;
            xr = r;
        }
    }
};

// quadrature sum of node row r - 1 as rows r of v are pushed, w from Curv2
template <typename T, bool NODAL>
struct QuadV2 {
    T xl = 0, xr = 0, guL = 0, guR = 0;
    __device__ __forceinline__ T push(T v, const T* w)
    {
        if constexpr (NODAL) {
            const T r = w[0] * xl;
            xl = v;
            return r;
        } else {
            const T gp = (T)GP, gm = (T)GM;
            const T dv = from_right(v) - v;
            const T l = fmaT(gm, dv, v), r = fmaT(gp, dv, v);
            const T e0 = l - xl, e1 = r - xr;
            const T PL0 = w[0] * fmaT(gm, e0, xl), PL1 = w[1] * fmaT(gp, e0, xl);
            const T PR0 = w[2] * fmaT(gm, e1, xr), PR1 = w[3] * fmaT(gp, e1, xr);
            const T dL = PL0 - PL1, dR = PR0 - PR1;
            const T HL = guL + fmaT(gp, dL, PL1), HR = guR + fmaT(gp, dR, PR1);
            guL = fmaT(gm, dL, PL1);
            guR = fmaT(gm, dR, PR1);
            const T dH = HL - HR;
            xl = l;
            xr = r;
            return fmaT(gp, dH, HR) + from_left(fmaT(gm, dH, HR));
        }
    }
};

template <typename T, int OP, int S, bool MIRROR, bool NODAL>
__global__ __launch_bounds__(256) void k_cheb2d(ChebP<T> p, int nx, int ny, int nstrips, int nwaves, int ty,
                                                unsigned bytes, MC2<T> k)
{
    constexpr int DL = OP == MOP_SCHUR ? 2 : 1;  // rows a stage lags behind its input
    constexpr int H = S * DL;
    constexpr int OUTW = WAVE - 2 * H;
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
    const T xs = MIRROR && edge_count(x, nx) ? (T)0.5 : (T)1;
    const int iters = (y1 - y0) + 2 * H;  // rows y0 - H .. y1 + H - 1
    const int rowb = nx * (int)sizeof(T);
    const int vx = x * (int)sizeof(T);
    const bool first = p.z == nullptr;
    const auto ru = make_rsrc(p.u, bytes);
    const auto rb = make_rsrc(p.b, bytes);
    const auto rp = make_rsrc(p.pinv, bytes);
    const auto rz = make_rsrc(first ? p.b : p.z, bytes);
    const auto rm = make_rsrc(first ? p.b : p.zm, bytes);
    const auto ro = make_rsrc(p.out, bytes);
    const auto ro2 = make_rsrc(p.out2 ? p.out2 : p.out, bytes);
    // rows read lie in [-H, ny + H - 1] and are wrapped or reflected once (the launcher
    // keeps ny > H).  Reflected rows and columns of every input make each stage's halo the
    // reflection of its inner rows, so only rows 0 and ny - 1 themselves are halved.
    auto row_off = [&](int t) {
        int r = min(y0 - H + t, y1 + H - 1);  // past the chunk the last row is read again (a cache hit)
        if constexpr (MIRROR) {
            r = r < 0 ? -r : (r >= ny ? 2 * (ny - 1) - r : r);
        } else {
            r = r < 0 ? r + ny : (r >= ny ? r - ny : r);
        }
        return r * rowb;
    };
    T fu[MPF], fb[MPF], fp[MPF], fz[MPF], fm[MPF];
    auto fetch = [&](int t, int i) {
        const int off = row_off(t);
        fu[i] = bload<T>(ru, vx, off);
        fb[i] = bload<T>(rb, vx, off);
        fp[i] = bload<T>(rp, vx, off);
        fz[i] = first ? (T)0 : bload<T>(rz, vx, off);
        fm[i] = first ? (T)0 : bload<T>(rm, vx, off);
    };
#pragma unroll
    for (int i = 0; i < MPF; ++i) fetch(i, i);
    constexpr int NW = Curv2<T, NODAL>::NW, WD = (S - 1) * DL;
    Curv2<T, NODAL> cv;
    QuadV2<T, NODAL> qd[S];
    Lap2<T, NODAL> lp[S], lw[S];
    // rows behind the newest one: [d] holds row R - d (inputs), the stage's argument and
    // the iterate before it
    T wr[WD + 1][NW] = {}, br[H + 1] = {}, pr[H + 1] = {}, mr[DL + 1] = {};
    T cr[S][DL + 1] = {}, dr[S][DL + 1] = {};
    for (int t0 = 0; t0 < iters; t0 += MPF) {
#pragma unroll
        for (int i = 0; i < MPF; ++i) {
            const int t = t0 + i;
#pragma unroll
            for (int d = H; d > 0; --d) {
                br[d] = br[d - 1];
                pr[d] = pr[d - 1];
            }
#pragma unroll
            for (int d = DL; d > 0; --d) mr[d] = mr[d - 1];
#pragma unroll
            for (int d = WD; d > 0; --d)
#pragma unroll
                for (int n = 0; n < NW; ++n) wr[d][n] = wr[d - 1][n];
            cv.push(fu[i], k, wr[0]);
            br[0] = fb[i];
            pr[0] = fp[i];
            mr[0] = fm[i];
            T zin = first ? fp[i] * fb[i] : fz[i];
            fetch(t + MPF, i);
            T zb = mr[DL];  // the iterate before the stage's argument, at the stage's output row
            T c = 0;
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const T s = qd[j].push(zin, wr[j * DL]);
                T o = fmaT(k.kv, lp[j].push(zin), s);
                if constexpr (OP == MOP_SCHUR) o = k.kw * lw[j].push(o);
#pragma unroll
                for (int d = DL; d > 0; --d) {
                    cr[j][d] = cr[j][d - 1];
                    dr[j][d] = dr[j][d - 1];
                }
                cr[j][0] = zin;
                c = cr[j][DL];
                const int yo = y0 - H + t - (j + 1) * DL;
                const T ib = MIRROR && (yo == 0 || yo == ny - 1) ? xs * (T)0.5 : xs;
                const T jz = fmaT(k.s0, c, o) * ib;
                const T r = fmaT(p.s1[j], c - zb, c) + p.s2[j] * pr[(j + 1) * DL] * (br[(j + 1) * DL] - jz);
                zin = j == S - 1 && p.product ? jz : r;
                // the next stage's output row lies DL behind this one's
                dr[j][0] = c;
                zb = dr[j][DL];
            }
            if (t >= 2 * H && t < iters && out_lane) {
                const int off = (y0 - 2 * H + t) * rowb;
                bstore(zin, ro, vx, off);
                if (p.out2) bstore(c, ro2, vx, off);
            }
        }
    }
}

// Rows per wave.  A wave marches its rows and 2 H more, in whole groups of MPF, and the
// kernel is bound by issue: its time is that times the waves a SIMD takes in turn, of
// which it needs two to stay busy (one wave alone counts as 1.6).  Whole numbers of waves
// per SIMD matter: 2048^2 FP32 (three steps a pass, 36 strips) 38 rows, 1.9 waves: 4.37 ms
// a Newton step; 19 rows, 3.97 waves: 4.53; 54 rows, 1.3 waves: 4.91; 78 rows, 0.95: 5.10.
int cheb_rows(int ny, int nstrips, int H)
{
    const double simds = 4.0 * device_cus();
    int best = 1;
    double cost = 0.0;
    for (int len = (2 * H + 4 + MPF - 1) / MPF * MPF; len <= 128; len += MPF) {
        const int ty = std::min(len - 2 * H, ny);
        const double w = (double)nstrips * ((ny + ty - 1) / ty) / simds;
        const double c = len * std::max(1.6, std::ceil(w));
        if (cost == 0.0 || c < cost) {
            cost = c;
            best = ty;
        }
        if (ty == ny) break;
    }
    return best;
}

}  // namespace

template <typename T>
bool launch_cheb2d(const Geom& g, int op, const FreeEnergy& f, const March<T>& m, const ChebGroup<T>& q, int S,
                   hipStream_t s)
{
    const int dl = op == MOP_SCHUR ? 2 : 1, H = S * dl;
    // 32-bit buffer offsets; one reflection or wrap of a halo row
    if (g.dim != 2 || g.cm || (size_t)g.N * sizeof(T) >= (size_t(1) << 31)) return false;
    const int nx = g.n[0], ny = g.n[1], outw = WAVE - 2 * H;
    if (ny <= H || S < 1 || H > 4) return false;
    const int nstrips = (nx + outw - 1) / outw;
    const int tov = tune_stream2d_rows();
    const int ty = tov > 0 ? std::min(tov, ny) : cheb_rows(ny, nstrips, H);
    const long long nwaves = (long long)nstrips * ((ny + ty - 1) / ty);
    if (nwaves > (1ll << 30)) return false;
    MC2<T> k = march2_coef<T>(g, op, f, m.nq, m.kv, m.kw);
    k.s0 = (T)m.s0;
    ChebP<T> p{m.u, m.p0, m.p1, q.z, q.zm, m.out, q.out2, {}, {}, q.product};
    for (int j = 0; j < S; ++j) {
        p.s1[j] = (T)q.s1[j];
        p.s2[j] = (T)q.s2[j];
    }
    const unsigned blocks = (unsigned)((nwaves + 3) / 4), bytes = (unsigned)((size_t)g.N * sizeof(T));
#define CH2(OP, SS, MIR, NOD) \
    k_cheb2d<T, OP, SS, MIR, NOD><<<blocks, 256, 0, s>>>(p, nx, ny, nstrips, (int)nwaves, ty, bytes, k)
#define CH2S(OP, SS)                                           \
    do {                                                       \
        if (g.bc && g.quad) CH2(OP, SS, true, true);           \
        else if (g.bc) CH2(OP, SS, true, false);               \
        else if (g.quad) CH2(OP, SS, false, true);             \
        else CH2(OP, SS, false, false);                        \
        return true;                                           \
    } while (0)
    if (op == MOP_SCHUR) {
        if (S == 1) CH2S(MOP_SCHUR, 1);
        CH2S(MOP_SCHUR, 2);
    }
    if (S == 1) CH2S(MOP_JVP, 1);
    if (S == 2) CH2S(MOP_JVP, 2);
    if (S == 3) CH2S(MOP_JVP, 3);
    CH2S(MOP_JVP, 4);
#undef CH2S
#undef CH2
}

template bool launch_cheb2d<float>(const Geom&, int, const FreeEnergy&, const March<float>&, const ChebGroup<float>&,
                                   int, hipStream_t);
template bool launch_cheb2d<double>(const Geom&, int, const FreeEnergy&, const March<double>&,
                                    const ChebGroup<double>&, int, hipStream_t);

}  // namespace pfk
