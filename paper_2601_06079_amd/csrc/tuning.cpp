// tuning.cpp -- launch-shape choices for the fused 2-D explicit kernel:
// rows per wavefront (chunk length) and prefetch depth.  Defaults come from
// measurements on MI355X; pf_tune_set overrides them (the autotuner uses it).
#include <algorithm>
#include <atomic>
#include <cmath>

#include "api_internal.hpp"

namespace pfapi {
namespace {
std::atomic<int> g_rows_override{0};
std::atomic<int> g_depth_override{0};
std::atomic<int> g_fuse_override{0};
std::atomic<int> g_jvp3d_planes{0};
std::atomic<int> g_el_planes{0};
std::atomic<int> g_el_mg{0};
std::atomic<int> g_seam{0};
std::atomic<int> g_nn_group{0};
std::atomic<int> g_gs_reorth{0};
std::atomic<int> g_gg_stream{0};
std::atomic<int> g_jvp2d_stream{0};
}  // namespace

namespace {
// The plan for a grid of many rounds of waves.  Measured on MI355X: enough chunks for
// about four waves per SIMD hide latency, and stopping just below a whole number of waves
// per SIMD avoids a partly filled last round.  Chunks are never shorter than 8 rows.
// Longer chunks mean a grid of many rounds, where the measured best is 32 rows for single
// steps and 48 for fused ones.  (The launch splits each strip into balanced chunks, whose
// sizes differ by at most one row.)
// (coupled model: six, measured at 512^2..2048^2; its pipeline is VALU-bound and light on
// registers)
int full_rows(const pf_problem* p, int ks, int S)
{
    const int HK = (p->model == PF_ALLEN_CAHN ? 1 : 2) * ks;  // Cahn-Hilliard and coupled: 2 per step
    const long long nx = p->n[0], ny = p->n[1];
    const long long strips = (nx + (64 - 2 * HK) - 1) / (64 - 2 * HK);
    const long long waves = p->model == PF_COUPLED ? 6 : 4;
    long long nch = std::max<long long>(1, waves * S / strips);
    // periodic fused launches run on the seam-sharing kernel, which rounds the chunks
    // up to whole workgroups of 4: round down here so that the total stays in one round
    if (!p->bc && ks >= 2 && p->model != PF_COUPLED) nch = std::max<long long>(4, nch / 4 * 4);
    nch = std::min(nch, std::max<long long>(1, ny / 8));
    long long ty = (ny + nch - 1) / nch;
    const long long tmax = ks == 1 ? 32 : 48;
    if (ty > tmax) ty = tmax;
    return (int)std::max<long long>(ty, 1);
}

// Relative time per step of launches of ks fused steps with about ty rows per wave:
//   [ launch + pushes (r + 0.6) + memory ] / ks
// in units of one row through one stage.  pushes: the rows all stages of a wave take,
// warm-up included -- with the seams shared ks (ty + 2H) and the top wave's H ks (ks - 1)
// / 4, else whole groups of four rows less the stages' late starts; r: waves a SIMD takes
// in turn (a last round that is not full counts 0.3 of what it lacks); 0.6: one wave alone
// leaves a SIMD idle for three of eight cycles; launch and memory: fitted.  Against 24-step
// runs at 16 sizes from 96^2 to 4096^2, both models, types, boundaries and quadratures,
// 51 launch shapes each, its choice is 1.6% off the best on average (full_rows with four
// steps: 18%) and at most 2% slower than the latter.  us per run before and after: 128^2
// Allen-Cahn FP64 100 steps 187 / 145, 800 x 700 Cahn-Hilliard FP64 20 steps 123 / 86, 1200
// x 1300 Allen-Cahn FP32 37 steps 180 / 114, 1448^2 Cahn-Hilliard FP32 30 steps 227 / 187.
double plan_cost(const pf_problem* p, int ks, int ty, int S)
{
    const int H = p->model == PF_ALLEN_CAHN ? 1 : 2, HK = H * ks;
    const int nx = (int)p->n[0], ny = (int)p->n[1];
    const int strips = (nx + (64 - 2 * HK) - 1) / (64 - 2 * HK);
    const int nch = (ny + ty - 1) / ty;
    double waves = 0.0, pushes = 0.0;
    if (!p->bc) {
        // the seam kernel's own conditions (launch_seam)
        const int n4 = (nch + 3) / 4 * 4, rmin = ny / (n4 / 4), sh = H * (ks - 1);
        const int shortest = rmin - 3 * (rmin + sh) / 4;
        if (shortest >= (2 * HK + 3) / 4 * 4 + 4 - 2 * H && shortest >= 8) {
            waves = (double)strips * n4;
            pushes = ks * ((ny + n4 - 1) / n4 + 2 * H) + 0.25 * H * ks * (ks - 1);
        }
    }
    if (pushes == 0.0) {
        waves = (double)strips * nch;
        pushes = ks * (((ny + nch - 1) / nch + 2 * HK + 3) / 4 * 4) - H * ks * (ks - 1);
    }
    const bool lob = p->quad == PF_QUAD_LOBATTO;
    const double w = waves / S, full = std::ceil(w), r = std::max(1.0, w + 0.3 * (full - w));
    const double mb = 1e-6 * nx * ny * (p->dtype == PF_F64 ? 8 : 4);
    return ((lob ? 80.0 : 50.0) + pushes * (r + 0.6) + (lob ? 10.0 : 2.0) * mb) / ks;
}
// Rows of single steps (explicit steps one at a time; the coupled model): the pushes of a
// wave, in whole groups of four, times the waves a SIMD takes in turn (the last round as
// above; for the coupled model, whose waves are longer, as a full one), with the share a
// SIMD idles under one wave (fitted; smaller in FP64).  Single steps at the 16 sizes above:
// 1.5% off the best on average (full_rows: 11%); with nodal quadrature, a third of the
// arithmetic, it would be up to 10% slower than full_rows.  Coupled, us for 20 steps: 128^2
// 135 / 105, 500^2 173 / 149, 900^2 252 / 212, FP64 768^2 272 / 230, 1024^2 346 / 307.
int single_rows(const pf_problem* p, int S)
{
    const int H = p->model == PF_ALLEN_CAHN ? 1 : 2, outw = 64 - 2 * H;
    const int strips = ((int)p->n[0] + outw - 1) / outw, ny = (int)p->n[1];
    const bool cp = p->model == PF_COUPLED;
    if (p->quad == PF_QUAD_LOBATTO) return full_rows(p, 1, S);
    const double idle = p->dtype == PF_F64 ? (cp ? 0.7 : 0.3) : (cp ? 1.0 : 0.6), part = cp ? 1.0 : 0.3;
    auto cost = [&](int ty) {
        const int nch = (ny + ty - 1) / ty;
        const double w = (double)strips * nch / S, r = std::max(1.0, w + part * (std::ceil(w) - w));
        return (((ny + nch - 1) / nch + 2 * H + 3) / 4 * 4) * (r + idle);
    };
    const int full = full_rows(p, 1, S);
    int best = full;
    double c = 0.97 * cost(full);
    for (int len = (2 * H + 2 + 3) / 4 * 4; len <= 36; len += 4) {
        const int ty = std::min(len - 2 * H, ny);
        const double ct = cost(ty);
        if (ct < c) {
            c = ct;
            best = ty;
        }
        if (ty == ny) break;
    }
    return best;
}

}  // namespace

int stream2d_rows(const pf_problem* p, int cus)
{
    const int ov = g_rows_override.load();
    return ov > 0 ? ov : single_rows(p, 4 * (cus > 0 ? cus : 256));
}

Stream2DPlan stream2d_plan(const pf_problem* p, int cus, int64_t nsteps)
{
    const int S = 4 * (cus > 0 ? cus : 256);  // SIMDs
    const int rows = g_rows_override.load(), fuse = g_fuse_override.load();
    Stream2DPlan q;
    q.ty[1] = rows > 0 ? rows : single_rows(p, S);
    if (fuse == 0 && nsteps <= 2) return q;
    // The plan of grids of many rounds.  Four fused steps are fastest there for
    // Allen-Cahn; Cahn-Hilliard on the seam-sharing kernel is fastest with three from
    // 2048^2 (7.7 us/step; two: 8.1, and 10% slower than three at 8192^2); with nodal
    // quadrature the step is a third of the arithmetic and four are fastest (2048^2: 3.9
    // us/step; three 4.1, two 4.9).
    const int kf = p->model == PF_CAHN_HILLIARD && p->quad == PF_QUAD_GAUSS && p->n[0] * p->n[1] >= (1ll << 22) ? 3 : 4;
    q.fixed = fuse > 0;
    static const int cand[] = {2, 4, 6, 8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 36, 40, 48};
    const int tf = full_rows(p, kf, S);
    const double cf = plan_cost(p, kf, tf, S);
    double best = 0.0;
    int kb = kf;
    for (int k = 2; k <= 4; ++k) {
        q.ty[k] = full_rows(p, k, S);
        double c = plan_cost(p, k, q.ty[k], S);
        for (int t : cand) {
            if (t > p->n[1]) break;
            const double ct = plan_cost(p, k, t, S);
            if (ct < c) {
                c = ct;
                q.ty[k] = t;
            }
        }
        if (best == 0.0 || c < best) {
            best = c;
            kb = k;
        }
    }
    // (that plan keeps its place where the estimate gains less than 3%)
    if (best > 0.97 * cf) {
        kb = kf;
        q.ty[kf] = tf;
    }
    q.ks = fuse > 0 ? std::min(fuse, 4) : kb;
    if (rows > 0) q.ty[2] = q.ty[3] = q.ty[4] = rows;
    return q;
}

int stream2d_depth(const pf_problem* p)
{
    (void)p;
    const int ov = g_depth_override.load();
    return ov > 0 ? ov : 4;
}

}  // namespace pfapi

namespace pfk {
int tune_jvp3d_planes() { return pfapi::g_jvp3d_planes.load(); }
int tune_el_planes() { return pfapi::g_el_planes.load(); }
int tune_el_mg() { return pfapi::g_el_mg.load(); }
int tune_stream2d_seam() { return pfapi::g_seam.load(); }
int tune_nn_group() { return pfapi::g_nn_group.load(); }
int tune_gs_reorth() { return pfapi::g_gs_reorth.load(); }
int tune_gg_stream() { return pfapi::g_gg_stream.load(); }
int tune_jvp2d_stream() { return pfapi::g_jvp2d_stream.load(); }
int tune_stream2d_rows() { return pfapi::g_rows_override.load(); }
}  // namespace pfk

using namespace pfapi;
extern "C" {
int pf_tune_set(int key, int value)
{
    if (value < 0) return fail(PF_EINVAL, "tuning value must be >= 0");
    if (key == PF_TUNE_STREAM2D_ROWS)
        g_rows_override.store(value);
    else if (key == PF_TUNE_STREAM2D_DEPTH)
        g_depth_override.store(value);
    else if (key == PF_TUNE_STREAM2D_FUSE)
        g_fuse_override.store(value);
    else if (key == PF_TUNE_JVP3D_PLANES)
        g_jvp3d_planes.store(value);
    else if (key == PF_TUNE_EL_PLANES)
        g_el_planes.store(value);
    else if (key == PF_TUNE_EL_MG)
        g_el_mg.store(value);
    else if (key == PF_TUNE_STREAM2D_SEAM)
        g_seam.store(value);
    else if (key == PF_TUNE_NN_GROUP)
        g_nn_group.store(value);
    else if (key == PF_TUNE_GS_REORTH)
        g_gs_reorth.store(value);
    else if (key == PF_TUNE_GG_STREAM)
        g_gg_stream.store(value);
    else if (key == PF_TUNE_JVP2D_STREAM)
        g_jvp2d_stream.store(value);
    else
        return fail(PF_EINVAL, "unknown tuning key %d", key);
    return PF_OK;
}
int pf_launch_shape(const pf_ctx* ctx, const pf_problem* p, int* ks, int* ty, int* depth)
{
    return guarded("pf_launch_shape", [&]() -> int {
        if (int rc = check_ctx(ctx)) return rc;
        if (int rc = validate(p)) return rc;
        if (!ks || !ty || !depth) return fail(PF_EINVAL, "NULL output pointer");
        const Stream2DPlan q = stream2d_plan(p, ctx->cus, INT64_MAX);  // of a run of many steps
        *ks = q.ks;
        *ty = q.ty[q.ks];
        *depth = stream2d_depth(p);
        return PF_OK;
    });
}

int pf_tune_get(int key, int* value)
{
    if (!value) return fail(PF_EINVAL, "value is NULL");
    if (key == PF_TUNE_STREAM2D_ROWS)
        *value = g_rows_override.load();
    else if (key == PF_TUNE_STREAM2D_DEPTH)
        *value = g_depth_override.load();
    else if (key == PF_TUNE_STREAM2D_FUSE)
        *value = g_fuse_override.load();
    else if (key == PF_TUNE_JVP3D_PLANES)
        *value = g_jvp3d_planes.load();
    else if (key == PF_TUNE_EL_PLANES)
        *value = g_el_planes.load();
    else if (key == PF_TUNE_EL_MG)
        *value = g_el_mg.load();
    else if (key == PF_TUNE_STREAM2D_SEAM)
        *value = g_seam.load();
    else if (key == PF_TUNE_NN_GROUP)
        *value = g_nn_group.load();
    else if (key == PF_TUNE_GS_REORTH)
        *value = g_gs_reorth.load();
    else if (key == PF_TUNE_GG_STREAM)
        *value = g_gg_stream.load();
    else if (key == PF_TUNE_JVP2D_STREAM)
        *value = g_jvp2d_stream.load();
    else
        return fail(PF_EINVAL, "unknown tuning key %d", key);
    return PF_OK;
}
}
