// api_internal.hpp -- helpers shared by the C-ABI translation units.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <exception>
#include <new>

#include "../../include/pf.h"
#include "ctx.hpp"
#include "kernels.hpp"

namespace pfapi {

int fail(int status, const char* fmt, ...);
int check_launch(const char* what);
int validate(const pf_problem* p);
int check_ptr(const void* ptr, const pf_problem* p, const char* name);
pfk::Geom geom_of(const pf_problem* p);
long long ndof(const pf_problem* p);
size_t elem_size(const pf_problem* p);
int grain_implicit_ok(const pf_problem* p);
// the explicit trajectory calls: model, mass, dt, step count, field size
int explicit_trajectory_ok(const pf_problem* p, double dt, int64_t nsteps);

// Runs an entry point's body; a C++ exception (a host allocation that failed, an
// internal error) becomes PF_EDEVICE with a message instead of crossing the ABI.
template <class F>
int guarded(const char* name, F&& body) noexcept
{
    try {
        return body();
    } catch (const std::bad_alloc&) {
        return fail(PF_EDEVICE, "%s: host memory exhausted", name);
    } catch (const std::exception& e) {
        return fail(PF_EDEVICE, "%s: %s", name, e.what());
    } catch (...) {
        return fail(PF_EDEVICE, "%s: unexpected internal error", name);
    }
}

// launch shape of the 2-D explicit kernels for this problem on a device of `cus` compute
// units: rows per wave of single steps; steps fused per launch and rows per wave for each
// count of fused steps (fixed: the count was set by pf_tune_set; else calls of one or two
// steps are not fused); prefetch depth
struct Stream2DPlan {
    int ks = 1, ty[5] = {};
    bool fixed = false;
};
int stream2d_rows(const pf_problem* p, int cus);
Stream2DPlan stream2d_plan(const pf_problem* p, int cus, int64_t nsteps);
int stream2d_depth(const pf_problem* p);

size_t newton_workspace_bytes(const pf_problem* p, int restart);
size_t vjp_workspace_bytes(const pf_problem* p);

}  // namespace pfapi
