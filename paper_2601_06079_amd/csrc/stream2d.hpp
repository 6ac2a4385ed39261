// stream2d.hpp -- helpers of the row-streaming 2-D kernels (one 64-lane
// wavefront per strip of columns, rows marched through registers).
#pragma once
#include <algorithm>
#include "device.hpp"

namespace pfk {
namespace {

// raw buffer access: the row offset is a scalar (one SGPR), the column offset
// a per-lane VGPR set once, so no per-row address arithmetic runs on the VALU.
// Out-of-range addresses read 0 and drop stores (the launcher keeps every
// access in range; this is the hardware's own bounds check on top).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <>
__device__ __forceinline__ float bload<float>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
template <>
__device__ __forceinline__ double bload<double>(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    return __hiloint2double((int)v.y, (int)v.x);
}
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, voff, soff, 0);
}
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    v2u w;
    w.x = (unsigned)__double2loint(v);
    w.y = (unsigned)__double2hiint(v);
    __builtin_amdgcn_raw_buffer_store_b64(w, r, voff, soff, 0);
}

// wave index made provably uniform so that all row bookkeeping stays scalar
__device__ __forceinline__ int uniform_wave()
{
    return (int)(blockIdx.x * (blockDim.x / WAVE)) +
           __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
}

}  // namespace
// Rows per wave of one row-streamed pass over ny rows and nstrips strips, H halo rows a
// side, rows taken in groups of four.  Where one wave per SIMD covers the grid the shortest
// chunks win (2-D products, FP32, us: 300 x 260 2 rows 2.7, 6 3.4, 8 4.1; 500^2 6 rows 3.6,
// 8 4.2; FP64 500^2 4.5 / 5.4).  Else chunks for about four waves per SIMD, never shorter
// than 8 rows, which nothing tried beats by more than it loses elsewhere.  any = false:
// only the latter (waves with sums of their own, whose number a workspace bounds).
inline int pass_rows(int ny, int nstrips, int H, int cus, bool any = true)
{
    const long long simds = 4ll * cus;
    for (int len = 4; any && len <= 8; len += 4) {
        const int ty = std::min(len - 2 * H, ny);
        if (ty > 0 && (long long)nstrips * ((ny + ty - 1) / ty) <= simds) return ty;
    }
    long long nch = std::max<long long>(1, 4 * simds / nstrips);
    nch = std::min<long long>(nch, std::max(1, ny / 8));
    return (int)((ny + nch - 1) / nch);
}

}  // namespace pfk
