// Columns of a field read through the cache: what the kernels share in which
// a thread owns one column (i1, i2) of several consecutive planes of axis 0
// (ace_col3d.hip, ace_pop.hip).  In-plane byte offsets are 32-bit (planes of
// fewer than 2^28 nodes); an offset past the plane makes a buffer load return
// 0, the Dirichlet wall; a Neumann neighbour past the end is the node itself.
#pragma once

#include "ace_device.h"

namespace ace {
namespace col {

constexpr int CNT = 256;  // threads per workgroup
constexpr int kBufWord3 = 0x00020000;    // fourth descriptor word of the gfx9 family
constexpr uint32_t kNone = 0x80000000u;  // byte offset past any plane: loads 0, stores nothing

using BufB64 = decltype(__builtin_amdgcn_raw_buffer_load_b64(__amdgpu_buffer_rsrc_t(), 0, 0, 0));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const double *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), (short)0, bytes, kBufWord3);
}

__device__ __forceinline__ double load(const __amdgpu_buffer_rsrc_t &r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

// Byte offsets in a plane of flat node j (kNone past the end) and of its
// in-plane neighbours, and where the node lies on the axes' ends.
struct Col {
    uint32_t o, ym, yp, xm, xp;
    bool y0, x0;
};

template <int BC>
__device__ __forceinline__ Col column(int j, int M1, int M2)
{
    Col c;
    const int PS = M1 * M2;
    const bool in = j < PS;
    const int y = in ? j / M2 : 0, x = in ? j - y * M2 : 0;
    const int jj = in ? j : 0;
    auto at = [&](bool inside, int inner, int wrapped) -> uint32_t {
        if (inside) return (uint32_t)inner * 8u;
        if (BC == BC_HN) return (uint32_t)jj * 8u;
        if (BC == BC_HD) return kNone;
        return (uint32_t)wrapped * 8u;
    };
    c.ym = at(y > 0, jj - M2, jj + (M1 - 1) * M2);
    c.yp = at(y < M1 - 1, jj + M2, jj - (M1 - 1) * M2);
    c.xm = at(x > 0, jj - 1, jj + (M2 - 1));
    c.xp = at(x < M2 - 1, jj + 1, jj - (M2 - 1));
    c.o = in ? (uint32_t)j * 8u : kNone;
    c.y0 = y == 0;
    c.x0 = x == 0;
    return c;
}

// Plane z under the BC as a buffer (no bytes, so all zero, past a Dirichlet
// wall).
template <int BC>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_at(const double *in, int z, int M0, int PS)
{
    int m = z, bytes = PS * 8;
    if (z < 0) {
        m = BC == BC_P ? z + M0 : 0;
        if (BC == BC_HD) bytes = 0;
    } else if (z >= M0) {
        m = BC == BC_P ? z - M0 : M0 - 1;
        if (BC == BC_HD) bytes = 0;
    }
    return plane_rsrc(in + (int64_t)m * PS, bytes);
}

}  // namespace col
}  // namespace ace
