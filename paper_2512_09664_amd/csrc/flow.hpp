// Bilinear sampling of a pair's cell-centred flow grid (shared by the
// advection kernel and its adjoint).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "synthpix.h"

namespace sp {

// Two consecutive (u, v) nodes as one 16-byte load (8-byte aligned address; the
// hardware handles the unaligned vector access), from global memory also where
// the pointer came out of a descriptor.
__device__ __forceinline__ float4 load_pair(const float2* p)
{
    typedef float vec4 __attribute__((ext_vector_type(4), aligned(8)));
    const vec4 v = *(const __attribute__((address_space(1))) vec4*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}

struct FlowView {
    const float2* __restrict__ F;
    int Gh, Gw;
    float sx, sy;      // Gw / W, Gh / H (correctly rounded)
};

// A rectangle of a pair's grid nodes copied to LDS (rows wi0 .., columns wj0 ..,
// wh x ww nodes, row-major, wh and ww >= 1); NO_WIN (a single node, which holds
// no whole cell) means none.  The nodes themselves are passed separately, as
// the workgroup's LDS arrays of (u, v) pairs and, for motion out of the plane, w.
struct FlowWin {
    int wi0, wj0, wh, ww;
};

constexpr FlowWin NO_WIN = {0, 0, 1, 1};

typedef float vec2f __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) const vec2f lds_vec2;     // LDS (group segment) (u, v) node
typedef __attribute__((address_space(3))) const float lds_float;    // LDS word

// The grid cell of image position (px, py), clamped to the node hull (not a
// number: cell 0), and the position inside it.  A median clamps in one
// instruction; truncation is the floor of the clamped, non-negative coordinate.
struct FlowCell {
    int i0, j0;
    float fx, fy;
};

__device__ __forceinline__ FlowCell flow_cell(const FlowView& fv, float px, float py)
{
    const float gx = __builtin_amdgcn_fmed3f(px * fv.sx - 0.5f, 0.0f, (float)(fv.Gw - 1));
    const float gy = __builtin_amdgcn_fmed3f(py * fv.sy - 0.5f, 0.0f, (float)(fv.Gh - 1));
    FlowCell c;
    c.j0 = min((int)gx, fv.Gw - 2);
    c.i0 = min((int)gy, fv.Gh - 2);
    c.fx = gx - (float)c.j0;
    c.fy = gy - (float)c.i0;
    return c;
}

__device__ __forceinline__ float bilinear(float a, float b, float c, float e, float fx, float fy)
{
    const float top = __builtin_fmaf(fx, b - a, a);
    const float bot = __builtin_fmaf(fx, e - c, c);
    return __builtin_fmaf(fy, bot - top, top);
}

// Whether the cell lies in the window: 0 <= li < wh - 1 and 0 <= lj < ww - 1, each
// as one unsigned comparison.
__device__ __forceinline__ bool in_window(const FlowCell& c, const FlowWin& win)
{
    return ((unsigned)(c.i0 - win.wi0) < (unsigned)(win.wh - 1)) & ((unsigned)(c.j0 - win.wj0) < (unsigned)(win.ww - 1));
}

__device__ __forceinline__ unsigned window_node(const FlowCell& c, const FlowWin& win)
{
    return __umul24((unsigned)(c.i0 - win.wi0), (unsigned)win.ww) + (unsigned)(c.j0 - win.wj0);
}

// The (u, v) nodes of a cell, (left, right) of its upper and of its lower grid row:
// adjacent, one 16-byte load per row, or from the LDS window when the cell lies
// inside it.
__device__ __forceinline__ void cell_nodes(const FlowView& fv, const FlowCell& c, bool inside, const FlowWin& win,
                                           lds_vec2* lds, float4& r0, float4& r1)
{
    if (inside) {
        lds_vec2* w0 = lds + window_node(c, win);
        lds_vec2* w1 = w0 + win.ww;
        const vec2f a = w0[0], b = w0[1], d = w1[0], e = w1[1];
        r0 = make_float4(a.x, a.y, b.x, b.y);
        r1 = make_float4(d.x, d.y, e.x, e.y);
    } else {
        // nodes of one pair's grid (at most 2^26): 32-bit offsets
        const uint32_t k = (uint32_t)c.i0 * (uint32_t)fv.Gw + (uint32_t)c.j0;
        r0 = load_pair(fv.F + k);
        r1 = load_pair(fv.F + k + fv.Gw);
    }
}

// (u, v) in a cell.
__device__ __forceinline__ float2 sample_cell(const FlowView& fv, const FlowCell& c, bool inside, const FlowWin& win,
                                              lds_vec2* lds)
{
    float4 r0, r1;
    cell_nodes(fv, c, inside, win, lds, r0, r1);
    return make_float2(bilinear(r0.x, r0.z, r1.x, r1.z, c.fx, c.fy), bilinear(r0.y, r0.w, r1.y, r1.w, c.fx, c.fy));
}

__device__ __forceinline__ float2 sample_flow(const FlowView& fv, float px, float py)
{
    return sample_cell(fv, flow_cell(fv, px, py), false, NO_WIN, nullptr);
}

__device__ __forceinline__ float2 sample_flow(const FlowView& fv, const FlowWin& win, lds_vec2* lds, float px,
                                              float py)
{
    const FlowCell c = flow_cell(fv, px, py);
    return sample_cell(fv, c, in_window(c, win), win, lds);
}

__device__ __forceinline__ FlowView flow_view(const synthpix_pair& P, const float* flow)
{
    FlowView fv;
    fv.F = reinterpret_cast<const float2*>(flow + P.flow_offset);
    fv.Gh = P.Gh;
    fv.Gw = P.Gw;
    fv.sx = (float)P.Gw / (float)P.W;
    fv.sy = (float)P.Gh / (float)P.H;
    return fv;
}

// (((k1 + 2 k2) + 2 k3) + k4) / 6, each sum rounded (2 k is exact, so the doubled
// terms fuse).
__device__ __forceinline__ float rk4_mean(float k1, float k2, float k3, float k4)
{
    return (__builtin_fmaf(2.0f, k3, __builtin_fmaf(2.0f, k2, k1)) + k4) / 6.0f;
}

// One substep of the frozen-field integrator, the same operations in the same
// order as the advection kernel: Euler p = fma(h, u, p); RK4 stages at
// fma(h/2, k, p) and fma(h, k3, p), update fma(h, (((k1 + 2 k2) + 2 k3) + k4) / 6, p).
__device__ __forceinline__ void substep(const FlowView& fv, const FlowWin& win, lds_vec2* lds, float& px, float& py,
                                        float h, float hh, int integrator)
{
    if (integrator == SP_EULER) {
        const float2 u = sample_flow(fv, win, lds, px, py);
        px = __builtin_fmaf(h, u.x, px);
        py = __builtin_fmaf(h, u.y, py);
        return;
    }
    const float2 k1 = sample_flow(fv, win, lds, px, py);
    const float2 k2 = sample_flow(fv, win, lds, __builtin_fmaf(hh, k1.x, px), __builtin_fmaf(hh, k1.y, py));
    const float2 k3 = sample_flow(fv, win, lds, __builtin_fmaf(hh, k2.x, px), __builtin_fmaf(hh, k2.y, py));
    const float2 k4 = sample_flow(fv, win, lds, __builtin_fmaf(h, k3.x, px), __builtin_fmaf(h, k3.y, py));
    px = __builtin_fmaf(h, rk4_mean(k1.x, k2.x, k3.x, k4.x), px);
    py = __builtin_fmaf(h, rk4_mean(k1.y, k2.y, k3.y, k4.y), py);
}

}  // namespace sp
