// Particle seeding and inter-frame advection kernels (gfx950).
//
// Seeding follows Section 2, "Sampling the particles": n_max candidates per
// pair drawn over the image, the pair's ppp drawn uniformly, particles past
// n_active masked with zero intensity; per-particle parameters uniform in
// their ranges (the paragraph after Eq. 1), the diameter optionally a clipped
// normal.  Advection implements the same passage's x -> x + u(x), generalised to
// dt with Euler or RK4 substeps on a bilinear, cell-centred flow grid.
//
// One thread per particle; SoA float stores are fully coalesced.  Both kernels
// are bound by Philox / interpolation arithmetic, not by memory.
#include "device_math.hpp"
#include "flow.hpp"
#include "launch.hpp"

namespace sp {

// The pair's drawn ppp and active-particle count (Philox stream 5, index 0).
__device__ __forceinline__ int pair_active(const synthpix_pair& P, uint64_t pid, const synthpix_seed_params& prm,
                                           uint64_t seed, double* ppp_out)
{
    const u32x4 w = draw(0u, STREAM_PAIR, pid, seed);
    const double ppp = prm.ppp_lo + (prm.ppp_hi - prm.ppp_lo) * (double)u24(w.a);
    const double na = floor((double)P.H * (double)P.W * ppp + 0.5);
    *ppp_out = ppp;
    return na < (double)P.n_max ? (int)na : P.n_max;
}

// Workgroups below `blocks` seed the particles, the ones after them write the
// pairs' counts and densities.
__global__ void __launch_bounds__(256)
seed_kernel(const synthpix_pair* __restrict__ pairs, int n_pairs, int64_t n_span, unsigned blocks,
            synthpix_seed_params prm, uint64_t seed,
            float* __restrict__ x, float* __restrict__ y, float* __restrict__ z,
            float* __restrict__ d, float* __restrict__ I0, int32_t* __restrict__ n_active_out,
            double* __restrict__ ppp_out, const synthpix_batch_io* __restrict__ iod,
            int32_t* __restrict__ live_out)
{
    if (blockIdx.x >= blocks) {
        const int p = (int)(blockIdx.x - blocks) * 256 + (int)threadIdx.x;
        if (p >= n_pairs) return;
        uint64_t base = 0;
        if (iod) {
            seed = iod->seed;
            base = iod->pair_id_base;
            n_active_out = iod->n_active;
            ppp_out = iod->ppp;
        }
        double ppp;
        const int na = pair_active(pairs[p], pairs[p].pair_id + base, prm, seed, &ppp);
        if (n_active_out) n_active_out[p] = na;
        if (ppp_out) ppp_out[p] = ppp;
        if (live_out) live_out[p] = na;
        return;
    }
    const bool masked_still = iod && live_out;
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t g = g0 + threadIdx.x;
    if (g >= n_span) return;
    const int p = find_pair_from(pairs, n_pairs, g0, g);
    const synthpix_pair P = pairs[p];
    const int64_t i64 = g - P.particle_offset;
    if (i64 < 0 || i64 >= P.n_max) return;
    const uint32_t i = (uint32_t)i64;
    uint64_t pid = P.pair_id;
    if (iod) {
        x = iod->x1;
        y = iod->y1;
        z = iod->z;
        d = iod->d;
        I0 = iod->I0;
        seed = iod->seed;
        pid += iod->pair_id_base;
    }

    double ppp;
    const int n_active = pair_active(P, pid, prm, seed, &ppp);

    const u32x4 gw = draw(i, STREAM_GEOM, pid, seed);
    const u32x4 hw = draw(i, STREAM_PHOTO, pid, seed);
    const float px = u24(gw.a) * (float)P.W, py = u24(gw.b) * (float)P.H;
    x[g] = px;
    y[g] = py;
    if (masked_still && (int)i >= n_active) {
        // a masked candidate is not advected: its frame-2 position is its frame-1 one
        iod->x2[g] = px;
        iod->y2[g] = py;
    }
    z[g] = __builtin_fmaf(prm.z_hi - prm.z_lo, u24(gw.c), prm.z_lo);
    float dv;
    if (prm.d_dist == SP_DIST_UNIFORM) {
        dv = __builtin_fmaf(prm.d_b - prm.d_a, u24(gw.d), prm.d_a);
    } else {
        const float l = log_ra(u24_open0(hw.b));
        const float R = __builtin_sqrtf(-2.0f * l);
        const float n = R * cos2pi_ra(u24(hw.c));
        float v = __builtin_fmaf(prm.d_b, n, prm.d_a);
        v = __builtin_fmaxf(v, prm.d_lo);
        dv = __builtin_fminf(v, prm.d_hi);
    }
    d[g] = dv;
    I0[g] = ((int)i < n_active) ? __builtin_fmaf(prm.I0_hi - prm.I0_lo, u24(hw.a), prm.I0_lo) : 0.0f;
}

constexpr int ADVECT_WIN_NODES = 2048;   // LDS window of grid nodes (16 KB, 24 KB with w)
constexpr int ADVECT_WIN_MARGIN = 4;     // cells added around the starting cells

struct Velocity {
    float u, v, w;
};

// (u, v) and, with W3, the out-of-plane velocity w (one float per node, registered
// like the (u, v) grid) at (px, py).
template <bool W3>
__device__ __forceinline__ Velocity velocity(const FlowView& fv, const float* __restrict__ G, float px, float py,
                                             const FlowWin& win, lds_vec2* lds, lds_float* ldsw)
{
    const FlowCell c = flow_cell(fv, px, py);
    const bool inside = in_window(c, win);
    const float2 u = sample_cell(fv, c, inside, win, lds);
    Velocity o = {u.x, u.y, 0.0f};
    if constexpr (W3) {
        float a, b, d, e;
        if (inside) {
            lds_float* w0 = ldsw + window_node(c, win);
            lds_float* w1 = w0 + win.ww;
            a = w0[0];
            b = w0[1];
            d = w1[0];
            e = w1[1];
        } else {
            const float* w0 = G + (size_t)c.i0 * fv.Gw + c.j0;
            const float* w1 = w0 + fv.Gw;
            a = w0[0];
            b = w0[1];
            d = w1[0];
            e = w1[1];
        }
        o.w = bilinear(a, b, d, e, c.fx, c.fy);
    }
    return o;
}

// One particle per thread through the frozen field; the update order is fixed
// (see the reference arithmetic): Euler p = fma(h, u, p); RK4 stages at
// fma(h/2, k, p) and fma(h, k3, p), update p = fma(h, (((k1 + 2 k2) + 2 k3) + k4) /
// 6, p).  W3 (Remark 1's particles in 3-D space under a 3-D flow): z integrates
// w(x, y) with the same stages, w_k at the k-th stage position.
//
// SORTED: thread slots follow the home-block order (neighbouring lanes sample
// neighbouring grid cells, so the bilinear gathers share cache lines); each
// slot reads its particle index from the order's entry list, and the grid nodes
// around the workgroup's starting cells are copied to LDS.  (Sorting the
// positions themselves and taking the results back to index order in a launch of
// its own moves the random accesses out of this kernel: 64 pairs of 1024^2, order
// and advection 154 -> 177 us, 32 dense pairs of 2048^2 960 -> 952.)
//
// Where all of a wave's slots belong to one pair, the pair's grid, scales and window are
// wave-uniform (scalar) values; else each lane has its own pair's.  (A wave's pairs one
// after another, for scalar values throughout: 64 pairs of 8 particles, RK4 x 4, 41 us for
// 8.5; 1024 of 82 in pairs of two 10.6 for 8.9.)
// Bound together by VALU issue (0.87 of the nominal rate), the LDS window's reads
// (active 0.74 of the time, half of it bank conflicts) and, for large pairs, the
// random reads and writes of the positions: 64 pairs of 1024^2, RK4 x 4, 110 us, 80
// with no substep at all; 32 dense pairs of 2048^2, RK4 x 8, 750 us, 685 without.
// Motion out of the plane (16 pairs of 1024^2) took 222 us in index order without
// the window, 48 us and 24 for the order with it.
template <bool SORTED, bool W3>
__global__ void __launch_bounds__(256)
advect_kernel(const synthpix_pair* __restrict__ pairs, int n_pairs, int64_t n_span,
              const float* __restrict__ flow, const float* __restrict__ wflow, synthpix_advect_params ap,
              const float* __restrict__ x1, const float* __restrict__ y1, const float* __restrict__ z1,
              float* __restrict__ x2, float* __restrict__ y2, float* __restrict__ z2, AdvectOrder order,
              const synthpix_batch_io* __restrict__ iod)
{
    if (iod) {
        flow = iod->flow;
        x1 = iod->x1;
        y1 = iod->y1;
        x2 = iod->x2;
        y2 = iod->y2;
    }
    // consecutive particle blocks (same pair, same flow grid) stay on one XCD
    const int64_t g0 = (int64_t)xcd_contiguous(blockIdx.x, gridDim.x) * 256;
    const int64_t slot = g0 + threadIdx.x;
    float px = 0.0f, py = 0.0f, pz = 0.0f;
    int64_t g = 0;
    int p = -1;                              // the slot's pair (-1: no particle to move)
    if (slot < n_span) {
        const int q = find_pair_from(pairs, n_pairs, g0, slot);
        const int64_t i = slot - pairs[q].particle_offset;
        if (i >= 0 && i < (order.live ? (int64_t)order.live[q] : (int64_t)pairs[q].n_max)) {
            p = q;
            g = SORTED ? pairs[q].particle_offset + order.entries[order.L[q].entry_base + i] : slot;
            px = x1[g];
            py = y1[g];
            if (W3) pz = z1[g];
        }
    }
    // SORTED: the workgroup's particles start in a compact patch of the image;
    // the grid nodes around their starting cells (those of the first slot's
    // pair, grown by a margin) are copied to LDS when they fit
    __shared__ vec2f s_win[SORTED ? ADVECT_WIN_NODES : 1];
    __shared__ float s_winw[SORTED && W3 ? ADVECT_WIN_NODES : 1];
    __shared__ int s_box[4][4];
    __shared__ int s_pair;
    FlowWin win0 = NO_WIN;                   // the window and its pair
    int pw = -1;
    if (SORTED) {
        if (threadIdx.x == 0) s_pair = p;
        __syncthreads();
        pw = __builtin_amdgcn_readfirstlane(s_pair);
        int bi0 = 1 << 30, bj0 = 1 << 30, bi1 = -1, bj1 = -1;
        if (pw >= 0 && p == pw) {
            const FlowCell c = flow_cell(flow_view(pairs[pw], flow), px, py);
            bj0 = bj1 = c.j0;
            bi0 = bi1 = c.i0;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            bi0 = min(bi0, __shfl_xor(bi0, o, 64));
            bj0 = min(bj0, __shfl_xor(bj0, o, 64));
            bi1 = max(bi1, __shfl_xor(bi1, o, 64));
            bj1 = max(bj1, __shfl_xor(bj1, o, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            s_box[threadIdx.x >> 6][0] = bi0;
            s_box[threadIdx.x >> 6][1] = bj0;
            s_box[threadIdx.x >> 6][2] = bi1;
            s_box[threadIdx.x >> 6][3] = bj1;
        }
        __syncthreads();
        if (pw >= 0) {
            const synthpix_pair Q = pairs[pw];
            bi0 = max(min(min(s_box[0][0], s_box[1][0]), min(s_box[2][0], s_box[3][0])) - ADVECT_WIN_MARGIN, 0);
            bj0 = max(min(min(s_box[0][1], s_box[1][1]), min(s_box[2][1], s_box[3][1])) - ADVECT_WIN_MARGIN, 0);
            bi1 = min(max(max(s_box[0][2], s_box[1][2]), max(s_box[2][2], s_box[3][2])) + ADVECT_WIN_MARGIN + 1,
                      Q.Gh - 1);
            bj1 = min(max(max(s_box[0][3], s_box[1][3]), max(s_box[2][3], s_box[3][3])) + ADVECT_WIN_MARGIN + 1,
                      Q.Gw - 1);
            const int wi0 = __builtin_amdgcn_readfirstlane(bi0), wj0 = __builtin_amdgcn_readfirstlane(bj0);
            const int wh = __builtin_amdgcn_readfirstlane(bi1) - wi0 + 1;
            const int ww = __builtin_amdgcn_readfirstlane(bj1) - wj0 + 1;
            if (wh >= 1 && ww >= 1 && wh * ww <= ADVECT_WIN_NODES) {
                const vec2f* F = reinterpret_cast<const vec2f*>(flow + Q.flow_offset);
                // window row of node k without an integer division: (k + 1/2) / ww lies at
                // least 1/(2 ww) from an integer and, for k < 2048, the float product errs
                // by under 2048 * 2^-21 / ww, so truncation gives floor(k / ww)
                const float inv_ww = 1.0f / (float)ww;
                for (int k = threadIdx.x; k < wh * ww; k += 256) {
                    const int r = (int)(((float)k + 0.5f) * inv_ww);
                    const int64_t node = (int64_t)(wi0 + r) * Q.Gw + wj0 + (k - r * ww);
                    s_win[k] = F[node];
                    if (W3) s_winw[k] = wflow[Q.flow_offset / 2 + node];
                }
                win0 = FlowWin{wi0, wj0, wh, ww};
            }
        }
        __syncthreads();
    }
    const float h = ap.dt / (float)ap.substeps;
    const float hh = h * 0.5f;
    lds_vec2* lds = (lds_vec2*)s_win;
    lds_float* ldsw = (lds_float*)s_winw;
    auto move = [&](const FlowView& fv, const float* G, const FlowWin& win) {
        if (ap.integrator == SP_EULER) {
            for (int s = 0; s < ap.substeps; ++s) {
                const Velocity k = velocity<W3>(fv, G, px, py, win, lds, ldsw);
                px = __builtin_fmaf(h, k.u, px);
                py = __builtin_fmaf(h, k.v, py);
                if (W3) pz = __builtin_fmaf(h, k.w, pz);
            }
        } else {
            for (int s = 0; s < ap.substeps; ++s) {
                const Velocity k1 = velocity<W3>(fv, G, px, py, win, lds, ldsw);
                const Velocity k2 = velocity<W3>(fv, G, __builtin_fmaf(hh, k1.u, px), __builtin_fmaf(hh, k1.v, py),
                                                 win, lds, ldsw);
                const Velocity k3 = velocity<W3>(fv, G, __builtin_fmaf(hh, k2.u, px), __builtin_fmaf(hh, k2.v, py),
                                                 win, lds, ldsw);
                const Velocity k4 = velocity<W3>(fv, G, __builtin_fmaf(h, k3.u, px), __builtin_fmaf(h, k3.v, py),
                                                 win, lds, ldsw);
                px = __builtin_fmaf(h, rk4_mean(k1.u, k2.u, k3.u, k4.u), px);
                py = __builtin_fmaf(h, rk4_mean(k1.v, k2.v, k3.v, k4.v), py);
                if (W3) pz = __builtin_fmaf(h, rk4_mean(k1.w, k2.w, k3.w, k4.w), pz);
            }
        }
    };
    const unsigned long long some = __builtin_amdgcn_ballot_w64(p >= 0);
    if (some != 0) {
        const int q = __builtin_amdgcn_readlane(p, __builtin_ctzll(some));
        if (__builtin_amdgcn_ballot_w64(p == q) == some) {
            if (p == q)
                move(flow_view(pairs[q], flow), W3 ? wflow + pairs[q].flow_offset / 2 : nullptr,
                     SORTED && q == pw ? win0 : NO_WIN);
        } else if (p >= 0) {
            move(flow_view(pairs[p], flow), W3 ? wflow + pairs[p].flow_offset / 2 : nullptr,
                 SORTED && p == pw ? win0 : NO_WIN);
        }
    }
    if (p >= 0) {
        x2[g] = px;
        y2[g] = py;
        if (W3) z2[g] = pz;
    }
}

// Second diameter d_y and correlation rho of Eq. 1 per candidate particle
// (anisotropic particle images; the sentence after Eq. 1 draws every shape
// parameter per particle): d_y from the seed's diameter distribution, rho
// uniform in [rho_lo, rho_hi]; Philox stream 6 (word 0: uniform d_y; words 1, 2:
// Box-Muller of a normal d_y; word 3: rho).
__global__ void __launch_bounds__(256)
seed_shape_kernel(const synthpix_pair* __restrict__ pairs, int n_pairs, int64_t n_span, synthpix_seed_params prm,
                  float rho_lo, float rho_hi, uint64_t seed, float* __restrict__ dy, float* __restrict__ rho)
{
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x;
    const int64_t g = g0 + threadIdx.x;
    if (g >= n_span) return;
    const int p = find_pair_from(pairs, n_pairs, g0, g);
    const synthpix_pair P = pairs[p];
    const int64_t i64 = g - P.particle_offset;
    if (i64 < 0 || i64 >= P.n_max) return;
    const u32x4 w = draw((uint32_t)i64, STREAM_SHAPE, P.pair_id, seed);
    float v;
    if (prm.d_dist == SP_DIST_UNIFORM) {
        v = __builtin_fmaf(prm.d_b - prm.d_a, u24(w.a), prm.d_a);
    } else {
        const float R = __builtin_sqrtf(-2.0f * log_ra(u24_open0(w.b)));
        v = __builtin_fmaf(prm.d_b, R * cos2pi_ra(u24(w.c)), prm.d_a);
        v = __builtin_fminf(__builtin_fmaxf(v, prm.d_lo), prm.d_hi);
    }
    dy[g] = v;
    rho[g] = __builtin_fmaf(rho_hi - rho_lo, u24(w.d), rho_lo);
}

// Ground-truth flow of each pair (the sampler's flow_fields): the pair's (u, v)
// grid sampled bilinearly at every pixel centre, (c + 1/2, r + 1/2), exactly
// as the advection samples it; written as [H][W][2] floats at the pair's image
// offset (2 H W floats, the extent of its two float frames).
// Bound by its stores.  A thread takes FIELD_PX consecutive pixels (whole 16-byte
// stores) of up to FIELD_PAIRS consecutive pairs: pairs that share a grid and a
// shape, as a sampler's B / F pairs per field do, are sampled once.  64 pairs of
// 512^2 under one field (134 MB): one pixel of one pair per thread, with a 64-bit
// division, 41 us; two of one pair 35; of 8 pairs 27 (4.9 TB/s); four pixels 30.
constexpr int FIELD_PX = 2, FIELD_PAIRS = 8;

__global__ void __launch_bounds__(256)
flow_field_kernel(const synthpix_pair* __restrict__ pairs, int n_pairs, const float* __restrict__ flow,
                  float* __restrict__ out)
{
    typedef float vec4 __attribute__((ext_vector_type(4), aligned(8)));
    const int p0 = blockIdx.y * FIELD_PAIRS, p1 = min(p0 + FIELD_PAIRS, n_pairs);
    const uint32_t k0 = (blockIdx.x * 256u + threadIdx.x) * FIELD_PX;
    float2 u[FIELD_PX];
    for (int p = p0; p < p1; ++p) {
        const synthpix_pair P = pairs[p];
        const uint32_t n = (uint32_t)P.H * (uint32_t)P.W;       // at most 2^28
        bool fresh = p == p0;
        if (!fresh) {
            const synthpix_pair& Q = pairs[p - 1];
            fresh = P.flow_offset != Q.flow_offset || P.H != Q.H || P.W != Q.W || P.Gh != Q.Gh || P.Gw != Q.Gw;
        }
        if (k0 >= n) continue;
        if (fresh) {
            const FlowView fv = flow_view(P, flow);
            int r = (int)(k0 / (uint32_t)P.W), c = (int)(k0 - (uint32_t)r * (uint32_t)P.W);
#pragma unroll
            for (int q = 0; q < FIELD_PX; ++q) {
                u[q] = sample_flow(fv, (float)c + 0.5f, (float)r + 0.5f);
                if (++c == P.W) {
                    c = 0;
                    ++r;
                }
            }
        }
        float* o = out + P.image_offset + 2 * (int64_t)k0;
        if (k0 + FIELD_PX <= n) {
#pragma unroll
            for (int q = 0; q < FIELD_PX; q += 2) {
                const vec4 v = {u[q].x, u[q].y, u[q + 1].x, u[q + 1].y};
                *reinterpret_cast<vec4*>(o + 2 * q) = v;
            }
        } else {
#pragma unroll
            for (int q = 0; q < FIELD_PX; ++q)
                if (k0 + q < n) *reinterpret_cast<float2*>(o + 2 * q) = u[q];
        }
    }
}

hipError_t launch_flow_field(const synthpix_pair* pairs_dev, int n_pairs, int64_t max_px, const float* flow, float* out,
                             hipStream_t s)
{
    if (max_px <= 0) return hipSuccess;
    TimedScope ts("flow_field", s);
    const int64_t per = 256 * FIELD_PX;
    hipLaunchKernelGGL(flow_field_kernel,
                       dim3((unsigned)((max_px + per - 1) / per), (unsigned)((n_pairs + FIELD_PAIRS - 1) / FIELD_PAIRS)),
                       dim3(256), 0, s, pairs_dev, n_pairs, flow, out);
    return hipGetLastError();
}

hipError_t launch_seed_shape(const synthpix_pair* pairs_dev, int n_pairs, int64_t n_span,
                             const synthpix_seed_params& prm, float rho_lo, float rho_hi, uint64_t seed, float* dy,
                             float* rho, hipStream_t s)
{
    if (n_span <= 0) return hipSuccess;
    TimedScope ts("seed_shape", s);
    hipLaunchKernelGGL(seed_shape_kernel, dim3((unsigned)((n_span + 255) / 256)), dim3(256), 0, s, pairs_dev, n_pairs,
                       n_span, prm, rho_lo, rho_hi, seed, dy, rho);
    return hipGetLastError();
}

// Moves a captured plan's descriptor on to the next batch of the same shape:
// the pair-id offset grows by `step` (the batch size), so replays draw fresh
// particles.
__global__ void advance_pair_ids(synthpix_batch_io* __restrict__ iod, uint64_t step)
{
    if (threadIdx.x == 0) iod->pair_id_base += step;
}

__global__ void store_io(synthpix_batch_io* __restrict__ iod, synthpix_batch_io io)
{
    if (threadIdx.x == 0) *iod = io;
}

hipError_t launch_advance(synthpix_batch_io* iod, uint64_t step, hipStream_t s)
{
    hipLaunchKernelGGL(advance_pair_ids, dim3(1), dim3(64), 0, s, iod, step);
    return hipGetLastError();
}

hipError_t launch_store_io(synthpix_batch_io* iod, const synthpix_batch_io& io, hipStream_t s)
{
    hipLaunchKernelGGL(store_io, dim3(1), dim3(64), 0, s, iod, io);
    return hipGetLastError();
}

hipError_t launch_seed(const synthpix_pair* pairs_dev, int n_pairs, int64_t n_span,
                       const synthpix_seed_params& prm, uint64_t seed, float* x, float* y, float* z,
                       float* d, float* I0, int32_t* n_active, double* ppp, hipStream_t s,
                       const synthpix_batch_io* iod, int32_t* live)
{
    TimedScope ts("seed", s);
    const unsigned blocks = (unsigned)((n_span + 255) / 256);
    const unsigned more = n_active || ppp || iod || live ? (unsigned)((n_pairs + 255) / 256) : 0u;
    if (blocks + more > 0)
        hipLaunchKernelGGL(seed_kernel, dim3(blocks + more), dim3(256), 0, s, pairs_dev, n_pairs, n_span, blocks, prm,
                           seed, x, y, z, d, I0, n_active, ppp, iod, live);
    return hipGetLastError();
}

hipError_t launch_advect(const synthpix_pair* pairs_dev, int n_pairs, int64_t n_span, const float* flow,
                         const synthpix_advect_params& ap, const float* x1, const float* y1, float* x2,
                         float* y2, hipStream_t s, AdvectOrder order, const synthpix_batch_io* iod,
                         const float* wflow, const float* z1, float* z2)
{
    if (n_span <= 0) return hipSuccess;
    TimedScope ts("advect", s);
    const dim3 grid((unsigned)((n_span + 255) / 256)), block(256);
#define SP_ADVECT(SORTED_, W3_)                                                                                    \
    hipLaunchKernelGGL((advect_kernel<SORTED_, W3_>), grid, block, 0, s, pairs_dev, n_pairs, n_span, flow, wflow,   \
                       ap, x1, y1, z1, x2, y2, z2, order, iod)
    if (order.entries && wflow) SP_ADVECT(true, true);
    else if (order.entries) SP_ADVECT(true, false);
    else if (wflow) SP_ADVECT(false, true);
    else SP_ADVECT(false, false);
#undef SP_ADVECT
    return hipGetLastError();
}

}  // namespace sp
