// Adjoint of advect -> render -> blur (gfx950): given dL/dJ of the float images,
// the gradients with respect to frame-1 positions, z, d, I0, each pair's sheet
// width and each pair's flow grid.
//
// Render adjoint (Eq. 1 with sigma = d/4 and peak A = I0 exp(-z^2 / (2 s^2))):
// every particle's footprint is separable, t = A gx(c) gy(r), so with the
// zero-padded blur B (also separable) the four per-particle sums the chain rule
// needs,
//     S0 = sum_q e_q G_q,  Sx = sum e G dx,  Sy = sum e G dy,  Sr = sum e G (dx^2 + dy^2),
// e = B^T dL/dJ, equal sum_q (dL/dJ)_q Ty_j(r) Tx_k(c) with 1-D tables
// Tx_k = w * (gx dx^k) (the blur folded into the particle's factor tables).
// The gather is particle-major: a group of 8 or 16 lanes per particle reads its
// patch rows of dL/dJ with coalesced loads.  Once no blur is left to fold (none, or
// its adjoint has run per pixel), the sums are added in one order by two forms: a
// workgroup stages what the particles of a 64 x 64 pixel block cover in LDS and two
// lanes per particle gather from there, or, for small and sparse batches, eight
// lanes per particle gather row by row from global memory.  Nothing is scattered,
// no partial sums cross workgroups, and which form runs leaves no trace in the bits.
//
// Flow adjoint: a reverse sweep through the recomputed Euler / RK4 substeps
// (checkpointed).  Each bilinear sample passes its upstream gradient to its
// four grid nodes; consecutive samples in one cell are merged per particle,
// and node sums are accumulated in 64-bit fixed point, so the result does not
// depend on the order of the additions.  The fixed-point scale is a power of
// two from an a-priori bound on every upstream value (largest dL/dx2 and the
// flow's Lipschitz constant through the stage recurrences) and the sample
// count, so no sum can leave the int64 range.
#include "device_math.hpp"
#include "flow.hpp"
#include "launch.hpp"

namespace sp {

// Patch rows loaded per batch of the column walk (independent loads in flight; 4
// and 16 measured slower).  The rows' terms are added in row order whatever the
// batch.
constexpr int GROWS = 8;

// A particle's lane group: G = 16 lanes (a DPP row) or 8 (half of one); a
// workgroup of 256 threads holds 256 / G particles.  BT table slots cover the
// pixel range (<= 3 d_max + 3 pixels) plus 4 b of zero padding.  The raw
// factors are stored as the Gaussian values e alone (their dx and dx^2
// multiples are formed where they are read).
template <int G, int BT>
struct GatherLds {
    float rx[256 / G][BT];                      // raw column factors e(c) (slot = c - c0 + 2b)
    float ry[256 / G][BT];                      // raw row factors e(r)
    float4 ty[256 / G][BT];                     // blurred row tables (Ty0, Ty1, Ty2, 0)
};

// Sum over a particle's G lanes, result in every lane: quad butterflies
// (quad_perm [1,0,3,2] and [2,3,0,1]), then, for 16 lanes, rotations of the
// row by 4 and 8 lanes, for 8 lanes the mirror of each half row (the other
// quad of the eight).
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// A particle's lane group lies inside one wavefront and its LDS tables are
// private to it, so the group synchronises with a wave-level fence instead of
// a workgroup barrier (LDS operations of one wave complete in issue order).
__device__ __forceinline__ void group_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    static_assert(G == 8 || G == 16, "a lane group is a DPP row or half of one");
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    if constexpr (G == 16) {
        v += dpp<0x124>(v);
        v += dpp<0x128>(v);
    } else {
        v += dpp<0x141>(v);
    }
    return v;
}

// exp(-q) for the gradient's factor tables: the hardware base-2 exponential
// (relative error about 1e-6 over the support's q <= 18, well inside the
// gradient's tolerance; the images themselves use the exact polynomial).
// Zero for q >= 80 or not a number.
__device__ __forceinline__ float expneg_hw(float q)
{
    return q < 80.0f ? __builtin_amdgcn_exp2f(q * -LOG2E_F) : 0.0f;
}

// Pixel indices that may hold the support |(k + 1/2) - p| <= R, clipped to
// [0, n): a superset by at most one index per side (the exact binary32 test
// is applied per pixel where the factor tables are filled).
__device__ __forceinline__ bool cover_range(float p, float R, int n, int& lo, int& hi)
{
    if (!__builtin_isfinite(p)) return false;
    const float a = p - R - 0.5f, b = p + R - 0.5f;
    if (b < -1.0f || a > (float)n) return false;
    const int l = (int)__builtin_floorf(a), h = (int)__builtin_ceilf(b);
    lo = l < 0 ? 0 : l;
    hi = h > n - 1 ? n - 1 : h;
    return lo <= hi;
}

// One lane group's sums for one frame of its particle: the raw factor tables,
// the blurred row tables (B > 0) and the gather
//     S0 = sum e G,  Sx = sum e G dx,  Sy = sum e G dy,  Sr = sum e G (dx^2 + dy^2)
// over the blurred support inside the image, reading pixel (r, c) of the
// frame's dL/dJ (B > 0) or B^T dL/dJ (B = 0) at src[r * W + c].  Every lane returns
// the group's sums.  on: the particle is valid and its support [c0, c1] x [r0, r1]
// is not empty.
template <int B, int BT, int G>
__device__ __forceinline__ float4 frame_sums(GatherLds<G, BT>& S, int grp, int lane, bool on, float x, float y,
                                             float kap, float R, int c0, int c1, int r0, int r1, int W, int H,
                                             const float* __restrict__ src, const float* blur_w)
{
    // raw factor tables over the slots the gather reads, 0 .. max(c1 - c0, r1 - r0)
    // + 4b (zeros outside the support); a group stops after its last one
    const int n_raw = on ? max(c1 - c0, r1 - r0) + 4 * B + 1 : 0;
#pragma unroll
    for (int m = 0; m < BT / G; ++m) {
        if (G * m >= n_raw) break;
        const int slot = lane + G * m;
        const int c = c0 - 2 * B + slot;
        float v0 = 0.0f;
        const float dx = ((float)c + 0.5f) - x;
        if (on && c >= c0 && c <= c1 && __builtin_fabsf(dx) <= R) v0 = expneg_hw(kap * (dx * dx));
        S.rx[grp][slot] = v0;
        const int r = r0 - 2 * B + slot;
        float u0 = 0.0f;
        const float dy = ((float)r + 0.5f) - y;
        if (on && r >= r0 && r <= r1 && __builtin_fabsf(dy) <= R) u0 = expneg_hw(kap * (dy * dy));
        if constexpr (B == 0) {
            const float u1 = u0 * dy;
            S.ty[grp][slot] = make_float4(u0, u1, u1 * dy, 0.0f);
        } else {
            S.ry[grp][slot] = u0;
        }
    }
    group_sync();
    if constexpr (B > 0) {
        // blurred row tables (the column ones are formed per column in the gather);
        // table slot t is pixel r0 - b + t; raw slot t + 2b - k holds pixel
        // r0 + t - k, whose offset dy gives the e dy and e dy^2 terms
        const int n_ty = on ? (r1 - r0 + 1) + 2 * B : 0;
#pragma unroll
        for (int m = 0; m < BT / G; ++m) {
            if (G * m >= n_ty) break;
            const int t = lane + G * m;
            if (t < BT - 2 * B) {
                float Y0 = 0.0f, Y1 = 0.0f, Y2 = 0.0f;
#pragma unroll
                for (int k = 0; k <= 2 * B; ++k) {
                    const float w = blur_w[k];
                    const float u0 = S.ry[grp][t + 2 * B - k];
                    const float dy = ((float)(r0 + t - k) + 0.5f) - y;
                    const float u1 = u0 * dy;
                    Y0 = __builtin_fmaf(w, u0, Y0);
                    Y1 = __builtin_fmaf(w, u1, Y1);
                    Y2 = __builtin_fmaf(w, u1 * dy, Y2);
                }
                S.ty[grp][t] = make_float4(Y0, Y1, Y2, 0.0f);
            }
        }
        group_sync();
    }

    // gather: sum_q (dL/dJ)_q Ty(r) Tx(c) over the blurred support, inside the
    // image.  The column factors are constant along a column, so each lane
    // first forms P_j = sum_r (dL/dJ) Ty_j(r) down a column, or a slice of one
    // (three FMAs per pixel), and applies Tx afterwards.  Columns go to lanes
    // in blocks of G; a block of m < G columns splits its rows into
    // G / m' slices (m' = m rounded up to a power of two), so the lanes a
    // narrow block would leave idle shorten its walk instead.
    float s0 = 0.0f, s_x = 0.0f, s_y = 0.0f, s_r = 0.0f;
    if (on) {
        const int nt = (c1 - c0 + 1) + 2 * B, nu = (r1 - r0 + 1) + 2 * B;
        const int tlo = B - c0 > 0 ? B - c0 : 0;
        const int thi = nt < W - c0 + B ? nt : W - c0 + B;
        const int ulo = B - r0 > 0 ? B - r0 : 0;
        const int uhi = nu < H - r0 + B ? nu : H - r0 + B;
        constexpr int LG = G == 16 ? 4 : 3;
        const float* T = S.rx[grp];
        const int ncol = thi - tlo, nrow = uhi - ulo;
        for (int cb = 0; cb < ncol; cb += G) {
            const int m = ncol - cb < G ? ncol - cb : G;
            const int lm = m > 8 ? 4 : m > 4 ? 3 : m > 2 ? 2 : m > 1 ? 1 : 0;   // log2 m'
            const int cl = lane & ((1 << lm) - 1);
            const int per = (nrow + (G >> lm) - 1) >> (LG - lm);                // rows per slice
            const int ua = ulo + (lane >> lm) * per;
            const int ub = ua + per < uhi ? ua + per : uhi;
            if (cl >= m || ua >= ub) continue;
            const int t = tlo + cb + cl;
            // walk down the column slice with a row pointer: whole batches of GROWS
            // rows (their loads issued together), then batches of 4, 2 and 1
            const float* __restrict__ q = src + (int64_t)(r0 - B + ua) * W + (c0 - B + t);
            float P0 = 0.0f, P1 = 0.0f, P2 = 0.0f;
            int u = ua;
#pragma unroll 1
            for (; u + GROWS <= ub; u += GROWS) {
                float e[GROWS];
#pragma unroll
                for (int k = 0; k < GROWS; ++k) {
                    e[k] = *q;
                    q += W;
                }
#pragma unroll
                for (int k = 0; k < GROWS; ++k) {
                    const float4 ty = S.ty[grp][u + k];
                    P0 = __builtin_fmaf(ty.x, e[k], P0);
                    P1 = __builtin_fmaf(ty.y, e[k], P1);
                    P2 = __builtin_fmaf(ty.z, e[k], P2);
                }
            }
#pragma unroll
            for (int nb = GROWS / 2; nb >= 1; nb >>= 1) {
                if (ub - u >= nb) {
                    float e[GROWS / 2];
#pragma unroll
                    for (int k = 0; k < nb; ++k) {
                        e[k] = *q;
                        q += W;
                    }
#pragma unroll
                    for (int k = 0; k < nb; ++k) {
                        const float4 ty = S.ty[grp][u + k];
                        P0 = __builtin_fmaf(ty.x, e[k], P0);
                        P1 = __builtin_fmaf(ty.y, e[k], P1);
                        P2 = __builtin_fmaf(ty.z, e[k], P2);
                    }
                    u += nb;
                }
            }
            // blurred column factors of this column, from the raw ones (raw slot
            // t + 2b - k holds column c0 + t - k)
            float X0 = 0.0f, X1 = 0.0f, X2 = 0.0f;
#pragma unroll
            for (int k = 0; k <= 2 * B; ++k) {
                const float w = B > 0 ? blur_w[k] : 1.0f;
                const float v0 = T[t + 2 * B - k];
                const float dx = ((float)(c0 + t - k) + 0.5f) - x;
                const float v1 = v0 * dx;
                X0 = __builtin_fmaf(w, v0, X0);
                X1 = __builtin_fmaf(w, v1, X1);
                X2 = __builtin_fmaf(w, v1 * dx, X2);
            }
            s0 = __builtin_fmaf(P0, X0, s0);
            s_x = __builtin_fmaf(P0, X1, s_x);
            s_y = __builtin_fmaf(P1, X0, s_y);
            s_r = __builtin_fmaf(P0, X2, __builtin_fmaf(P2, X0, s_r));
        }
    }
    const float4 out = make_float4(group_sum<G>(s0), group_sum<G>(s_x), group_sum<G>(s_y), group_sum<G>(s_r));
    group_sync();
    return out;
}

// Gradients of one particle from its two frames' sums.
struct ParticleGrads {
    float gx1, gy1, gx2, gy2, gd, gz, gI0, sheet;
};

__device__ __forceinline__ ParticleGrads particle_grads(float z, float d, float I0, float sheet_sigma, float4 f0,
                                                        float4 f1)
{
    const float kap = 8.0f / (d * d);
    const float sum0 = f0.x + f1.x, sumr = f0.w + f1.w;
    const float s = sheet_sigma;
    const float Sz = expneg((z * z) * (0.5f / (s * s)));
    const float A = I0 * Sz;
    const float k2 = 2.0f * kap;                // d/dx of -kap dx^2 is 2 kap dx
    ParticleGrads o;
    o.gx1 = A * k2 * f0.y;
    o.gy1 = A * k2 * f0.z;
    o.gx2 = A * k2 * f1.y;
    o.gy2 = A * k2 * f1.z;
    o.gd = A * (k2 / d) * sumr;                 // d kap / d d = -2 kap / d
    o.gI0 = sum0 * Sz;
    o.gz = sum0 * A * (-z / (s * s));
    o.sheet = sum0 * A * ((z * z) / (s * s * s));
    return o;
}

// Where the gather leaves dL/dx1, dL/dy1 of frame 1's render for the flow adjoint, which
// adds its own part and stores the sums: the first 2 KB of the partial of the adjoint
// workgroup that takes the particle (256 consecutive places of the pair's home-block
// order), which writes its partial after it has read them.
__device__ __forceinline__ float2* start_grads(const BwdArgs& a, int p, int64_t place)
{
    return reinterpret_cast<float2*>(a.grid.part + (a.grid.wg_base[p] + (place >> 8)) * (2 * WIN_NODES)) + (place & 255);
}

// Particle-major gather: G lanes per particle read their patch rows of the
// frame's gradient image from global memory (a blur of radius 1 folded into the
// tables, or diameters beyond the block and row gathers).
template <int B, int BT, int G>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(G == 8 ? 6 : 4)))
bwd_gather(BwdArgs a, int64_t n_span)
{
    __shared__ GatherLds<G, BT> S;
    const int grp = threadIdx.x / G, lane = threadIdx.x % G;
    const int64_t g0 = (int64_t)xcd_contiguous(blockIdx.x, gridDim.x) * (256 / G);
    int64_t g = g0 + grp;
    const int64_t slot = g;              // of the home-block order

    bool in_pair = false, valid = false;
    int H = 1, W = 1;
    int64_t img = 0;
    float2* start = nullptr;
    float z = 0.0f, d = 1.0f, I0 = 0.0f;
    if (g < n_span) {
        const int p = find_pair_from(a.pairs, a.n_pairs, g0, g);
        const synthpix_pair P = a.pairs[p];
        int64_t i = g - P.particle_offset;
        if (i >= 0 && i < P.n_max) {
            start = start_grads(a, p, i);
            // slots follow the home-block order: neighbouring groups read
            // overlapping rows of dL/dJ
            if (a.order.entries) i = a.order.entries[a.order.L[p].entry_base + i];
            g = P.particle_offset + i;
            in_pair = true;
            H = P.H;
            W = P.W;
            img = P.image_offset;
            z = a.z[g];
            d = a.d[g];
            I0 = a.I0[g];
            valid = (I0 > 0.0f) && (d > 0.0f);
            if (valid && !(d <= a.d_max)) {
                if (lane == 0) atomicOr(a.status, SP_STATUS_D_ABOVE_MAX);
                valid = false;
            }
        }
    }
    const float kap = 8.0f / (d * d);
    const float R = 1.5f * d;
    float4 fs[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        float x = 0.0f, y = 0.0f;
        if (in_pair) {
            x = f ? a.x2[g] : a.x1[g];
            y = f ? a.y2[g] : a.y1[g];
        }
        int c0 = 0, c1 = -1, r0 = 0, r1 = -1;
        bool on = valid && cover_range(x, R, W, c0, c1);
        on = on && cover_range(y, R, H, r0, r1);
        fs[f] = frame_sums<B, BT, G>(S, grp, lane, on, x, y, kap, R, c0, c1, r0, r1, W, H,
                                     a.grad + img + (int64_t)f * H * W, a.blur_w);
    }

    if (lane != 0) return;
    if (!in_pair) {
        // a slot in no pair's particle range (a gap of the packed arrays): zero gradients
        if (g < n_span) {
            a.g_x1[g] = 0.0f;
            a.g_y1[g] = 0.0f;
            a.g_z[g] = 0.0f;
            a.g_d[g] = 0.0f;
            a.g_I0[g] = 0.0f;
        }
        return;
    }
    ParticleGrads o{};
    if (valid) o = particle_grads(z, d, I0, a.sheet_sigma, fs[0], fs[1]);
    *start = make_float2(o.gx1, o.gy1);
    a.g_z[g] = o.gz;
    a.g_d[g] = o.gd;
    a.g_I0[g] = o.gI0;
    a.gx2[slot] = o.gx2;
    a.gy2[slot] = o.gy2;
    a.sheet[g] = o.sheet;
}

// ------------------------------------------------------------------ block gather

typedef float vec4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) const float glb_float;

__device__ __forceinline__ bool support_box(float x, float y, float d, int W, int H, int& c0, int& c1, int& r0,
                                            int& r1)
{
    const float R = 1.5f * d;
    return support_range(x, R, W, c0, c1) && support_range(y, R, H, r0, r1);
}

// Value of lane N of each pair of lanes.
template <int N>
__device__ __forceinline__ float pair_lane(float v)
{
    return dpp<N ? 0xF5 : 0xA0>(v);
}

// One lane's part of a particle's sums over rows r0 .. r1 and columns c, c + 2, ..,
// N of them (a particle has two lanes, c the first column of this one); columns past c1
// count as zeros.  q points at row r0, column c.  The column factors stay in
// registers; the two lanes form every other row's factor and exchange them.  Without
// GUARD, reads run past c1, up to column c + 2 N - 2, and meet zero factors there (a
// value that is not finite makes the sums NaN: the caller then takes gather_exact).
template <int N, bool GUARD, typename SRC>
__device__ __forceinline__ void gather_columns(SRC* q, int stride, float x, float y, float kap, int c, int c1,
                                               int r0, int r1, int h, float4& s)
{
    float g0[N], g1[N], g2[N];
    const float fx = (float)c + 0.5f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float dx = (fx + (float)(2 * k)) - x;
        const float v = expneg_hw(kap * (dx * dx));
        g0[k] = c + 2 * k <= c1 ? v : 0.0f;
        g1[k] = g0[k] * dx;
        g2[k] = g1[k] * dx;
    }
    float fy = (float)(r0 + h) + 0.5f;
#pragma unroll 1
    for (int r = r0; r <= r1; r += 2) {
        const int next = r < r1 ? stride : 0;
        float ea[N], eb[N];
#pragma unroll
        for (int k = 0; k < N; ++k) ea[k] = !GUARD || c + 2 * k <= c1 ? q[2 * k] : 0.0f;
#pragma unroll
        for (int k = 0; k < N; ++k) eb[k] = !GUARD || c + 2 * k <= c1 ? q[next + 2 * k] : 0.0f;
        const float dy = fy - y;
        float u = expneg_hw(kap * (dy * dy));
        u = r + h <= r1 ? u : 0.0f;
        const float u1 = u * dy, u2 = u1 * dy;
        float A0 = 0.0f, A1 = 0.0f, A2 = 0.0f, B0 = 0.0f, B1 = 0.0f, B2 = 0.0f;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            A0 = __builtin_fmaf(ea[k], g0[k], A0);
            A1 = __builtin_fmaf(ea[k], g1[k], A1);
            A2 = __builtin_fmaf(ea[k], g2[k], A2);
            B0 = __builtin_fmaf(eb[k], g0[k], B0);
            B1 = __builtin_fmaf(eb[k], g1[k], B1);
            B2 = __builtin_fmaf(eb[k], g2[k], B2);
        }
        const float a0 = pair_lane<0>(u), b0 = pair_lane<1>(u);
        s.x = __builtin_fmaf(B0, b0, __builtin_fmaf(A0, a0, s.x));
        s.y = __builtin_fmaf(B1, b0, __builtin_fmaf(A1, a0, s.y));
        s.z = __builtin_fmaf(B0, pair_lane<1>(u1), __builtin_fmaf(A0, pair_lane<0>(u1), s.z));
        s.w = __builtin_fmaf(B2, b0, __builtin_fmaf(A2, a0, s.w));
        s.w = __builtin_fmaf(B0, pair_lane<1>(u2), __builtin_fmaf(A0, pair_lane<0>(u2), s.w));
        fy += 2.0f;
        q += 2 * stride;
    }
}

// The lane's sums in the same order from its own pixels alone, read from the image.
__device__ __noinline__ float4 gather_exact(const float* src, int W, float x, float y, float kap, int c0, int c1,
                                            int r0, int r1)
{
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll 1
    for (int cb = c0; cb <= c1; cb += 16) {
#pragma unroll 1
        for (int r = r0; r <= r1; r += 2) {
            float R[2][3] = {{0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f}}, u[2][3];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float dy = ((float)(r + j) + 0.5f) - y;
                u[j][0] = r + j <= r1 ? expneg_hw(kap * (dy * dy)) : 0.0f;
                u[j][1] = u[j][0] * dy;
                u[j][2] = u[j][1] * dy;
                if (r + j > r1) continue;
#pragma unroll 1
                for (int c = cb; c <= min(c1, cb + 15); c += 2) {
                    const float dx = ((float)c + 0.5f) - x;
                    const float v = expneg_hw(kap * (dx * dx)), v1 = v * dx;
                    const float e = src[(int64_t)(r + j) * W + c];
                    R[j][0] = __builtin_fmaf(e, v, R[j][0]);
                    R[j][1] = __builtin_fmaf(e, v1, R[j][1]);
                    R[j][2] = __builtin_fmaf(e, v1 * dx, R[j][2]);
                }
            }
            s.x = __builtin_fmaf(R[1][0], u[1][0], __builtin_fmaf(R[0][0], u[0][0], s.x));
            s.y = __builtin_fmaf(R[1][1], u[1][0], __builtin_fmaf(R[0][1], u[0][0], s.y));
            s.z = __builtin_fmaf(R[1][0], u[1][1], __builtin_fmaf(R[0][0], u[0][1], s.z));
            s.w = __builtin_fmaf(R[1][2], u[1][0], __builtin_fmaf(R[0][2], u[0][0], s.w));
            s.w = __builtin_fmaf(R[1][0], u[1][2], __builtin_fmaf(R[0][0], u[0][2], s.w));
        }
    }
    return s;
}

// Block gather.  A workgroup takes the particles of a 64 x 64 pixel block (gb x gb
// home blocks of the frame-1 positions) of one pair, NP at a time, sorted by
// diameter (a counting sort on LDS counters, so that a wave's patches are nearly
// equal).  For each frame in turn, the rectangle of dL/dJ or B^T dL/dJ that the
// particles' supports cover is staged in LDS (where it holds at most `cap` pixels,
// else it is read from global memory) and each particle's two lanes walk down its
// rows, every other column each.  The order of a particle's sums depends on its own
// support alone.
// Two lanes of contiguous work and one LDS word per pixel against eight or sixteen
// lanes with a row-factor vector of LDS per pixel: 64 pairs of 512^2 at 0.05 ppp, d
// about 2.5: 207 -> 117 us; 4 pairs of 2048^2 at 0.1 ppp, d to 6: 636 -> 377 us (from
// LDS before as well, one frame and 32-pixel block at a time, which also took an order
// of the frame-2 positions, 60 us), of which 85 came from leaving dL/dx1 and dL/dx2 in
// the home-block order instead of at the particles' own addresses.  Of the first, 20
// us are the sums and 28 us the staging; the rest are the particle arrays (seven
// reads and four writes at unrelated addresses) and the waits between the phases,
// which is why small workgroups do better: NP = 256 with room for four per CU 116 us,
// NP = 512 131 us; on the second batch, whose blocks hold 410 particles (two passes of
// 256), 507 and 459 us (before the home-block order of the results).  Straight from
// global memory (16-byte loads, one or two lanes per row) the first took 167-172 us:
// each lane's row is a cache line of its own.
// Particles may crowd, and one workgroup would take a full block's passes one after
// another: those of a home block past the first `most` are for the first n_rest
// workgroups, a segment of the home-block order at a time.  100 k particles of one pair in
// one place / in 32 x 32 pixels 4050 / 3270 -> 29 / 31 us, 64 pairs of 13 k 630 / 540 -> 153 /
// 165, in one row of pixels 135 -> 157; spread evenly 99 -> 100, 64 pairs of 3 k 29 -> 31
// (two copies of the passes in one kernel; one copy with both kinds of list in one loop
// 114 for 99, the further workgroups in a launch of their own 111, last in the grid 108).
constexpr int REGION_PAD = 32;          // floats past the region that a row's last reads may reach

// The particles of a pass.
template <int NP>
struct BlockLds {
    float4 pos[NP];          // x1, y1, x2, y2
    float4 par[NP];          // z, d, I0 (0: invalid), particle of the pair (as bits)
    int slot[NP];            // its place in the pair's home-block order
    uint32_t hist[64];
    int box[2][4];           // per frame: first column, first row, last column, last row
};

// The largest region: up to diameters of 12, with the particles of the larger pass within
// the 64 KB that a workgroup may have.
constexpr int REGION_SIDE_MAX = 108;
static_assert(sizeof(BlockLds<512>) + sizeof(float) * (REGION_SIDE_MAX * REGION_SIDE_MAX + REGION_PAD) <= 64 * 1024,
              "a workgroup's LDS");

// The particles of a home block past the first `most` in a segment of `most` places of the
// home-block order: where it holds any of them, its first particle is of the same block (at
// most `most` places before them), so that block alone is looked up.
struct Segment {
    int pair, first, end;       // places of the pair's order; none: first >= end
};

__device__ __forceinline__ Segment crowded_segment(const BwdArgs& a, int64_t n_span, int most, int64_t seg)
{
    Segment none{0, 0, 0};
    if (seg * most >= n_span) return none;
    const int64_t slot = seg * most;
    // the pair where even ones would have it, else searched for (64 pairs: 0.7 us)
    int p = min((int)((float)slot * ((float)a.n_pairs / (float)n_span)), a.n_pairs - 1);
    if (a.pairs[p].particle_offset > slot || a.pairs[min(p + 1, a.n_pairs - 1)].particle_offset <= slot)
        p = find_pair_by_particle(a.pairs, a.n_pairs, slot);
    const synthpix_pair P = a.pairs[p];
    const int64_t i = slot - P.particle_offset;
    if (i < 0 || i >= P.n_max) return none;
    const PairLayout L = a.order.L[p];
    const int64_t g = P.particle_offset + a.order.entries[L.entry_base + i];
    const int64_t b = L.tile_base + home_block(a.x1[g], a.y1[g], P.W, P.H, L.ntx, L.nty, a.order.log_block,
                                               a.order.log_block);
    const int64_t at = a.order.offset[b] - L.entry_base;        // its first place
    return {p, (int)max(i, at + most), (int)min(i + most, at + (int64_t)a.order.count[b])};
}

// A value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ int64_t uniform(int64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | lo);
}

// The passes over the `total` particles of pair p at the places o0 + k of the order's
// entries for the k below e0, o1 + k for the next below e1, and so on.
template <int NP>
__device__ __forceinline__ void gather_list(const BwdArgs& a, BlockLds<NP>& lds, float* region, int cap, int p,
                                            int64_t o0, int64_t o1, int64_t o2, int64_t o3, int e0, int e1, int e2,
                                            int total)
{
    auto& s_pos = lds.pos;
    auto& s_par = lds.par;
    auto& s_slot = lds.slot;
    auto& s_hist = lds.hist;
    auto& s_box = lds.box;
    const int t = (int)threadIdx.x, lane = t & 63, h = t & 1;
    const int W = uniform(a.pairs[p].W), H = uniform(a.pairs[p].H);
    const int64_t part0 = uniform(a.pairs[p].particle_offset), entry0 = uniform((int64_t)a.order.L[p].entry_base);
    const int64_t img = uniform(a.pairs[p].image_offset);
    for (int k0 = 0; k0 < total; k0 += NP) {
        if (t < 64) s_hist[t] = 0u;
        if (t < 8) s_box[t >> 2][t & 3] = (t & 2) ? -1 : 1 << 30;
        __syncthreads();
        const int n = min(NP, total - k0), k = k0 + t;
        float4 pos = make_float4(0.0f, 0.0f, 0.0f, 0.0f), par = make_float4(0.0f, 1.0f, 0.0f, 0.0f);
        int size = 0, place = 0;
        uint32_t rank = 0;
        int box[2][4] = {{1 << 30, 1 << 30, -1, -1}, {1 << 30, 1 << 30, -1, -1}};
        if (t < n) {
            const int64_t o = k < e0 ? o0 : k < e1 ? o1 : k < e2 ? o2 : o3;
            const int i = a.order.entries[o + k];
            place = (int)(o + k - entry0);
            const int64_t g = part0 + i;
            pos = make_float4(a.x1[g], a.y1[g], a.x2[g], a.y2[g]);
            const float d = a.d[g], I0 = a.I0[g];
            bool valid = (I0 > 0.0f) && (d > 0.0f);
            if (valid && !(d <= a.d_max)) {
                atomicOr(a.status, SP_STATUS_D_ABOVE_MAX);
                valid = false;
            }
            par = make_float4(a.z[g], d, valid ? I0 : 0.0f, __int_as_float(i));
            size = valid ? (int)__builtin_fminf(3.0f * d + 1.0f, 63.0f) : 0;
            rank = atomicAdd(&s_hist[size], 1u);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                int c0, c1, r0, r1;
                if (valid && support_box(f ? pos.z : pos.x, f ? pos.w : pos.y, d, W, H, c0, c1, r0, r1)) {
                    box[f][0] = c0;
                    box[f][1] = r0;
                    box[f][2] = c1;
                    box[f][3] = r1;
                }
            }
        }
        if ((t & ~63) < n) {                             // the wave has particles
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int v = __shfl_xor(box[f][m], o, 64);
                        box[f][m] = m < 2 ? min(box[f][m], v) : max(box[f][m], v);
                    }
            if (lane < 8) {
                int v = box[0][0];
#pragma unroll
                for (int m = 1; m < 8; ++m) v = lane == m ? box[m >> 2][m & 3] : v;
                if (lane & 2) atomicMax(&s_box[lane >> 2][lane & 3], v);
                else atomicMin(&s_box[lane >> 2][lane & 3], v);
            }
        }
        __syncthreads();
        // largest first: lane l scans size 63 - l
        if ((t & ~63) < n) {
            const uint32_t inc = wave_scan(s_hist[63 - lane]);
            const uint32_t above = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (62 - size), (int)inc);
            if (t < n) {
                const int slot = (int)((size < 63 ? above : 0u) + rank);
                s_pos[slot] = pos;
                s_par[slot] = par;
                s_slot[slot] = place;
            }
        }
#pragma unroll 1
        for (int f = 0; f < 2; ++f) {
            const float* __restrict__ src = a.grad + img + (int64_t)f * H * W;
            const int bc = uniform(s_box[f][0]), br = uniform(s_box[f][1]);
            const int bw = uniform(s_box[f][2]) - bc + 1, bh = uniform(s_box[f][3]) - br + 1;
            const int rs = (bw + 3) & ~3;                // a row's stride, whole 16-byte groups
            const bool any = bw > 0 && bh > 0;
            const bool staged = any && (int64_t)rs * bh <= cap;
            if (staged) {
                const int nq = rs >> 2;
                const float inv = 1.0f / (float)nq;
                const float* q0 = src + (int64_t)br * W + bc;
                for (int m = t; m < nq * bh; m += NP) {
                    const int r = (int)(((float)m + 0.5f) * inv);         // m / nq: both below 2^16
                    const int c = 4 * (m - r * nq);
                    glb_float* q = (glb_float*)q0 + ((int64_t)r * W + c);
                    vec4u v = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (bc + c + 3 < W) {
                        v = *(const __attribute__((address_space(1))) vec4u*)q;
                    } else {                             // the image's last columns
                        if (bc + c < W) v.x = q[0];
                        if (bc + c + 1 < W) v.y = q[1];
                        if (bc + c + 2 < W) v.z = q[2];
                    }
                    reinterpret_cast<float4*>(region)[m] = make_float4(v.x, v.y, v.z, v.w);
                }
                if (t < REGION_PAD) region[rs * bh + t] = 0.0f;
            }
            __syncthreads();
            for (int sl = t >> 1; sl < n; sl += NP / 2) {
                pos = s_pos[sl];
                par = s_par[sl];
                const bool valid = par.z > 0.0f;
                const float d = par.y, x = f ? pos.z : pos.x, y = f ? pos.w : pos.y;
                const float kap = 8.0f / (d * d);
                int c0 = 0, c1 = -1, r0 = 0, r1 = -1;
                const bool on = valid && support_box(x, y, d, W, H, c0, c1, r0, r1);
                const int w = on ? c1 - c0 + 1 : 0;
                c0 += h;
                float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (on) {
                    if (staged) {
                        lds_float* q = (lds_float*)region + (r0 - br) * rs + (c0 - bc);
#define SP_COLS(N_) gather_columns<N_, false>(q, rs, x, y, kap, c0, c1, r0, r1, h, s)
                        if (!__builtin_amdgcn_ballot_w64(w > 4)) SP_COLS(2);
                        else if (!__builtin_amdgcn_ballot_w64(w > 6)) SP_COLS(3);
                        else if (!__builtin_amdgcn_ballot_w64(w > 8)) SP_COLS(4);
                        else if (!__builtin_amdgcn_ballot_w64(w > 10)) SP_COLS(5);
                        else if (!__builtin_amdgcn_ballot_w64(w > 12)) SP_COLS(6);
                        else
#pragma unroll 1
                            for (int c = 0; c < w; c += 16)
                                gather_columns<8, false>(q + c, rs, x, y, kap, c0 + c, c1, r0, r1, h, s);
#undef SP_COLS
                    } else {
                        glb_float* q = (glb_float*)src + (int64_t)r0 * W + c0;
#pragma unroll 1
                        for (int c = 0; c < w; c += 16)
                            gather_columns<8, true>(q + c, W, x, y, kap, c0 + c, c1, r0, r1, h, s);
                    }
                    if (!__builtin_isfinite((s.x + s.y) + (s.z + s.w)))
                        s = gather_exact(src, W, x, y, kap, c0, c1, r0, r1);
                }
                s = make_float4(s.x + dpp<0xB1>(s.x), s.y + dpp<0xB1>(s.y), s.z + dpp<0xB1>(s.z),
                                s.w + dpp<0xB1>(s.w));
                // the two frames' sums meet in frame 2: frame 1 leaves its S0 and Sr in place
                // of its position, read by the particle's own two lanes alone
                ParticleGrads o{};
                if (valid) {
                    const float4 f0 = f ? make_float4(pos.x, 0.0f, 0.0f, pos.y) : s;
                    o = particle_grads(par.x, d, par.z, a.sheet_sigma, f0, s);
                }
                const int64_t g = part0 + __float_as_int(par.w);
                if (f == 0) {
                    reinterpret_cast<float*>(start_grads(a, p, s_slot[sl]))[h] = h ? o.gy1 : o.gx1;
                    if (h == 0) *reinterpret_cast<float2*>(&s_pos[sl]) = make_float2(s.x, s.w);
                } else {
                    (h ? a.gy2 : a.gx2)[part0 + s_slot[sl]] = h ? o.gy2 : o.gx2;
                    (h ? a.g_z : a.g_d)[g] = h ? o.gz : o.gd;
                    (h ? a.sheet : a.g_I0)[g] = h ? o.sheet : o.gI0;
                }
            }
            __syncthreads();
        }
    }
}

template <int NP>
__global__ void __launch_bounds__(NP)
bwd_gather_blocks(BwdArgs a, int64_t n_span, int most, unsigned n_rest, int gb, int ngx, int ngy, int cap)
{
    extern __shared__ __align__(16) float region[];
    __shared__ BlockLds<NP> lds;
    if (blockIdx.x < n_rest) {
        // each wave finds them for itself, the same in every one: the passes' barriers meet
        const int64_t segs = (n_span + most - 1) / most;
        for (int64_t s0 = blockIdx.x; s0 < segs; s0 += 64 * (int64_t)n_rest) {
            const Segment mine = crowded_segment(a, n_span, most, s0 + (int64_t)n_rest * (threadIdx.x & 63));
            for (unsigned long long left = __builtin_amdgcn_ballot_w64(mine.first < mine.end); left != 0;
                 left &= left - 1) {
                const int l = __builtin_ctzll(left), p = __builtin_amdgcn_readlane(mine.pair, l);
                const int first = __builtin_amdgcn_readlane(mine.first, l);
                const int total = __builtin_amdgcn_readlane(mine.end, l) - first;
                const int64_t o = uniform((int64_t)a.order.L[p].entry_base) + first;
                gather_list<NP>(a, lds, region, cap, p, o, o, o, o, total, total, total, total);
            }
        }
        return;
    }
    const int64_t bid = xcd_contiguous(blockIdx.x - n_rest, gridDim.x - n_rest);
    const int p = (int)(bid / ((int64_t)ngx * ngy));
    const int rem = (int)(bid - (int64_t)p * ngx * ngy);
    const int gy = rem / ngx, gx = rem - gy * ngx;
    const int ntx = uniform(a.order.L[p].ntx), nty = uniform(a.order.L[p].nty);
    if (gb * gx >= ntx || gb * gy >= nty) return;          // the whole workgroup, before its barriers
    // the blocks' lists; blocks are numbered in strips of four block rows, column by
    // column inside a strip, odd strips right to left
    int64_t off[4];
    int end[4], total = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int bx = gb * gx + (q & 1), by = gb * gy + (q >> 1);
        off[q] = 0;
        if (q < gb * gb && bx < ntx && by < nty) {
            const int s0 = by & ~3, rows = min(4, nty - s0);
            const int64_t b = a.order.L[p].tile_base + (int64_t)s0 * ntx +
                              ((s0 & 4) ? ntx - 1 - bx : bx) * rows + (by - s0);
            off[q] = uniform(a.order.offset[b] - total);
            total += min(uniform((int)a.order.count[b]), most);
        }
        end[q] = total;
    }
    gather_list<NP>(a, lds, region, cap, p, off[0], off[1], off[2], off[3], end[0], end[1], end[2], total);
}

// ------------------------------------------------------------------ row gather

// One frame's sums of a particle by eight lanes, added in the block gather's order: lane
// 2 j + h forms the row sums of every fourth row from row j on over the columns c, c + 2,
// .. (c the first column of parity h), and the particle's sums pass between the lanes of
// rows 0 and 2 of each four, which add their own and the next row as gather_columns does.
// Only the support's own pixels are read.
template <int N>
__device__ __forceinline__ void row_block(const float* __restrict__ src, int W, float x, float y, float kap, int c,
                                          int c1, int r0, int r1, int j, float4& s)
{
    float g0[N], g1[N], g2[N];
    const float fx = (float)c + 0.5f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const float dx = (fx + (float)(2 * k)) - x;
        const float v = expneg_hw(kap * (dx * dx));
        g0[k] = c + 2 * k <= c1 ? v : 0.0f;
        g1[k] = g0[k] * dx;
        g2[k] = g1[k] * dx;
    }
#pragma unroll 1
    for (int rb = r0; rb <= r1; rb += 4) {
        const int r = rb + j;
        const float* q = src + ((int64_t)r * W + c);
        float e[N];
#pragma unroll
        for (int k = 0; k < N; ++k) e[k] = r <= r1 && c + 2 * k <= c1 ? q[2 * k] : 0.0f;
        const float dy = ((float)r + 0.5f) - y;
        float u = expneg_hw(kap * (dy * dy));
        u = r <= r1 ? u : 0.0f;
        const float u1 = u * dy, u2 = u1 * dy;
        float A0 = 0.0f, A1 = 0.0f, A2 = 0.0f;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            A0 = __builtin_fmaf(e[k], g0[k], A0);
            A1 = __builtin_fmaf(e[k], g1[k], A1);
            A2 = __builtin_fmaf(e[k], g2[k], A2);
        }
        // the next row's, from two lanes on (row_shl:2)
        const float B0 = dpp<0x102>(A0), B1 = dpp<0x102>(A1), B2 = dpp<0x102>(A2);
        const float v = dpp<0x102>(u), v1 = dpp<0x102>(u1), v2 = dpp<0x102>(u2);
#pragma unroll
        for (int step = 0; step < 2; ++step) {
            s.x = __builtin_fmaf(B0, v, __builtin_fmaf(A0, u, s.x));
            s.y = __builtin_fmaf(B1, v, __builtin_fmaf(A1, u, s.y));
            s.z = __builtin_fmaf(B0, v1, __builtin_fmaf(A0, u1, s.z));
            s.w = __builtin_fmaf(B2, v, __builtin_fmaf(A2, u, s.w));
            s.w = __builtin_fmaf(B0, v2, __builtin_fmaf(A0, u2, s.w));
            // on to the lanes of rows 2 and 3 (row_shr:4) and back (row_shl:4)
            if (step == 0) s = make_float4(dpp<0x114>(s.x), dpp<0x114>(s.y), dpp<0x114>(s.z), dpp<0x114>(s.w));
            else s = make_float4(dpp<0x104>(s.x), dpp<0x104>(s.y), dpp<0x104>(s.z), dpp<0x104>(s.w));
        }
    }
}

// The sums, in lane 0 of the eight.
__device__ __forceinline__ float4 row_sums(const float* __restrict__ src, int W, float x, float y, float kap, int c0,
                                           int c1, int r0, int r1, int lane)
{
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int h = lane & 1, w = c1 - c0 + 1;
#define SP_ROWS(N_) row_block<N_>(src, W, x, y, kap, c0 + h + c, c1, r0, r1, lane >> 1, s)
#pragma unroll 1
    for (int c = 0; c < w; c += 16) {
        if (!__builtin_amdgcn_ballot_w64(w - c > 4)) SP_ROWS(2);
        else if (!__builtin_amdgcn_ballot_w64(w - c > 8)) SP_ROWS(4);
        else if (!__builtin_amdgcn_ballot_w64(w - c > 12)) SP_ROWS(6);
        else SP_ROWS(8);
    }
#undef SP_ROWS
    return make_float4(s.x + dpp<0xB1>(s.x), s.y + dpp<0xB1>(s.y), s.z + dpp<0xB1>(s.z), s.w + dpp<0xB1>(s.w));
}

// Row gather, for batches with too few blocks or particles for the block gather: the same
// sums in the same order, so a particle's gradients have the same bits whatever batch it
// comes in.  Eight lanes per particle read its support from global memory; BOTH: sixteen,
// one half for each frame.
// Bound by the latency of its loads for few particles, by the rows' cache lines (one per
// row and load) and VALU for many.  Against bwd_gather<0, 32, 8 or 16>, which added in an
// order of its own: one pair of 256^2 at 0.05 ppp, d about 2.5, 11.6 -> 8.3 us, of 512^2
// with d 2 to 6 14.6 -> 18.2 us; 64 of 512^2 at 0.005 / 0.01 ppp 43.6 / 64.6 -> 42.0 /
// 62.9 us; 4 of 2048^2, d 2 to 6, 65 / 112 -> 76 / 122 us.  The next rows' pixels loaded
// ahead: 67 us for 62.9 (registers); eight rows at a time by sixteen lanes: 90 us.
template <bool BOTH>
__global__ void __launch_bounds__(256)
bwd_gather_rows(BwdArgs a, int64_t n_span)
{
    constexpr int G = BOTH ? 16 : 8;
    const int lane = threadIdx.x % G;
    const int64_t g0 = (int64_t)xcd_contiguous(blockIdx.x, gridDim.x) * (256 / G);
    const int64_t slot = g0 + threadIdx.x / G;          // of the home-block order
    if (slot >= n_span) return;
    const int p = find_pair_from(a.pairs, a.n_pairs, g0, slot);
    const synthpix_pair P = a.pairs[p];
    const int64_t i = slot - P.particle_offset;
    if (i < 0 || i >= P.n_max) {
        // a slot in no pair's particle range (a gap of the packed arrays): zero gradients
        if (lane == 0) {
            a.g_x1[slot] = 0.0f;
            a.g_y1[slot] = 0.0f;
            a.g_z[slot] = 0.0f;
            a.g_d[slot] = 0.0f;
            a.g_I0[slot] = 0.0f;
        }
        return;
    }
    const int64_t g = P.particle_offset + a.order.entries[a.order.L[p].entry_base + i];
    const float z = a.z[g], d = a.d[g], I0 = a.I0[g];
    bool valid = (I0 > 0.0f) && (d > 0.0f);
    if (valid && !(d <= a.d_max)) {
        if (lane == 0) atomicOr(a.status, SP_STATUS_D_ABOVE_MAX);
        valid = false;
    }
    const float kap = 8.0f / (d * d);
    auto frame = [&](int f) {
        const float x = f ? a.x2[g] : a.x1[g], y = f ? a.y2[g] : a.y1[g];
        int c0, c1, r0, r1;
        if (!valid || !support_box(x, y, d, P.W, P.H, c0, c1, r0, r1)) return make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return row_sums(a.grad + P.image_offset + (int64_t)f * P.H * P.W, P.W, x, y, kap, c0, c1, r0, r1, lane & 7);
    };
    const float4 s1 = frame(BOTH ? lane >> 3 : 0);
    float4 s2;
    if constexpr (BOTH) s2 = make_float4(dpp<0x108>(s1.x), dpp<0x108>(s1.y), dpp<0x108>(s1.z), dpp<0x108>(s1.w));
    else s2 = frame(1);
    if (lane != 0) return;
    ParticleGrads o{};
    if (valid) o = particle_grads(z, d, I0, a.sheet_sigma, s1, s2);
    *start_grads(a, p, i) = make_float2(o.gx1, o.gy1);
    a.g_z[g] = o.gz;
    a.g_d[g] = o.gd;
    a.g_I0[g] = o.gI0;
    a.gx2[slot] = o.gx2;
    a.gy2[slot] = o.gy2;
    a.sheet[g] = o.sheet;
}

// Zero gradients of the slots in no pair's particle range (gaps of the packed arrays).
__global__ void __launch_bounds__(256) bwd_gaps(BwdArgs a, int64_t n_span)
{
    const int64_t g0 = (int64_t)blockIdx.x * 256, g = g0 + threadIdx.x;
    if (g >= n_span) return;
    const int p = find_pair_from(a.pairs, a.n_pairs, g0, g);
    const int64_t i = g - a.pairs[p].particle_offset;
    if (i >= 0 && i < a.pairs[p].n_max) return;
    a.g_x1[g] = 0.0f;
    a.g_y1[g] = 0.0f;
    a.g_z[g] = 0.0f;
    a.g_d[g] = 0.0f;
    a.g_I0[g] = 0.0f;
}

// One input column x of a strip of the per-pixel pass: its SH + 2b rows from
// Y0 - b (zeros outside the image) blurred vertically into vb[.][k].  MSE: the
// values are scale (J - T); returns the float64 sum of (J - T)^2 over the
// strip's own rows (Y0 .. Y0 + SH - 1, inside the image), 0 otherwise.
template <int B, bool MSE, int SH, int VW>
__device__ __forceinline__ double blur_column(const BwdArgs& a, int64_t base, int W, int H, int x, int Y0, int k,
                                              float (*vb)[VW])
{
    const bool xin = x >= 0 && x < W;
    float g[SH + 2 * B];
    double sq = 0.0;
#pragma unroll
    for (int r = 0; r < SH + 2 * B; ++r) {
        const int y = Y0 - B + r;
        const bool in = xin && y >= 0 && y < H;
        if constexpr (MSE) {
            const int64_t i = base + (int64_t)(in ? y : 0) * W + (in ? x : 0);
            const float j = in ? a.J[i] : 0.0f, tv = in ? a.T[i] : 0.0f;
            g[r] = a.mse_scale * (j - tv);
            if (in && r >= B && r < SH + B) {
                const double e = (double)j - (double)tv;
                sq = __builtin_fma(e, e, sq);
            }
        } else {
            g[r] = in ? a.grad[base + (int64_t)y * W + x] : 0.0f;
        }
    }
#pragma unroll
    for (int r = 0; r < SH; ++r) {
        float v = 0.0f;
#pragma unroll
        for (int q = 0; q <= 2 * B; ++q) v = __builtin_fmaf(a.blur_w[q], g[r + q], v);
        vb[r][k] = v;
    }
    return sq;
}

// e = B^T dL/dJ, once per pixel: the zero-padded blur's adjoint sums
// w_k dL/dJ(q + k) over the taps that land inside the image (the same blur,
// its weights being symmetric).  A workgroup owns a strip of SH output rows
// by 256 output columns of one frame: each thread takes one column (the first
// 2b threads also one of the b apron columns on either side), issues its
// SH + 2b loads together and blurs them vertically in registers; the rows then
// pass through LDS for the horizontal taps.  Rows of 256 floats keep the reads
// and writes in whole 1 KB segments, and images 256 k pixels wide split into
// whole strips.  Workgroups are numbered (pair, frame, strip row, strip
// column) over the batch's largest pair, XCD-contiguously.
// MSE: dL/dJ is the mean-squared-difference loss's gradient scale (J - T),
// formed from the images and the target as they are read (the same binary32
// products synthpix_mse_grad stores), and with loss_part each workgroup also
// writes the float64 sum of (J - T)^2 over the pixels of its strip (every
// pixel lies in exactly one strip); b = 0 is then a plain pass.
template <int B, bool MSE>
__global__ void __launch_bounds__(256)
bwd_blur_grad(BwdArgs a, int nsx, int nsy)
{
    constexpr int SH = blur_strip_rows(MSE), VW = 256 + 2 * B;
    __shared__ float vb[SH][VW];
    __shared__ double red[MSE ? 256 : 1];
    const int64_t bid = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t per_pair = (int64_t)2 * nsx * nsy;
    const int p = (int)(bid / per_pair);
    int rem = (int)(bid - (int64_t)p * per_pair);
    const int f = rem / (nsx * nsy);
    rem -= f * nsx * nsy;
    const int sy = rem / nsx, sx = rem - sy * nsx;
    const int H = a.pairs[p].H, W = a.pairs[p].W;
    const int X0 = sx * 256, Y0 = sy * SH;
    if (X0 >= W || Y0 >= H) {                    // the whole workgroup, before its barrier
        if (MSE && a.loss_part && threadIdx.x == 0) a.loss_part[bid] = 0.0;
        return;
    }
    const int64_t base = a.pairs[p].image_offset + (int64_t)f * H * W;
    const int t = (int)threadIdx.x;
    // vb column k holds input column X0 - b + k
    double sq = 0.0;
    const int nc = t < 2 * B ? 2 : 1;
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {             // own column, then an apron column
        const int xc = c == 0 ? X0 + t : t < B ? X0 - B + t : X0 + 256 + (t - B);
        const int k = c == 0 ? B + t : t < B ? t : 256 + t;
        const double s2 = blur_column<B, MSE, SH, VW>(a, base, W, H, xc, Y0, k, vb);
        if (c == 0) sq = s2;
    }
    if (MSE && a.loss_part) {
        red[t] = sq;
        __syncthreads();
        for (int w = 128; w >= 1; w >>= 1) {
            if (t < w) red[t] += red[t + w];
            __syncthreads();
        }
        if (t == 0) a.loss_part[bid] = red[0];
    }
    __syncthreads();
    const int x = X0 + t;
    if (x >= W) return;
    const int nr = H - Y0 < SH ? H - Y0 : SH;
#pragma unroll 4
    for (int r = 0; r < nr; ++r) {
        float e = 0.0f;
#pragma unroll
        for (int q = 0; q <= 2 * B; ++q) e = __builtin_fmaf(a.blur_w[q], vb[r][t + q], e);
        a.eblur[base + (int64_t)(Y0 + r) * W + x] = e;
    }
}

// ------------------------------------------------------------------ flow adjoint

struct Sample {
    float2 val;
    float2 jx, jy;        // dU/dpx, dU/dpy (zero along clamped axes)
    int i0, j0;
    float fx, fy;
};

// Value bit-identical to sample_flow, plus Jacobian and node weights.
__device__ __forceinline__ Sample sample_jac(const FlowView& fv, const FlowWin& fw, lds_vec2* lds, float px, float py)
{
    Sample o;
    const float gxr = px * fv.sx - 0.5f;
    const float gyr = py * fv.sy - 0.5f;
    const FlowCell cell = flow_cell(fv, px, py);
    const int i0 = cell.i0, j0 = cell.j0;
    const float fx = cell.fx, fy = cell.fy;
    float4 r0, r1;
    cell_nodes(fv, cell, in_window(cell, fw), fw, lds, r0, r1);
    const float2 A = make_float2(r0.x, r0.y), Bn = make_float2(r0.z, r0.w);
    const float2 C = make_float2(r1.x, r1.y), E = make_float2(r1.z, r1.w);
    {
        const float top = __builtin_fmaf(fx, Bn.x - A.x, A.x);
        const float bot = __builtin_fmaf(fx, E.x - C.x, C.x);
        o.val.x = __builtin_fmaf(fy, bot - top, top);
    }
    {
        const float top = __builtin_fmaf(fx, Bn.y - A.y, A.y);
        const float bot = __builtin_fmaf(fx, E.y - C.y, C.y);
        o.val.y = __builtin_fmaf(fy, bot - top, top);
    }
    const float inx = (gxr > 0.0f && gxr < (float)(fv.Gw - 1)) ? fv.sx : 0.0f;
    const float iny = (gyr > 0.0f && gyr < (float)(fv.Gh - 1)) ? fv.sy : 0.0f;
    o.jx.x = ((1.0f - fy) * (Bn.x - A.x) + fy * (E.x - C.x)) * inx;
    o.jx.y = ((1.0f - fy) * (Bn.y - A.y) + fy * (E.y - C.y)) * inx;
    o.jy.x = ((1.0f - fx) * (C.x - A.x) + fx * (E.x - Bn.x)) * iny;
    o.jy.y = ((1.0f - fx) * (C.y - A.y) + fx * (E.y - Bn.y)) * iny;
    o.i0 = i0;
    o.j0 = j0;
    o.fx = fx;
    o.fy = fy;
    return o;
}

// Per-particle accumulation of node contributions, merged while consecutive
// samples stay in one grid cell, flushed as 64-bit fixed-point atomic adds
// (integer sums: the result does not depend on their order).  A run is flushed
// as soon as the sample leaves its cell (holding the two runs before it back,
// so that lanes flush together, took 40 more registers and a wave per SIMD).
struct CellRun {
    int i0 = -1, j0 = 0;
    float acc[8];
};

struct NodeRun {
    CellRun cur;
    int Gw;
    double scale;         // 2^e; 0 when the flow gradient is not accumulated
    // the workgroup's LDS window of node sums (rows wi0 .., cols wj0 .., wh x ww
    // nodes, (u, v) interleaved); nodes outside it become overflow records
    unsigned long long* win;
    int wi0, wj0, wh, ww;
    GridRecord* ovf;      // the workgroup's overflow records (global memory)
    unsigned* n_ovf;      // their count (LDS)
    // grid cells this lane has added to
    int ti0 = 1 << 30, tj0 = 1 << 30, ti1 = -1, tj1 = -1;

    __device__ void add_node(int ni, int nj, int c, unsigned long long q)
    {
        const int li = ni - wi0, lj = nj - wj0;
        if ((unsigned)li < (unsigned)wh && (unsigned)lj < (unsigned)ww) {
            atomicAdd(win + 2 * (li * ww + lj) + c, q);
        } else {
            const unsigned k = atomicAdd(n_ovf, 1u);
            if (k < GRID_OVF_CAP) ovf[k] = GridRecord{2 * (ni * Gw + nj) + c, 0u, q};
        }
    }

    __device__ void flush(const CellRun& r)
    {
        if (r.i0 < 0) return;
        ti0 = min(ti0, r.i0);
        ti1 = max(ti1, r.i0);
        tj0 = min(tj0, r.j0);
        tj1 = max(tj1, r.j0);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float v = r.acc[2 * n + c];
                if (v != 0.0f)
                    add_node(r.i0 + (n >> 1), r.j0 + (n & 1), c,
                             (unsigned long long)(long long)__builtin_rint((double)v * scale));
            }
        }
    }

    __device__ void finish() { flush(cur); }

    __device__ void add(const Sample& s, float ku, float kv)
    {
        if (scale == 0.0) return;
        if (s.i0 != cur.i0 || s.j0 != cur.j0) {
            flush(cur);
            cur.i0 = s.i0;
            cur.j0 = s.j0;
#pragma unroll
            for (int k = 0; k < 8; ++k) cur.acc[k] = 0.0f;
        }
        const float w[4] = {(1.0f - s.fx) * (1.0f - s.fy), s.fx * (1.0f - s.fy), (1.0f - s.fx) * s.fy, s.fx * s.fy};
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            cur.acc[2 * n] = __builtin_fmaf(w[n], ku, cur.acc[2 * n]);
            cur.acc[2 * n + 1] = __builtin_fmaf(w[n], kv, cur.acc[2 * n + 1]);
        }
    }
};

// Back-propagate one sample with upstream (ku, kv); J^T k in (bx, by).
__device__ __forceinline__ void sample_back(NodeRun& run, const Sample& s, float ku, float kv, float& bx, float& by)
{
    run.add(s, ku, kv);
    bx = s.jx.x * ku + s.jx.y * kv;
    by = s.jy.x * ku + s.jy.y * kv;
}

// One substep's adjoint from its start (px, py): (gpx, gpy) becomes the gradient with
// respect to the start.  RK4 keeps the later three stages' samples from the forward
// walk to the sweep; the first is taken again, as all four leave no registers for
// four waves per SIMD (4 pairs of 2048^2, 8 substeps: all four 431 us, three 327,
// two 334, none 346; 64 of 512^2, 4 substeps: 101 / 102 / 105 / 110).
template <bool RK4>
__device__ __forceinline__ void substep_adjoint(const FlowView& fv, const FlowWin& fw, lds_vec2* lds, NodeRun& run,
                                                float px, float py, float h, float hh, float& gpx, float& gpy)
{
    if constexpr (!RK4) {
        float bx, by;
        sample_back(run, sample_jac(fv, fw, lds, px, py), h * gpx, h * gpy, bx, by);
        gpx += bx;
        gpy += by;
        return;
    }
    const float2 k1 = sample_flow(fv, fw, lds, px, py);
    const Sample s2 = sample_jac(fv, fw, lds, __builtin_fmaf(hh, k1.x, px), __builtin_fmaf(hh, k1.y, py));
    const Sample s3 = sample_jac(fv, fw, lds, __builtin_fmaf(hh, s2.val.x, px), __builtin_fmaf(hh, s2.val.y, py));
    const Sample s4 = sample_jac(fv, fw, lds, __builtin_fmaf(h, s3.val.x, px), __builtin_fmaf(h, s3.val.y, py));
    const float c = h / 6.0f;
    float b4x, b4y, b3x, b3y, b2x, b2y, b1x, b1y;
    sample_back(run, s4, c * gpx, c * gpy, b4x, b4y);
    sample_back(run, s3, 2.0f * c * gpx + h * b4x, 2.0f * c * gpy + h * b4y, b3x, b3y);
    sample_back(run, s2, 2.0f * c * gpx + hh * b3x, 2.0f * c * gpy + hh * b3y, b2x, b2y);
    sample_back(run, sample_jac(fv, fw, lds, px, py), c * gpx + hh * b2x, c * gpy + hh * b2y, b1x, b1y);
    gpx += ((b1x + b2x) + b3x) + b4x;
    gpy += ((b1y + b2y) + b3y) + b4y;
}

// Words of the fixed-point scale block in the workspace.
enum { SC_G2MAX = 0, SC_LIP = 1, SC_EXP = 2, SC_STATE = 3 };
enum { SC_NONE = 0, SC_VALID = 1, SC_NONFINITE = 2 };

// Reverse sweep of every particle: final position gradient (frame 1's
// plus the sweep's, to g_x1, g_y1) and node sums into the fixed-point grid.  CK checkpoints of the
// trajectory are kept, one every L = ceil(substeps / CK) substeps; each segment
// is recomputed into SK >= L slots during the sweep.
// The grid nodes around the workgroup's particles are copied to LDS, so that the
// samples of neighbouring lanes do not go through the vector cache line by line, and
// the box of the nodes to write out follows from the cells added to instead of a
// search of the window.  4 pairs of 2048^2 at 0.1 ppp, RK4 x 8: 386 -> 327 us (the
// copy 353, the box 346, the kept samples 327) and, with dL/dx1 and dL/dx2 read in the
// home-block order, 308; 64 of 512^2 at 0.05 ppp, RK4 x 4: 112 -> 98 us.  Without the
// node sums it would take 281 and 89 us: what remains is VALU work and the particle
// arrays at unrelated addresses.
// The integrators are apart, as RK4's kept samples cost Euler its registers (spills at 1,
// 8 and more than 16 substeps): 64 of 512^2, Euler x 12 / 24 / 48 105 / 188 / 483 -> 86 /
// 159 / 291 us (before the kept samples 117 / 169 / 367), RK4 x 8 / 16 / 33 160 / 293 /
// 844 -> 156 / 289 / 693.
constexpr int ADJ_FLOW_NODES = 896;     // LDS copy of grid nodes: 7 KB, with which four workgroups still share a CU
constexpr int ADJ_FLOW_MARGIN = 4;      // cells around the particles' starting ones

template <int CK, int SK, bool RK4>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CK <= 8 ? 4 : 3)))
bwd_advect(BwdArgs a, synthpix_advect_params ap)
{
    __shared__ __align__(16) unsigned long long win[2 * WIN_NODES];
    __shared__ vec2f s_flow[ADJ_FLOW_NODES];
    __shared__ int s_box[4][4];
    __shared__ unsigned s_novf;
    // workgroup -> (pair, 256-particle chunk of the pair's ordered particles)
    const int64_t wg = xcd_contiguous(blockIdx.x, gridDim.x);
    int p = 0;
    {
        int lo = 0, hi = a.n_pairs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.grid.wg_base[mid] <= wg) lo = mid;
            else hi = mid - 1;
        }
        p = lo;
    }
    const synthpix_pair P = a.pairs[p];
    const int64_t chunk = wg - a.grid.wg_base[p];
    int64_t i = chunk * 256 + threadIdx.x;
    int64_t g = -1;
    const int64_t place = i;
    bool live = false;
    float gpx = 0.0f, gpy = 0.0f, px = 0.0f, py = 0.0f;
    if (i < P.n_max) {
        // slots follow the home-block order: neighbouring lanes sample, and add
        // into, neighbouring grid cells
        gpx = a.gx2[P.particle_offset + i];      // stored in that order
        gpy = a.gy2[P.particle_offset + i];
        if (a.order.entries) i = a.order.entries[a.order.L[p].entry_base + i];
        g = P.particle_offset + i;
        px = a.x1[g];
        py = a.y1[g];
        live = (gpx != 0.0f || gpy != 0.0f) && __builtin_isfinite(px) && __builtin_isfinite(py);
    }
    NodeRun run;
    run.Gw = P.Gw;
    run.scale = a.scale[SC_STATE] == SC_VALID ? __builtin_ldexp(1.0, (int)a.scale[SC_EXP]) : 0.0;
    const FlowView fv = flow_view(P, a.flow);

    // window: the box of the live particles' starting cells, grown on every side
    // by as many cells as the LDS window holds (at least one)
    int bi0 = 1 << 30, bj0 = 1 << 30, bi1 = -1, bj1 = -1;
    if (live) {
        const float gx = __builtin_fminf(__builtin_fmaxf(px * fv.sx - 0.5f, 0.0f), (float)(fv.Gw - 1));
        const float gy = __builtin_fminf(__builtin_fmaxf(py * fv.sy - 0.5f, 0.0f), (float)(fv.Gh - 1));
        bj0 = bj1 = (int)gx;
        bi0 = bi1 = (int)gy;
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
    if (threadIdx.x == 0) s_novf = 0u;
    __syncthreads();
    bi0 = min(min(s_box[0][0], s_box[1][0]), min(s_box[2][0], s_box[3][0]));
    bj0 = min(min(s_box[0][1], s_box[1][1]), min(s_box[2][1], s_box[3][1]));
    bi1 = max(max(s_box[0][2], s_box[1][2]), max(s_box[2][2], s_box[3][2])) + 1;
    bj1 = max(max(s_box[0][3], s_box[1][3]), max(s_box[2][3], s_box[3][3])) + 1;
    const bool any = bi1 >= bi0 && run.scale != 0.0;
    int m = 0;                                   // margin in cells
    if (any) {
        const int h0 = bi1 - bi0 + 1, w0 = bj1 - bj0 + 1;
        m = 1;
        while ((h0 + 2 * (m + 1)) * (w0 + 2 * (m + 1)) <= WIN_NODES) ++m;
        if (h0 + 2 * m > WIN_NODES || (h0 + 2 * m) * (w0 + 2 * m) > WIN_NODES) m = 0;
    }
    const int wh = any ? bi1 - bi0 + 1 + 2 * m : 0, ww = any ? bj1 - bj0 + 1 + 2 * m : 0;
    const bool use_win = any && wh * ww <= WIN_NODES;
    run.win = win;
    run.wi0 = bi0 - m;
    run.wj0 = bj0 - m;
    run.wh = use_win ? wh : 0;                   // no window: every node becomes a record
    run.ww = ww;
    run.ovf = a.grid.ovf + wg * GRID_OVF_CAP;
    run.n_ovf = &s_novf;
    if (use_win) {
        for (int k = threadIdx.x; k < wh * ww; k += 256) reinterpret_cast<uint4*>(win)[k] = make_uint4(0u, 0u, 0u, 0u);
    }
    // the grid nodes around the starting cells, for the samples
    FlowWin fw = NO_WIN;
    lds_vec2* lds = (lds_vec2*)s_flow;
    if (bi1 >= bi0) {
        const int i0 = __builtin_amdgcn_readfirstlane(max(bi0 - ADJ_FLOW_MARGIN, 0));
        const int j0 = __builtin_amdgcn_readfirstlane(max(bj0 - ADJ_FLOW_MARGIN, 0));
        const int nh = __builtin_amdgcn_readfirstlane(min(bi1 + ADJ_FLOW_MARGIN, P.Gh - 1)) - i0 + 1;
        const int nw = __builtin_amdgcn_readfirstlane(min(bj1 + ADJ_FLOW_MARGIN, P.Gw - 1)) - j0 + 1;
        if ((int64_t)nh * nw <= ADJ_FLOW_NODES) {
            const vec2f* F = reinterpret_cast<const vec2f*>(fv.F) + (int64_t)i0 * P.Gw + j0;
            const float inv = 1.0f / (float)nw;
            for (int k = threadIdx.x; k < nh * nw; k += 256) {
                const int row = (int)(((float)k + 0.5f) * inv);          // k / nw: both below 2^10
                s_flow[k] = F[(int64_t)row * P.Gw + (k - row * nw)];
            }
            fw = FlowWin{i0, j0, nh, nw};
        }
    }
    __syncthreads();

    if (live) {
        const int S = ap.substeps;
        const float h = ap.dt / (float)S;
        const float hh = h * 0.5f;
        const int L = (S + CK - 1) / CK;
        const int nseg = (S + L - 1) / L;
        float cpx[CK], cpy[CK];
        float qx = px, qy = py;
        for (int s = 0; s < S; ++s) {
            if (s % L == 0) {
                cpx[s / L] = qx;
                cpy[s / L] = qy;
            }
            if (s + 1 < S) substep(fv, fw, lds, qx, qy, h, hh, RK4 ? SP_RK4 : SP_EULER);
        }
        if constexpr (SK == 1) {
            // S <= CK: every substep's start is a checkpoint, the sweep walks them
            // (no segment slots, whose runtime indexing would live in scratch)
            for (int seg = nseg - 1; seg >= 0; --seg)
                substep_adjoint<RK4>(fv, fw, lds, run, cpx[seg], cpy[seg], h, hh, gpx, gpy);
        } else {
            float spx[SK], spy[SK];
            for (int seg = nseg - 1; seg >= 0; --seg) {
                const int s0 = seg * L;
                const int len = (S - s0) < L ? (S - s0) : L;
                spx[0] = cpx[seg];
                spy[0] = cpy[seg];
                for (int k = 1; k < len; ++k) {
                    float tx = spx[k - 1], ty = spy[k - 1];
                    substep(fv, fw, lds, tx, ty, h, hh, RK4 ? SP_RK4 : SP_EULER);
                    spx[k] = tx;
                    spy[k] = ty;
                }
                for (int k = len - 1; k >= 0; --k)
                    substep_adjoint<RK4>(fv, fw, lds, run, spx[k], spy[k], h, hh, gpx, gpy);
            }
        }
        run.finish();
    }
    if (g >= 0) {
        const float2 b = *start_grads(a, p, place);
        a.g_x1[g] = live ? b.x + gpx : b.x;
        a.g_y1[g] = live ? b.y + gpy : b.y;
    }
    __syncthreads();

    // the window nodes of the cells added to, then their sums into this workgroup's
    // partial (rows of the box, (u, v) interleaved) and the header
    int ti0 = run.ti0, tj0 = run.tj0, ti1 = run.ti1, tj1 = run.tj1;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        ti0 = min(ti0, __shfl_xor(ti0, o, 64));
        tj0 = min(tj0, __shfl_xor(tj0, o, 64));
        ti1 = max(ti1, __shfl_xor(ti1, o, 64));
        tj1 = max(tj1, __shfl_xor(tj1, o, 64));
    }
    __syncthreads();                             // s_box is reused
    if ((threadIdx.x & 63) == 0) {
        s_box[threadIdx.x >> 6][0] = ti0;
        s_box[threadIdx.x >> 6][1] = tj0;
        s_box[threadIdx.x >> 6][2] = ti1;
        s_box[threadIdx.x >> 6][3] = tj1;
    }
    __syncthreads();
    ti0 = max(min(min(s_box[0][0], s_box[1][0]), min(s_box[2][0], s_box[3][0])) - run.wi0, 0);
    tj0 = max(min(min(s_box[0][1], s_box[1][1]), min(s_box[2][1], s_box[3][1])) - run.wj0, 0);
    ti1 = min(max(max(s_box[0][2], s_box[1][2]), max(s_box[2][2], s_box[3][2])) + 1 - run.wi0, run.wh - 1);
    tj1 = min(max(max(s_box[0][3], s_box[1][3]), max(s_box[2][3], s_box[3][3])) + 1 - run.wj0, ww - 1);
    const bool some = ti1 >= ti0 && tj1 >= tj0;
    const int th = some ? ti1 - ti0 + 1 : 0, tw = some ? tj1 - tj0 + 1 : 0;
    unsigned long long* part = a.grid.part + wg * (2 * WIN_NODES);
    const float inv_tw = 1.0f / (float)tw;
    for (int k = threadIdx.x; k < th * tw; k += 256) {
        const int r = (int)(((float)k + 0.5f) * inv_tw), c = k - r * tw;     // k / tw: both below 2^12
        const int src = (ti0 + r) * ww + (tj0 + c);
        part[2 * k] = win[2 * src];
        part[2 * k + 1] = win[2 * src + 1];
    }
    if (threadIdx.x == 0) {
        const unsigned n = s_novf;
        if (n > GRID_OVF_CAP) atomicOr(a.status, SP_STATUS_GRID_OVERFLOW);
        GridHeader hd;
        hd.i0 = run.wi0 + ti0;
        hd.j0 = run.wj0 + tj0;
        hd.h = th;
        hd.w = tw;
        hd.n_ovf = n < GRID_OVF_CAP ? n : GRID_OVF_CAP;
        a.grid.head[wg] = hd;
    }
}

// Flow-grid gradient of one 32 x 32-node tile of one pair: each thread holds
// four nodes' two fixed-point sums and adds, in workgroup order, the partial
// of every workgroup of the pair whose box covers them, then the overflow
// records that fall in the tile; the sums leave as floats (scaled by 2^-e).
// Workgroups are (pair, tile row, tile column) over the batch's largest grid.
constexpr int GRID_TILE = 32;

__global__ void __launch_bounds__(256)
bwd_grid_reduce(BwdArgs a, int ntx, int nty)
{
    const int64_t bid = blockIdx.x;
    const int p = (int)(bid / ((int64_t)ntx * nty));
    const int rem = (int)(bid - (int64_t)p * ntx * nty);
    const int ty = rem / ntx, tx = rem - ty * ntx;
    const synthpix_pair P = a.pairs[p];
    const int i0 = ty * GRID_TILE, j0 = tx * GRID_TILE;
    if (i0 >= P.Gh || j0 >= P.Gw) return;
    const uint32_t state = a.scale[SC_STATE];
    float* out = a.g_flow + P.flow_offset;
    // thread -> nodes (i0 + r + 8 q, j0 + c), r = threadIdx / 32, c = threadIdx % 32, q = 0..3
    const int r = threadIdx.x >> 5, c = threadIdx.x & 31;
    unsigned long long su[4] = {0ull, 0ull, 0ull, 0ull}, sv[4] = {0ull, 0ull, 0ull, 0ull};
    __shared__ int s_list[256];
    if (state == SC_VALID) {
        const int64_t w0 = a.grid.wg_base[p], w1 = a.grid.wg_base[p + 1];
        for (int64_t wb = w0; wb < w1; wb += 256) {
            // the covering workgroups of this stretch, in order
            const int64_t w = wb + threadIdx.x;
            bool hit = false;
            if (w < w1) {
                const GridHeader hd = a.grid.head[w];
                hit = (hd.h > 0 && hd.i0 < i0 + GRID_TILE && hd.i0 + hd.h > i0 && hd.j0 < j0 + GRID_TILE &&
                       hd.j0 + hd.w > j0) || hd.n_ovf > 0;
            }
            // ordered compaction: a workgroup-wide prefix count of the hits
            const unsigned long long bal = __ballot(hit);
            __shared__ int s_cnt[4];
            if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = __popcll(bal);
            __syncthreads();
            int before = 0;
            for (int k = 0; k < (int)(threadIdx.x >> 6); ++k) before += s_cnt[k];
            const int lane = threadIdx.x & 63;
            const unsigned long long lower = lane ? (bal & ((~0ull) >> (64 - lane))) : 0ull;
            if (hit) s_list[before + __popcll(lower)] = (int)(w - wb);
            const int nl = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
            __syncthreads();
            for (int k = 0; k < nl; ++k) {
                const int64_t wi = wb + s_list[k];
                const GridHeader hd = a.grid.head[wi];
                const unsigned long long* part = a.grid.part + wi * (2 * WIN_NODES);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ni = i0 + r + 8 * q, nj = j0 + c;
                    const int li = ni - hd.i0, lj = nj - hd.j0;
                    if ((unsigned)li < (unsigned)hd.h && (unsigned)lj < (unsigned)hd.w) {
                        su[q] += part[2 * (li * hd.w + lj)];
                        sv[q] += part[2 * (li * hd.w + lj) + 1];
                    }
                }
                for (unsigned e = 0; e < hd.n_ovf; ++e) {
                    const GridRecord rec = a.grid.ovf[wi * GRID_OVF_CAP + e];
                    const int node = rec.elem >> 1;
                    const int ni = node / P.Gw, nj = node - ni * P.Gw;
                    const int q = (ni - i0 - r) >> 3;
                    if (nj == j0 + c && ni >= i0 + r && ((ni - i0 - r) & 7) == 0 && q < 4) {
                        if (rec.elem & 1) sv[q] += rec.value;
                        else su[q] += rec.value;
                    }
                }
            }
            __syncthreads();
        }
    }
    const double inv = state == SC_VALID ? __builtin_ldexp(1.0, -(int)a.scale[SC_EXP]) : 0.0;
    const float fill = state == SC_NONFINITE ? __builtin_nanf("") : 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ni = i0 + r + 8 * q, nj = j0 + c;
        if (ni < P.Gh && nj < P.Gw) {
            const int64_t k = 2 * ((int64_t)ni * P.Gw + nj);
            out[k] = state == SC_VALID ? (float)((double)(long long)su[q] * inv) : fill;
            out[k + 1] = state == SC_VALID ? (float)((double)(long long)sv[q] * inv) : fill;
        }
    }
}

// Inputs of the fixed-point scale: the largest |dL/dx2|, |dL/dy2| and a bound L
// on the transposed velocity Jacobian's max-row-sum over every cell (the
// bilinear x-derivative is a blend of the cell's two edge differences, so its
// magnitude is at most the larger one).  Also each slice's float64 sum of the
// sheet-width terms, in a fixed order.  Blocks (pair, slice), ns <= BWD_SLICES
// slices per pair (more for pairs with many particles); float bits of
// non-negative values order like unsigned integers.
__global__ void __launch_bounds__(256)
bwd_bounds(BwdArgs a, int ns)
{
    const synthpix_pair P = a.pairs[blockIdx.x];
    const int sl = blockIdx.y;
    float gm = 0.0f;
    double sh = 0.0;
#pragma unroll 4
    for (int64_t i = (int64_t)sl * 256 + threadIdx.x; i < P.n_max; i += (int64_t)ns * 256) {
        const int64_t g = P.particle_offset + i;
        const float u = a.gx2[g], v = a.gy2[g];
        gm = __builtin_fmaxf(gm, __builtin_fmaxf(__builtin_fabsf(u), __builtin_fabsf(v)));
        if (!__builtin_isfinite(u) || !__builtin_isfinite(v)) gm = __builtin_inff();
        sh += (double)a.sheet[g];
    }
    const float2* F = reinterpret_cast<const float2*>(a.flow + P.flow_offset);
    const float sx = (float)P.Gw / (float)P.W, sy = (float)P.Gh / (float)P.H;
    float lm = 0.0f;
    for (int i = sl; i < P.Gh - 1; i += ns)
        for (int j = threadIdx.x; j < P.Gw - 1; j += 256) {
            const float2 A = F[(int64_t)i * P.Gw + j], B = F[(int64_t)i * P.Gw + j + 1];
            const float2 C = F[(int64_t)(i + 1) * P.Gw + j], E = F[(int64_t)(i + 1) * P.Gw + j + 1];
            const float lx = sx * (__builtin_fmaxf(__builtin_fabsf(B.x - A.x), __builtin_fabsf(E.x - C.x)) +
                                   __builtin_fmaxf(__builtin_fabsf(B.y - A.y), __builtin_fabsf(E.y - C.y)));
            const float ly = sy * (__builtin_fmaxf(__builtin_fabsf(C.x - A.x), __builtin_fabsf(E.x - B.x)) +
                                   __builtin_fmaxf(__builtin_fabsf(C.y - A.y), __builtin_fabsf(E.y - B.y)));
            lm = __builtin_fmaxf(lm, __builtin_fmaxf(lx, ly));
            if (!__builtin_isfinite(lx) || !__builtin_isfinite(ly)) lm = __builtin_inff();
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        gm = __builtin_fmaxf(gm, __shfl_xor(gm, o, 64));
        lm = __builtin_fmaxf(lm, __shfl_xor(lm, o, 64));
    }
    __shared__ float red[2][4];
    __shared__ double sred[256];
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = gm;
        red[1][threadIdx.x >> 6] = lm;
    }
    sred[threadIdx.x] = sh;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) sred[threadIdx.x] += sred[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        // per-block results (no same-address atomics); bwd_scale reduces them
        const int64_t k = (int64_t)blockIdx.x * ns + sl;
        a.bound_part[2 * k] = __builtin_fmaxf(__builtin_fmaxf(red[0][0], red[0][1]),
                                              __builtin_fmaxf(red[0][2], red[0][3]));
        a.bound_part[2 * k + 1] = __builtin_fmaxf(__builtin_fmaxf(red[1][0], red[1][1]),
                                                  __builtin_fmaxf(red[1][2], red[1][3]));
        a.sheet_part[k] = sred[0];
    }
}

// The fixed-point exponent e.  Every upstream value k of the reverse sweep obeys
// |k| <= K = G0 kfac growth^(S-1), from the stage recurrences with |J^T k| <= L |k|
// (Euler: kfac = |h|, growth = 1 + |h| L; RK4: k4 = c, k3 = 2c + |h| L k4,
// k2 = 2c + |h|/2 L k3, k1 = c + |h|/2 L k2 with c = |h|/6, growth = 1 + L sum k).
// A node sum has at most 2^en such terms of weight <= 1, so with
// e = 61 - ceil(log2 K) - en no partial sum leaves the int64 range.
__global__ void __launch_bounds__(256)
bwd_scale(uint32_t* __restrict__ sc, synthpix_advect_params ap, int en, const double* __restrict__ sheet_part,
          const float* __restrict__ bound_part, int n_pairs, int ns, float* __restrict__ g_sheet,
          float* __restrict__ g_sheet_total)
{
    // per-pair sheet-width gradient: the slices' float64 sums in slice order; each
    // thread takes a contiguous run of pairs, and the shared-sheet total adds
    // the runs' float64 sums in a fixed tree, so it too is reproducible
    __shared__ double s_tot[256];
    const int per = (n_pairs + 255) / 256;
    const int pa = (int)threadIdx.x * per, pb = min(n_pairs, pa + per);
    double run = 0.0;
    for (int p = pa; p < pb; ++p) {
        double t = 0.0;
        // unrolled so that the loads are issued together; the additions stay in slice order
#pragma unroll 16
        for (int k = 0; k < ns; ++k) t += sheet_part[(int64_t)p * ns + k];
        g_sheet[p] = (float)t;
        run += t;
    }
    s_tot[threadIdx.x] = run;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) s_tot[threadIdx.x] += s_tot[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0 && g_sheet_total) *g_sheet_total = (float)s_tot[0];
    // maxima over all (pair, slice) blocks
    float gm = 0.0f, lm = 0.0f;
    for (int64_t k = threadIdx.x; k < (int64_t)n_pairs * ns; k += blockDim.x) {
        gm = __builtin_fmaxf(gm, bound_part[2 * k]);
        lm = __builtin_fmaxf(lm, bound_part[2 * k + 1]);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        gm = __builtin_fmaxf(gm, __shfl_xor(gm, o, 64));
        lm = __builtin_fmaxf(lm, __shfl_xor(lm, o, 64));
    }
    __shared__ float red[2][4];
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = gm;
        red[1][threadIdx.x >> 6] = lm;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double G0 = (double)__builtin_fmaxf(__builtin_fmaxf(red[0][0], red[0][1]),
                                              __builtin_fmaxf(red[0][2], red[0][3]));
    const double L = (double)__builtin_fmaxf(__builtin_fmaxf(red[1][0], red[1][1]),
                                             __builtin_fmaxf(red[1][2], red[1][3]));
    sc[SC_G2MAX] = __float_as_uint((float)G0);
    sc[SC_LIP] = __float_as_uint((float)L);
    const int S = ap.substeps;
    const double h = __builtin_fabs((double)ap.dt / (double)S);
    double kfac, growth;
    if (ap.integrator == SP_EULER) {
        kfac = h;
        growth = 1.0 + h * L;
    } else {
        const double c = h / 6.0;
        const double k4 = c, k3 = 2.0 * c + h * L * k4, k2 = 2.0 * c + 0.5 * h * L * k3, k1 = c + 0.5 * h * L * k2;
        kfac = __builtin_fmax(__builtin_fmax(k1, k2), __builtin_fmax(k3, k4));
        growth = 1.0 + L * (k1 + k2 + k3 + k4);
    }
    const double K = G0 * kfac * pow(growth, (double)(S - 1)) * 1.0009765625;
    uint32_t state = SC_VALID;
    int e = 0;
    if (!(G0 > 0.0) || !(h > 0.0)) {
        state = SC_NONE;
    } else if (!__builtin_isfinite(K) || !(K > 0.0)) {
        state = SC_NONFINITE;
    } else {
        int k;
        (void)__builtin_frexp(K, &k);   // K < 2^k
        e = 61 - k - en;
    }
    sc[SC_EXP] = (uint32_t)e;
    sc[SC_STATE] = state;
}

// Status, scale block and sheet outputs cleared; the flow gradient zeroed (its
// pairs' grids are overwritten by the reduction, gaps between them stay 0).
__global__ void bwd_init(float* __restrict__ g_flow, int64_t n, uint32_t* __restrict__ status,
                         uint32_t* __restrict__ sc, float* __restrict__ g_sheet, int n_pairs,
                         float* __restrict__ g_sheet_total, const synthpix_pair* __restrict__ pairs,
                         int64_t* __restrict__ wg_base)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 4) {
        status[t] = 0u;
        sc[t] = 0u;
    }
    if (blockIdx.x == 0) {
        // workgroups of the flow adjoint, each pair's particles in chunks of 256:
        // an exclusive prefix over the pairs, 256 at a time (wave scans, then
        // the four wave totals)
        __shared__ int64_t s_tot[4];
        const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
        int64_t carry = 0;
        for (int b = 0; b < n_pairs; b += 256) {
            const int p = b + (int)threadIdx.x;
            const int64_t v = p < n_pairs ? (pairs[p].n_max + 255) / 256 : 0;
            int64_t inc = v;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t u = __shfl_up(inc, o, 64);
                if (lane >= o) inc += u;
            }
            if (lane == 63) s_tot[wid] = inc;
            __syncthreads();
            int64_t before = 0, total = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if (w < wid) before += s_tot[w];
                total += s_tot[w];
            }
            if (p < n_pairs) wg_base[p] = carry + before + inc - v;
            carry += total;
            __syncthreads();
        }
        if (threadIdx.x == 0) wg_base[n_pairs] = carry;
    }
    // sheet gradients of a batch without particles (otherwise overwritten later)
    if (t < n_pairs) g_sheet[t] = 0.0f;
    if (t == 0 && g_sheet_total) *g_sheet_total = 0.0f;
    for (int64_t k = t; k < n; k += (int64_t)gridDim.x * blockDim.x) g_flow[k] = 0.0f;
}


// ------------------------------------------------------------------ image loss

// grad = scale (J - T) over float4 groups, grid-stride in a fixed grid of
// MSE_BLOCKS workgroups; with loss partials, each workgroup's float64 sum of
// (J - T)^2 (each thread's terms in index order, then a fixed tree) goes to
// part[block].  The last n % 4 elements are workgroup 0's.
__global__ void __launch_bounds__(256)
mse_grad_kernel(const float* __restrict__ J, const float* __restrict__ T, int64_t n, float scale,
                float* __restrict__ grad, double* __restrict__ part)
{
    const int64_t n4 = n >> 2;
    const float4* J4 = reinterpret_cast<const float4*>(J);
    const float4* T4 = reinterpret_cast<const float4*>(T);
    float4* G4 = reinterpret_cast<float4*>(grad);
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n4; k += (int64_t)gridDim.x * 256) {
        const float4 j = J4[k], t = T4[k];
        const float4 d = make_float4(j.x - t.x, j.y - t.y, j.z - t.z, j.w - t.w);
        G4[k] = make_float4(scale * d.x, scale * d.y, scale * d.z, scale * d.w);
        if (part) {     // the differences exactly, in float64
            const double ex = (double)j.x - (double)t.x, ey = (double)j.y - (double)t.y;
            const double ez = (double)j.z - (double)t.z, ew = (double)j.w - (double)t.w;
            acc = __builtin_fma(ex, ex, acc);
            acc = __builtin_fma(ey, ey, acc);
            acc = __builtin_fma(ez, ez, acc);
            acc = __builtin_fma(ew, ew, acc);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) {
        const int64_t i = 4 * n4 + threadIdx.x;
        const float j = J[i], t = T[i];          // read before the write: grad may be J or T
        grad[i] = scale * (j - t);
        if (part) {
            const double e = (double)j - (double)t;
            acc = __builtin_fma(e, e, acc);
        }
    }
    if (!part) return;
    __shared__ double red[256];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// loss = (sum of the partials: each thread's in index order, then a fixed tree) / n.
// One workgroup, bound by the latency of its loads: 1024 threads with eight in
// flight each (256 threads, one at a time: 11 us for the 8192 partials of 64 pairs of
// 512^2 and 101 us for the 131072 of 32 pairs of 2048^2; 4.7 and 14.7 us so).
constexpr int FINISH_NT = 1024;

__global__ void __launch_bounds__(FINISH_NT)
mse_finish(const double* __restrict__ part, int64_t n_part, int64_t n, double* __restrict__ loss)
{
    constexpr int BATCH = 8;
    __shared__ double red[FINISH_NT];
    double v = 0.0;
    for (int64_t k = threadIdx.x; k < n_part; k += BATCH * FINISH_NT) {
        double e[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) e[j] = k + j * FINISH_NT < n_part ? part[k + j * FINISH_NT] : 0.0;
#pragma unroll
        for (int j = 0; j < BATCH; ++j) v += e[j];
    }
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = FINISH_NT / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = n > 0 ? red[0] / (double)n : 0.0;
}

hipError_t launch_mse_grad(const float* J, const float* T, int64_t n, float scale, float* grad, double* loss,
                           double* part, hipStream_t s)
{
    TimedScope ts("mse_grad", s);
    const int64_t want = (n / 4 + 255) / 256;
    const unsigned grid = loss ? (unsigned)MSE_BLOCKS : (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, MSE_BLOCKS));
    hipLaunchKernelGGL(mse_grad_kernel, dim3(grid), dim3(256), 0, s, J, T, n, scale, grad, loss ? part : nullptr);
    if (loss) hipLaunchKernelGGL(mse_finish, dim3(1), dim3(FINISH_NT), 0, s, part, (int64_t)MSE_BLOCKS, n, loss);
    return hipGetLastError();
}

// Workgroups of the per-pixel blur adjoint: (pair, frame, strip row, strip
// column) over the batch's largest pair.
int64_t blur_grad_blocks(int n_pairs, int max_w, int max_h, bool mse)
{
    const int sh = blur_strip_rows(mse);
    return (int64_t)n_pairs * 2 * ((max_w + 255) / 256) * ((max_h + sh - 1) / sh);
}

// Workgroups of the particle-major gather: 256 / G particles each.
static unsigned gather_blocks(int64_t n_span, int G)
{
    return (unsigned)((n_span + 256 / G - 1) / (256 / G));
}

// Workgroups for the crowded blocks' rest: a multiple of the 8 XCDs, so that the blocks
// after them keep their places.
static unsigned rest_workgroups(int64_t n_span, int most, int64_t blocks)
{
    const int64_t segs = (n_span + most - 1) / most, cus = device_cu_count();
    return (unsigned)((std::min(segs, std::max(cus, std::min(4 * cus, blocks / 16))) + 7) / 8 * 8);
}

// Diameter bound of the block and row gathers (wider particles take bwd_gather): the block
// gather's region then fits in LDS.
static bool narrow_particles(const BwdArgs& a)
{
    return block_region_side(a.d_max, BLOCK_LOG) <= REGION_SIDE_MAX;
}

// Whether the block gather is the faster one: enough particles to repay its phases (about
// 16 us however few) and its blocks (about 16 ns each), as the row gather costs 0.26 ns per
// particle of d about 2.5 and 0.55 of d to 6.  Row / block gather in us: one pair of 1024^2
// (256 blocks) at 123 / 205 / 410 particles a block 16 / 22 / 35 and 21 / 23 / 25; 64 pairs
// of 256^2 (1024 blocks) at 41 / 82 / 205 22 / 32 / 60 and 20 / 21 / 30; 64 of 512^2 (4096)
// at 20 / 41 / 61 / 82 42 / 63 / 82 / 103 and 67 / 72 / 76 / 78; 4 of 2048^2 with d to 6
// (4096) at 20 / 41 / 61 / 82 76 / 122 / 171 / 214 and 130 / 138 / 143 / 150.
static bool block_gather_pays(const BwdArgs& a)
{
    return a.slots >= 40 * a.block_groups + 24000 && a.order.log_block <= BLOCK_LOG;
}

// Whether the row gather gives each frame lanes of its own: while that leaves the chip
// unfilled (one pair of 512^2 at 0.05 ppp 11.5 us either way, 20 / 82 a block 11.1 / 11.0
// -> 8.4 / 8.7; 2 of them at 0.1 ppp, 52 k particles, 21.5 -> 23.7).
static bool rows_both(const BwdArgs& a) { return a.slots <= 64 * (int64_t)device_cu_count(); }

void launch_advect_adjoint(const BwdArgs& a, const synthpix_advect_params& ap, unsigned blocks, hipStream_t s)
{
    const int S = ap.substeps;
#define SP_ADJ(CK, SK)                                                                                              \
    do {                                                                                                            \
        if (ap.integrator == SP_RK4) hipLaunchKernelGGL((bwd_advect<CK, SK, true>), dim3(blocks), dim3(256), 0, s, a, ap); \
        else hipLaunchKernelGGL((bwd_advect<CK, SK, false>), dim3(blocks), dim3(256), 0, s, a, ap);                 \
    } while (0)
    if (S <= 1) SP_ADJ(1, 1);
    else if (S <= 2) SP_ADJ(2, 1);
    else if (S <= 4) SP_ADJ(4, 1);
    else if (S <= 8) SP_ADJ(8, 1);
    else if (S <= 16) SP_ADJ(16, 1);
    else if (S <= 32) SP_ADJ(32, 1);
    else SP_ADJ(32, 32);       // substeps <= 1024 = 32 * 32
#undef SP_ADJ
}

hipError_t launch_backward(const BwdArgs& a, int64_t n_span, int64_t n_flow, const synthpix_advect_params& ap,
                           int blur, int en, hipStream_t s)
{
    {
        TimedScope ts("bwd_init", s);
        const int64_t blocks = std::min<int64_t>(std::max<int64_t>((n_flow + 255) / 256 + 1, (a.n_pairs + 255) / 256),
                                                 65536);
        hipLaunchKernelGGL(bwd_init, dim3((unsigned)blocks), dim3(256), 0, s, a.g_flow, n_flow, a.status, a.scale,
                           a.g_sheet, a.n_pairs, a.g_sheet_total, a.pairs, a.grid.wg_base);
    }
    if (a.mse && !a.eblur) return hipErrorInvalidValue;
    // the blur's adjoint once per pixel (the gather then runs on the unblurred
    // footprints of B^T dL/dJ): for wide blurs, and always
    // for the loss-fused form, whose pass also forms dL/dJ (and the loss, which
    // the images define even when no pair holds a particle)
    const bool per_pixel = a.eblur && (a.mse || blur >= 2);
    if (per_pixel && (n_span > 0 || (a.mse && a.loss))) {
        TimedScope ts("bwd_blur", s);
        const int64_t nb = blur_grad_blocks(a.n_pairs, a.max_w, a.max_h, a.mse);
        if (nb < 1 || nb > 0xFFFFFFFFll) return hipErrorInvalidValue;
        const int sh = blur_strip_rows(a.mse);
        const int nsx = (a.max_w + 255) / 256, nsy = (a.max_h + sh - 1) / sh;
#define SP_BLUR(BB)                                                                                             \
    case BB:                                                                                                    \
        if (a.mse) hipLaunchKernelGGL((bwd_blur_grad<BB, true>), dim3((unsigned)nb), dim3(256), 0, s, a, nsx, nsy); \
        else hipLaunchKernelGGL((bwd_blur_grad<BB, false>), dim3((unsigned)nb), dim3(256), 0, s, a, nsx, nsy);     \
        break;
        switch (blur) {
        SP_BLUR(0) SP_BLUR(1) SP_BLUR(2) SP_BLUR(3)
        default: return hipErrorInvalidValue;
        }
#undef SP_BLUR
        if (a.mse && a.loss)
            hipLaunchKernelGGL(mse_finish, dim3(1), dim3(FINISH_NT), 0, s, a.loss_part, nb, a.loss_n, a.loss);
    }
    if (n_span > 0) {
        if (a.recompute_x2) {
            const hipError_t e = launch_advect(a.pairs, a.n_pairs, n_span, a.flow, ap, a.x1, a.y1, a.x2w, a.y2w, s,
                                               a.order);
            if (e != hipSuccess) return e;
        }
        BwdArgs b = a;
        if (per_pixel) b.grad = a.eblur;
        const bool unfolded = per_pixel || blur == 0;        // no blur left for the gather's tables
        if (unfolded && narrow_particles(a) && block_gather_pays(a)) {
            TimedScope ts("bwd_gather", s);
            const int gb = 1 << (BLOCK_LOG - a.order.log_block);
            const int side = block_region_side(a.d_max, BLOCK_LOG), cap = side * side;
            const int ngx = (a.max_w + 63) / 64, ngy = (a.max_h + 63) / 64;
            const int64_t nb = (int64_t)a.n_pairs * ngx * ngy;
            const size_t lds = sizeof(float) * ((size_t)cap + REGION_PAD);
            // one pass where a block's particles fit (both sides measured above)
            const int np = a.slots > 256 * a.block_groups ? 512 : 256;
            // twice the mean of a home block: evenly spread particles stay below
            const int64_t mean = (a.slots + a.order.blocks - 1) / a.order.blocks;
            const int most = (int)std::min<int64_t>(std::max<int64_t>(np, 2 * mean), 1 << 28);
            const unsigned rest = rest_workgroups(n_span, most, nb);
            if (nb + rest > 0xFFFFFFFFll) return hipErrorInvalidValue;
            const dim3 grid((unsigned)nb + rest);
            if (np == 512)
                hipLaunchKernelGGL(bwd_gather_blocks<512>, grid, dim3(512), lds, s, b, n_span, most, rest, gb, ngx, ngy,
                                   cap);
            else
                hipLaunchKernelGGL(bwd_gather_blocks<256>, grid, dim3(256), lds, s, b, n_span, most, rest, gb, ngx, ngy,
                                   cap);
            if (a.slots != n_span)
                hipLaunchKernelGGL(bwd_gaps, dim3((unsigned)((n_span + 255) / 256)), dim3(256), 0, s, b, n_span);
        } else if (unfolded && narrow_particles(a)) {
            TimedScope ts("bwd_gather", s);
            if (rows_both(a))
                hipLaunchKernelGGL(bwd_gather_rows<true>, dim3(gather_blocks(n_span, 16)), dim3(256), 0, s, b, n_span);
            else
                hipLaunchKernelGGL(bwd_gather_rows<false>, dim3(gather_blocks(n_span, 8)), dim3(256), 0, s, b, n_span);
        } else if (unfolded) {
            TimedScope ts("bwd_gather", s);
            hipLaunchKernelGGL((bwd_gather<0, 64, 16>), dim3(gather_blocks(n_span, 16)), dim3(256), 0, s, b, n_span);
        } else {
            TimedScope ts("bwd_gather", s);
            if (blur != 1) return hipErrorInvalidValue;
            // slots needed: floor(3 d_max) + 4 covered pixels + 4 of padding
            if ((int)(3.0f * a.d_max) + 8 <= 32)
                hipLaunchKernelGGL((bwd_gather<1, 32, 8>), dim3(gather_blocks(n_span, 8)), dim3(256), 0, s, a, n_span);
            else
                hipLaunchKernelGGL((bwd_gather<1, 64, 16>), dim3(gather_blocks(n_span, 16)), dim3(256), 0, s, a, n_span);
        }
        {
            TimedScope ts("bwd_bounds", s);
            // about 768 particles per slice (3 per thread), at least 32 slices per
            // pair: enough workgroups to keep the loads of every CU in flight
            const int64_t per = (n_span + (int64_t)a.n_pairs * 768 - 1) / ((int64_t)a.n_pairs * 768);
            const int ns = (int)std::min<int64_t>(std::max<int64_t>(per, 32), BWD_SLICES);
            hipLaunchKernelGGL(bwd_bounds, dim3((unsigned)a.n_pairs, ns), dim3(256), 0, s, a, ns);
            hipLaunchKernelGGL(bwd_scale, dim3(1), dim3(256), 0, s, a.scale, ap, en, a.sheet_part, a.bound_part,
                               a.n_pairs, ns, a.g_sheet, a.g_sheet_total);
        }
        if (a.grid.n_wg > 0) {
            TimedScope ts("bwd_advect", s);
            if (a.grid.n_wg > 0xFFFFFFFFll) return hipErrorInvalidValue;
            launch_advect_adjoint(a, ap, (unsigned)a.grid.n_wg, s);
        }
        {
            TimedScope ts("bwd_flow", s);
            const int ntx = (a.grid.max_gw + GRID_TILE - 1) / GRID_TILE, nty = (a.grid.max_gh + GRID_TILE - 1) / GRID_TILE;
            const int64_t nb = (int64_t)a.n_pairs * ntx * nty;
            if (nb > 0xFFFFFFFFll) return hipErrorInvalidValue;
            if (nb > 0) hipLaunchKernelGGL(bwd_grid_reduce, dim3((unsigned)nb), dim3(256), 0, s, a, ntx, nty);
        }
    }
    return hipGetLastError();
}

}  // namespace sp
