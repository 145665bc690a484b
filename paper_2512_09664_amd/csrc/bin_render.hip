// Screen-tile binning and the fused tile renderer (gfx950).
//
// Rendering follows Eq. 1 (rho = 0, sigma = d/4) with a Gaussian laser-sheet
// peak (Remark 1), point-sampled at pixel centres (Remark 2), summed over all
// particles (Section 2, "Considerations on the aggregation") on per-particle
// square patches |dx|, |dy| <= 1.5 d (Section 2, "Efficient rasterization").
//
// Pipeline of one call (all pairs of a batch at once):
//   bin_count   : per (pair, particle chunk), both frames' particle records (x, y,
//                 kappa, fixed-point peak) and patch boxes, and an LDS histogram of
//                 the tiles the boxes touch
//   scans       : per tile, chunk bases inside its list and its total; per
//                 (pair, frame), the exclusive scan of the totals -> list offsets
//   bin_scatter : per (pair, frame, chunk), LDS cursors -> particle indices into
//                 tile lists
//   (bins_small : the three of them in one launch, for small pairs)
//   render_tile : per (pair, frame, tile) stage the list in LDS, splat the patches
//                 into an LDS fixed-point accumulator (tile + blur apron), then
//                 blur, noise, quantise and store.
// No global atomics: counts, cursors and pixel sums all live in LDS.  Pixel sums
// are exact 32-bit fixed point, so the LDS atomics' order does not matter.
#include <map>
#include <mutex>
#include <utility>

#include "device_math.hpp"
#include "launch.hpp"

namespace sp {

__device__ __forceinline__ int find_pair_by_chunk(const PairLayout* L, int n_pairs, int64_t c)
{
    int lo = 0, hi = n_pairs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (L[mid].chunk_base <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Exclusive prefix over the lanes of a wave.
__device__ __forceinline__ int64_t wave_before(int64_t v)
{
    int64_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t u = __shfl_up(inc, o, 64);
        if ((int)(threadIdx.x & 63) >= o) inc += u;
    }
    return inc - v;
}

// ------------------------------------------------------------------ layout

// Batches of at most a wave of pairs need no layout launch: each wave of the
// first binning kernel sums the pairs' sizes itself, one pair per lane, and takes
// its workgroup's pair from them (one launch, about 5 us, less per call).
constexpr int INLINE_PAIRS = 64;

// Lane l's layout entry of pair l (l < n_pairs <= 64).
__device__ __forceinline__ PairLayout lane_layout(const synthpix_pair* __restrict__ pairs, int n_pairs,
                                                  const RenderConfig& cfg)
{
    const int l = (int)(threadIdx.x & 63);
    PairLayout o{};
    int64_t nt = 0, cap = 0;
    if (l < n_pairs) {
        const int n = pairs[l].n_max;
        o.n_chunks = (n + cfg.chunk - 1) / cfg.chunk;
        o.ntx = (pairs[l].W + cfg.tile_w - 1) >> cfg.log_tw;
        o.nty = (pairs[l].H + cfg.tile_h - 1) >> cfg.log_th;
        nt = (int64_t)o.ntx * o.nty;
        cap = (int64_t)n * cfg.kx * cfg.ky;
    }
    o.entry_cap = cap;
    o.chunk_base = (int32_t)wave_scan((uint32_t)o.n_chunks) - o.n_chunks;
    o.tile_base = (int32_t)(wave_scan((uint32_t)nt) - (uint32_t)nt);
    o.hist_base = wave_before(2 * (int64_t)o.n_chunks * nt);
    o.entry_base = wave_before(2 * cap);
    return o;
}

// The pair of chunk cb and its layout from the lanes' entries, as wave-uniform
// values; workgroup 0 stores all entries and clears the status words.
__device__ __forceinline__ int chunk_pair(const synthpix_pair* __restrict__ pairs, int n_pairs,
                                          const RenderConfig& cfg, int cb, PairLayout* __restrict__ L,
                                          uint32_t* __restrict__ status, PairLayout& o)
{
    const PairLayout mine = lane_layout(pairs, n_pairs, cfg);
    const int l = (int)(threadIdx.x & 63);
    if (blockIdx.x == 0 && threadIdx.x < 64) {
        if (l < n_pairs) L[l] = mine;
        if (l < 16 && status) status[l] = 0u;
    }
    const int p = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(l < n_pairs && mine.chunk_base <= cb));
    o.chunk_base = __builtin_amdgcn_readlane(mine.chunk_base, p);
    o.n_chunks = __builtin_amdgcn_readlane(mine.n_chunks, p);
    o.tile_base = __builtin_amdgcn_readlane(mine.tile_base, p);
    o.ntx = __builtin_amdgcn_readlane(mine.ntx, p);
    o.nty = __builtin_amdgcn_readlane(mine.nty, p);
    o.flags = 0u;
    o.hist_base = __shfl(mine.hist_base, p, 64);
    o.entry_base = __shfl(mine.entry_base, p, 64);
    o.entry_cap = __shfl(mine.entry_cap, p, 64);
    return p;
}

__global__ void __launch_bounds__(256)
bin_layout(const synthpix_pair* __restrict__ pairs, int n_pairs, RenderConfig cfg,
           PairLayout* __restrict__ L, uint32_t* __restrict__ status)
{
    __shared__ int64_t s_part[4][256];
    __shared__ int64_t s_carry[4];
    const int t = threadIdx.x;
    if (t < 4) s_carry[t] = 0;
    // status words, and the renderer's per-XCD work queues (words 8 .. 15)
    if (t < 16) status[t] = 0u;
    __syncthreads();
    for (int base = 0; base < n_pairs; base += 256) {
        const int p = base + t;
        int64_t v[4] = {0, 0, 0, 0};
        int n_chunks = 0, ntx = 0, nty = 0;
        int64_t cap = 0;
        if (p < n_pairs) {
            const synthpix_pair P = pairs[p];
            n_chunks = (P.n_max + cfg.chunk - 1) / cfg.chunk;
            ntx = (P.W + cfg.tile_w - 1) / cfg.tile_w;
            nty = (P.H + cfg.tile_h - 1) / cfg.tile_h;
            cap = (int64_t)P.n_max * cfg.kx * cfg.ky;
            v[0] = n_chunks;
            v[1] = (int64_t)ntx * nty;
            v[2] = 2 * (int64_t)n_chunks * ntx * nty;
            v[3] = 2 * cap;
        }
        for (int k = 0; k < 4; ++k) s_part[k][t] = v[k];
        __syncthreads();
        // Hillis-Steele inclusive scan of the four columns
        for (int off = 1; off < 256; off <<= 1) {
            int64_t add[4];
            for (int k = 0; k < 4; ++k) add[k] = t >= off ? s_part[k][t - off] : 0;
            __syncthreads();
            for (int k = 0; k < 4; ++k) s_part[k][t] += add[k];
            __syncthreads();
        }
        if (p < n_pairs) {
            PairLayout o;
            o.chunk_base = (int32_t)(s_carry[0] + s_part[0][t] - v[0]);
            o.n_chunks = n_chunks;
            o.tile_base = (int32_t)(s_carry[1] + s_part[1][t] - v[1]);
            o.ntx = ntx;
            o.nty = nty;
            o.flags = 0u;
            o.hist_base = s_carry[2] + s_part[2][t] - v[2];
            o.entry_base = s_carry[3] + s_part[3][t] - v[3];
            o.entry_cap = cap;
            L[p] = o;
        }
        __syncthreads();
        if (t < 4) s_carry[t] += s_part[t][255];
        __syncthreads();
    }
}

// ------------------------------------------------------------------ particle records

// One particle's record in one frame: (x, y, kappa_x, Af), its patch box clipped
// to the image, in the anisotropic layout (kappa_y, kappa_xy), and the status
// bits it raises.
struct Record {
    float4 rec;
    uint2 box;
    float2 shp;
    uint32_t flags;
};

// The isotropic record: kappa = 8 / (d d), Af = min(2^24 I0 exp(-z^2 / (2 s^2)),
// 2^32 - 256), the patch |dx|, |dy| <= 1.5 d.  Particles that add nothing (I0 <=
// 0, d <= 0 or not a number, non-finite position) or whose d exceeds d_max
// (flagged) get an empty box.
__device__ __forceinline__ void record_iso(float x, float y, float z, float d, float I0, int W, int H,
                                           float sheet_sigma, float d_max, Record& o)
{
    const float cs = 0.5f / (sheet_sigma * sheet_sigma);
    const float Af = fixed_peak(I0 * expneg((z * z) * cs));
    bool live = (I0 > 0.0f) && (d > 0.0f);
    o.flags = 0u;
    if (live && !(d <= d_max)) {
        o.flags = SP_STATUS_D_ABOVE_MAX;
        live = false;
    }
    const float R = 1.5f * d;
    o.rec = make_float4(x, y, live ? 8.0f / (d * d) : 0.0f, Af);
    o.box = live ? patch_box(x, y, R, R, W, H) : make_uint2(EMPTY_BOX, EMPTY_BOX);
}

// The full particle model's records (Eq. 1 with sigma_y and rho; frame-2
// parameter variation, the sentence after Eq. 1; per-frame hiding, Section 2
// "Considerations on the aggregation"; the Remark 1 sheet law; frame-2 z from
// the out-of-plane motion).  Frame-2 parameters are
// frame 1's plus zero-mean Gaussians (Philox stream 2: Box-Muller of words 0, 1
// and 2, 3, cosine then sine, for d, d_y, rho, I0), clipped to [0, d_max],
// [-0.99, 0.99] and [0, inf) (masked particles stay dark); a particle is hidden
// in frame f when word f of stream 7 is below hide_p.
__device__ __forceinline__ float model_peak(float I0, float z, const RenderArgs& a)
{
    if (a.sheet_law == 0) return I0 * expneg((z * z) * (0.5f / (a.sheet_sigma * a.sheet_sigma)));
    // Remark 1: exp(-(1/sqrt(2 pi)) v^s), v = z^2 (2 / DZ0^2); v^s = exp(s ln v)
    const float v = (z * z) * (2.0f / (a.sheet_dz0 * a.sheet_dz0));
    float pw = 0.0f;
    if (v >= 0x1p-126f) {
        const float e = a.sheet_shape * log_ra(v);
        if (!(e < 80.0f)) return 0.0f;
        pw = expneg(-e);
    }
    return I0 * expneg((float)0.39894228040143267794 * pw);
}

// The model's record of particle i (slot g) in frame f; hide: the particle's
// words of stream 7 (read where hide_p > 0).
__device__ __forceinline__ void record_model(const RenderArgs& a, int f, int64_t g, uint32_t i, uint64_t pid,
                                             const u32x4& hide, int W, int H, float d_max, Record& o)
{
    const float x = f ? a.x[1][g] : a.x[0][g], y = f ? a.y[1][g] : a.y[0][g];
    const float z = f && a.z2 ? a.z2[g] : a.z[g];
    float d = a.d[g];
    float dy = a.dy ? a.dy[g] : d;
    float r = a.rho ? a.rho[g] : 0.0f;
    float I = a.I0[g];
    if (f && (a.jit_d > 0.0f || a.jit_rho > 0.0f || a.jit_I0 > 0.0f)) {
        const u32x4 w = draw(i, STREAM_JITTER, pid, a.seed);
        const float R0 = __builtin_sqrtf(-2.0f * log_ra(u24_open0(w.a)));
        const float R1 = __builtin_sqrtf(-2.0f * log_ra(u24_open0(w.c)));
        const float2 t0 = cossin2pi_ra(u24(w.b));
        const float2 t1 = cossin2pi_ra(u24(w.d));
        if (a.jit_d > 0.0f) {
            d = __builtin_fminf(__builtin_fmaxf(__builtin_fmaf(a.jit_d, R0 * t0.x, d), 0.0f), d_max);
            dy = __builtin_fminf(__builtin_fmaxf(__builtin_fmaf(a.jit_d, R0 * t0.y, dy), 0.0f), d_max);
        }
        if (a.jit_rho > 0.0f) r = __builtin_fminf(__builtin_fmaxf(__builtin_fmaf(a.jit_rho, R1 * t1.x, r), -0.99f), 0.99f);
        if (a.jit_I0 > 0.0f) I = I > 0.0f ? __builtin_fmaxf(__builtin_fmaf(a.jit_I0, R1 * t1.y, I), 0.0f) : 0.0f;
    }
    if (a.hide_p > 0.0f && u24(f ? hide.b : hide.a) < a.hide_p) I = 0.0f;
    bool live = (I > 0.0f) && (d > 0.0f) && (dy > 0.0f);
    o.flags = 0u;
    if (live && !(d <= d_max && dy <= d_max)) {
        o.flags = SP_STATUS_D_ABOVE_MAX;
        live = false;
    }
    if (live && !(__builtin_fabsf(r) <= 0.99f)) {
        o.flags = SP_STATUS_BAD_SHAPE;
        live = false;
    }
    // om = 1 - rho^2; kappa_x = 8 / (om d^2), kappa_y = 8 / (om d_y^2),
    // kappa_xy = -16 rho / (om d d_y) (0 for rho = 0: the separable form)
    const float om = __builtin_fmaf(-r, r, 1.0f);
    const float kx = live ? 8.0f / (om * (d * d)) : 0.0f;
    const float ky = live ? 8.0f / (om * (dy * dy)) : 0.0f;
    const float kxy = (live && r != 0.0f) ? (-16.0f * r) / (om * (d * dy)) : 0.0f;
    o.rec = make_float4(x, y, kx, fixed_peak(model_peak(I, z, a)));
    o.box = live ? patch_box(x, y, 1.5f * d, 1.5f * dy, W, H) : make_uint2(EMPTY_BOX, EMPTY_BOX);
    o.shp = make_float2(ky, kxy);
}

// ------------------------------------------------------------------ count / scatter

// Both frames' records of a chunk's particles (computed once for every tile list
// and tile that uses them) and its tile histograms: frame f's count of a tile in
// half f of one LDS word (a chunk has at most 2^14 particles).  A particle whose
// diameter or rho is out of range gets an empty box that carries the status bits
// (the status words are cleared by this launch, so the scatter raises them).
// With live counts (captured plans), the masked slots past a pair's count are
// skipped, here and in the scatter.  INLINE: at most 64 pairs, no layout launch.
// Bound by the records' arithmetic and their traffic (28 B read, 48 B written per
// particle).  The records pass the caches by, so that the boxes and histograms
// the next launches read stay there; so do the inputs where they would fill the
// last-level cache by themselves (STREAM).  Layout, records, count, scans and
// scatter as six launches / as three: 64 pairs of 1024^2 139 / 107 us, 16 of
// 512^2 45 / 31, one of 512^2 37 / 26, uneven pairs (8.2 M particles) 295 / 280;
// 13.4 M particles in dense 2048^2 pairs the same.  1024 threads against 256: 16
// pairs of 512^2 31 / 37 us.
constexpr int COUNT_THREADS = 1024;

template <bool STREAM>
__device__ __forceinline__ float load_once(const float* p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load(p);
    else return *p;
}

__device__ __forceinline__ void store_once(float4* p, const float4& v)
{
    typedef float vec4 __attribute__((ext_vector_type(4)));
    const vec4 u = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(u, reinterpret_cast<vec4*>(p));
}

template <bool MODEL, bool INLINE, bool STREAM>
__global__ void __launch_bounds__(COUNT_THREADS)
bin_count(const synthpix_pair* __restrict__ pairs, PairLayout* __restrict__ L, int n_pairs, RenderArgs a,
          RenderConfig cfg, float4* __restrict__ rec0, float4* __restrict__ rec1, uint2* __restrict__ box0,
          uint2* __restrict__ box1, float2* __restrict__ shp0, float2* __restrict__ shp1,
          uint32_t* __restrict__ hist, unsigned n_chunks_total, const int32_t* __restrict__ live,
          uint32_t* __restrict__ status)
{
    extern __shared__ uint32_t lh[];
    const unsigned cb = xcd_contiguous(blockIdx.x, n_chunks_total);
    int p;
    PairLayout PL;
    if (INLINE) {
        p = chunk_pair(pairs, n_pairs, cfg, (int)cb, L, status, PL);
    } else {
        p = find_pair_by_chunk(L, n_pairs, cb);
        PL = L[p];
    }
    const synthpix_pair P = pairs[p];
    const int chunk = (int)cb - PL.chunk_base;
    const int nt = PL.ntx * PL.nty;
    const int i_end = min(live ? min(live[p], P.n_max) : P.n_max, (chunk + 1) * cfg.chunk);
    // a chunk past the live slots holds nothing (and is not scanned): the whole
    // workgroup returns before its barrier
    if (live && chunk * cfg.chunk >= i_end) return;
    if (!MODEL && a.iod) a.use(*a.iod);
    for (int k = threadIdx.x; k < nt; k += COUNT_THREADS) lh[k] = 0u;
    __syncthreads();
    for (int i = chunk * cfg.chunk + (int)threadIdx.x; i < i_end; i += COUNT_THREADS) {
        const int64_t g = P.particle_offset + i;
        u32x4 hide = {0u, 0u, 0u, 0u};
        float z = 0.0f, d = 0.0f, I0 = 0.0f;
        if (MODEL) {
            if (a.hide_p > 0.0f) hide = draw((uint32_t)i, STREAM_HIDE, P.pair_id, a.seed);
        } else {
            z = load_once<STREAM>(a.z + g);
            d = load_once<STREAM>(a.d + g);
            I0 = load_once<STREAM>(a.I0 + g);
        }
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            Record o;
            if (MODEL)
                record_model(a, f, g, (uint32_t)i, P.pair_id, hide, P.W, P.H, cfg.d_max, o);
            else
                record_iso(load_once<STREAM>(a.x[f] + g), load_once<STREAM>(a.y[f] + g), z, d, I0, P.W, P.H,
                           a.sheet_sigma, cfg.d_max, o);
            if (o.flags) o.box.y = EMPTY_BOX | (o.flags << EMPTY_FLAGS);
            store_once((f ? rec1 : rec0) + g, o.rec);
            (f ? box1 : box0)[g] = o.box;
            if (MODEL && a.aniso) (f ? shp1 : shp0)[g] = o.shp;
            int tx0, tx1, ty0, ty1;
            if (!tile_rect(o.box, cfg, PL.ntx, PL.nty, tx0, tx1, ty0, ty1)) continue;
            for (int ty = ty0; ty <= ty1; ++ty)
                for (int tx = tx0; tx <= tx1; ++tx) atomicAdd(&lh[ty * PL.ntx + tx], 1u << (16 * f));
        }
    }
    __syncthreads();
    uint32_t* gh = hist + PL.hist_base + (int64_t)chunk * nt;
    uint32_t* gh1 = gh + (int64_t)PL.n_chunks * nt;
    for (int k = threadIdx.x; k < nt; k += COUNT_THREADS) {
        const uint32_t v = lh[k];
        gh[k] = v & 0xffffu;
        gh1[k] = v >> 16;
    }
}

__global__ void __launch_bounds__(256)
bin_scatter(const synthpix_pair* __restrict__ pairs, const PairLayout* __restrict__ L, int n_pairs,
            const uint2* __restrict__ box0, const uint2* __restrict__ box1, RenderConfig cfg,
            const uint32_t* __restrict__ hist, const int64_t* __restrict__ tile_offset, int64_t tiles_total,
            int32_t* __restrict__ entries, unsigned n_chunks_total, const int32_t* __restrict__ live,
            uint32_t* __restrict__ status)
{
    extern __shared__ uint32_t lh[];
    const int f = blockIdx.y;
    const unsigned cb = xcd_contiguous(blockIdx.x, n_chunks_total);
    const int p = find_pair_by_chunk(L, n_pairs, cb);
    const synthpix_pair P = pairs[p];
    const PairLayout PL = L[p];
    const int chunk = (int)cb - PL.chunk_base;
    const int nt = PL.ntx * PL.nty;
    const uint32_t* gh = hist + PL.hist_base + ((int64_t)f * PL.n_chunks + chunk) * nt;
    int32_t* seg = entries + PL.entry_base + (int64_t)f * PL.entry_cap;
    // cursors start at the chunk's first slot in each tile list
    const int64_t* toff = tile_offset + f * tiles_total + PL.tile_base;
    const int64_t seg0 = PL.entry_base + (int64_t)f * PL.entry_cap;
    const int i_end = min(live ? min(live[p], P.n_max) : P.n_max, (chunk + 1) * cfg.chunk);
    // a chunk past the live slots holds nothing: the whole workgroup returns before its barrier
    if (live && chunk * cfg.chunk >= i_end) return;
    for (int t = threadIdx.x; t < nt; t += blockDim.x) lh[t] = gh[t] + (uint32_t)(toff[t] - seg0);
    __syncthreads();
    const uint2* __restrict__ bxs = f ? box1 : box0;
    // BIN_ILP particles per thread and step: their box loads and LDS atomic
    // round trips overlap
    constexpr int BIN_ILP = 4;
    for (int i0 = chunk * cfg.chunk + threadIdx.x; i0 < i_end; i0 += BIN_ILP * blockDim.x) {
        uint2 r[BIN_ILP];
#pragma unroll
        for (int q = 0; q < BIN_ILP; ++q) {
            const int i = i0 + q * blockDim.x;
            r[q] = i < i_end ? bxs[P.particle_offset + i] : make_uint2(EMPTY_BOX, EMPTY_BOX);
        }
#pragma unroll
        for (int q = 0; q < BIN_ILP; ++q) {
            const int i = i0 + q * blockDim.x;
            int tx0, tx1, ty0, ty1;
            if (!tile_rect(r[q], cfg, PL.ntx, PL.nty, tx0, tx1, ty0, ty1)) {
                if (r[q].y >> EMPTY_FLAGS) atomicOr(status, r[q].y >> EMPTY_FLAGS);
                continue;
            }
            for (int ty = ty0; ty <= ty1; ++ty)
                for (int tx = tx0; tx <= tx1; ++tx) seg[atomicAdd(&lh[ty * PL.ntx + tx], 1u)] = i;
        }
    }
}

// ------------------------------------------------------------------ home order

// A spatial processing order for per-particle work that samples the flow grid:
// particle i of a pair goes to the block (a "tile" of the order's config) that
// holds its clamped position.  Blocks are numbered in strips of four block
// rows, column by column inside a strip, odd strips from right to left (so the
// last block of a strip and the first of the next are neighbours): a run of
// consecutive entries (one workgroup's particles) covers a compact patch of
// the image.  Count and
// scatter passes as for the tile lists, one entry per particle, in the frame-1
// half of the lists.
__device__ __forceinline__ int home_block(float x, float y, int W, int H, const PairLayout& PL,
                                          const RenderConfig& cfg)
{
    return home_block(x, y, W, H, PL.ntx, PL.nty, cfg.log_tw, cfg.log_th);
}

template <bool SCATTER, bool INLINE>
__global__ void __launch_bounds__(256)
order_pass(const synthpix_pair* __restrict__ pairs, PairLayout* __restrict__ L, int n_pairs,
           const float* __restrict__ x, const float* __restrict__ y, RenderConfig cfg, uint32_t* __restrict__ hist,
           const int64_t* __restrict__ tile_offset, int32_t* __restrict__ entries, unsigned n_chunks_total,
           const synthpix_batch_io* __restrict__ iod, const int32_t* __restrict__ live)
{
    extern __shared__ uint32_t lh[];
    if (iod) {
        x = iod->x1;
        y = iod->y1;
    }
    const unsigned cb = xcd_contiguous(blockIdx.x, n_chunks_total);
    int p;
    PairLayout PL;
    if (INLINE) {
        p = chunk_pair(pairs, n_pairs, cfg, (int)cb, L, nullptr, PL);
    } else {
        p = find_pair_by_chunk(L, n_pairs, cb);
        PL = L[p];
    }
    const synthpix_pair P = pairs[p];
    const int chunk = (int)cb - PL.chunk_base;
    const int nt = PL.ntx * PL.nty;
    uint32_t* gh = hist + PL.hist_base + (int64_t)chunk * nt;
    int32_t* seg = entries + PL.entry_base;
    const int64_t* toff = tile_offset + PL.tile_base;
    const int i_end = min(live ? min(live[p], P.n_max) : P.n_max, (chunk + 1) * cfg.chunk);
    // a chunk past the live slots holds nothing (and is not scanned): the whole
    // workgroup returns before its barrier
    if (live && chunk * cfg.chunk >= i_end) return;
    for (int t = threadIdx.x; t < nt; t += blockDim.x)
        lh[t] = SCATTER ? gh[t] + (uint32_t)(toff[t] - PL.entry_base) : 0u;
    __syncthreads();
    for (int i = chunk * cfg.chunk + threadIdx.x; i < i_end; i += blockDim.x) {
        const int64_t g = P.particle_offset + i;
        const uint32_t slot = atomicAdd(&lh[home_block(x[g], y[g], P.W, P.H, PL, cfg)], 1u);
        if (SCATTER) seg[slot] = i;
    }
    if (!SCATTER) {
        __syncthreads();
        for (int t = threadIdx.x; t < nt; t += blockDim.x) gh[t] = lh[t];
    }
}

// ------------------------------------------------------------------ small pairs

// One workgroup does a whole pair's (and frame's) binning where the pairs are
// small: layout, records, tile counts, their scan and the scatter in one launch
// instead of six, the counts never leaving LDS.  It walks the particles twice
// with 1024 threads, or with 256 where there are more workgroups of 1024 than the chip
// holds at once (two to a CU): 4096 pairs of 20 particles 157 us / 43, 1000 of
// 205 45 / 19, 300 of 6554 63 / 68 (order of 4096 66 / 24).
static int small_threads(int64_t workgroups) { return workgroups <= 2 * (int64_t)device_cu_count() ? 1024 : 256; }

// Pair p's layout: the tiles and entry slots of the pairs before it, summed over
// the workgroup (the chunk tables of the chunked passes stay empty).
template <int NT>
__device__ __forceinline__ PairLayout small_layout(const synthpix_pair* __restrict__ pairs, int p,
                                                   const RenderConfig& cfg, int64_t (*s_part)[NT / 64])
{
    int64_t tiles = 0, slots = 0;
    for (int q = (int)threadIdx.x; q < p; q += NT) {
        const int tx = (pairs[q].W + cfg.tile_w - 1) >> cfg.log_tw, ty = (pairs[q].H + cfg.tile_h - 1) >> cfg.log_th;
        tiles += (int64_t)tx * ty;
        slots += 2 * (int64_t)pairs[q].n_max * cfg.kx * cfg.ky;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        tiles += __shfl_xor(tiles, o, 64);
        slots += __shfl_xor(slots, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        s_part[0][threadIdx.x >> 6] = tiles;
        s_part[1][threadIdx.x >> 6] = slots;
    }
    __syncthreads();
    tiles = slots = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        tiles += s_part[0][w];
        slots += s_part[1][w];
    }
    PairLayout o;
    o.chunk_base = 0;
    o.n_chunks = 0;
    o.tile_base = (int32_t)tiles;
    o.ntx = (pairs[p].W + cfg.tile_w - 1) >> cfg.log_tw;
    o.nty = (pairs[p].H + cfg.tile_h - 1) >> cfg.log_th;
    o.flags = 0u;
    o.hist_base = 0;
    o.entry_base = slots;
    o.entry_cap = (int64_t)pairs[p].n_max * cfg.kx * cfg.ky;
    return o;
}

// Exclusive scan of the nt tile counts in lh, in place; counts and list offsets
// (seg0 plus the prefix) go to count and offset.
template <int NT>
__device__ __forceinline__ void small_scan(uint32_t* lh, int nt, int64_t seg0, uint32_t* __restrict__ count,
                                           int64_t* __restrict__ offset, uint32_t* s_wave)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int b = 0; b < nt; b += NT) {
        const int t = b + (int)threadIdx.x;
        const uint32_t v = t < nt ? lh[t] : 0u;
        const uint32_t inc = wave_scan(v);
        if (lane == 63) s_wave[wid] = inc;
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) {
            const uint32_t sw = s_wave[w];
            if (w < wid) before += sw;
            total += sw;
        }
        if (t < nt) {
            const uint32_t at = carry + before + inc - v;
            lh[t] = at;
            count[t] = v;
            offset[t] = seg0 + at;
        }
        carry += total;
        __syncthreads();
    }
}

// Grid (pair, frame).  A status bit of pair p and frame f is left in the pair's
// layout: the renderer raises it (the status words are cleared here, by one of
// the workgroups).
template <bool MODEL, int NT>
__global__ void __launch_bounds__(NT)
bins_small(const synthpix_pair* __restrict__ pairs, RenderArgs a, RenderConfig cfg, PairLayout* __restrict__ L,
           float4* __restrict__ rec0, float4* __restrict__ rec1, uint2* __restrict__ box0, uint2* __restrict__ box1,
           float2* __restrict__ shp0, float2* __restrict__ shp1, uint32_t* __restrict__ tile_count,
           int64_t* __restrict__ tile_offset, int64_t tiles_total, int32_t* __restrict__ entries,
           const int32_t* __restrict__ live, uint32_t* __restrict__ status)
{
    extern __shared__ uint32_t lh[];
    __shared__ int64_t s_part[2][NT / 64];
    __shared__ uint32_t s_wave[NT / 64];
    __shared__ uint32_t s_flags;
    const int p = blockIdx.x, f = blockIdx.y, t = (int)threadIdx.x;
    if (!MODEL && a.iod) a.use(*a.iod);
    const synthpix_pair P = pairs[p];
    if (t == 0) s_flags = 0u;
    if (p == 0 && f == 0 && t < 16) status[t] = 0u;
    const PairLayout o = small_layout<NT>(pairs, p, cfg, s_part);
    const int nt = o.ntx * o.nty;
    for (int k = t; k < nt; k += NT) lh[k] = 0u;
    __syncthreads();
    float4* __restrict__ rec = (f ? rec1 : rec0) + P.particle_offset;
    uint2* __restrict__ box = (f ? box1 : box0) + P.particle_offset;
    float2* __restrict__ shp = (f ? shp1 : shp0) + P.particle_offset;
    const int n = live ? min(live[p], P.n_max) : P.n_max;
    uint32_t flags = 0u;
    // two particles per thread and step, so that their loads overlap
    for (int i0 = t; i0 < n; i0 += 2 * NT) {
        Record r[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = i0 + q * NT;
            const int64_t g = P.particle_offset + min(i, n - 1);
            if (MODEL) {
                u32x4 hide = {0u, 0u, 0u, 0u};
                if (a.hide_p > 0.0f) hide = draw((uint32_t)i, STREAM_HIDE, P.pair_id, a.seed);
                record_model(a, f, g, (uint32_t)i, P.pair_id, hide, P.W, P.H, cfg.d_max, r[q]);
            } else {
                record_iso((f ? a.x[1] : a.x[0])[g], (f ? a.y[1] : a.y[0])[g], a.z[g], a.d[g], a.I0[g], P.W, P.H, a.sheet_sigma, cfg.d_max, r[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int i = i0 + q * NT;
            if (i >= n) break;
            rec[i] = r[q].rec;
            box[i] = r[q].box;
            if (MODEL && a.aniso) shp[i] = r[q].shp;
            flags |= r[q].flags;
            int tx0, tx1, ty0, ty1;
            if (!tile_rect(r[q].box, cfg, o.ntx, o.nty, tx0, tx1, ty0, ty1)) continue;
            for (int ty = ty0; ty <= ty1; ++ty)
                for (int tx = tx0; tx <= tx1; ++tx) atomicAdd(&lh[ty * o.ntx + tx], 1u);
        }
    }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();
    const int64_t seg0 = o.entry_base + (int64_t)f * o.entry_cap;
    small_scan<NT>(lh, nt, seg0, tile_count + f * tiles_total + o.tile_base, tile_offset + f * tiles_total + o.tile_base,
               s_wave);
    if (t == 0) {
        if (f == 0) {
            L[p].tile_base = o.tile_base;
            L[p].ntx = o.ntx;
            L[p].nty = o.nty;
            L[p].entry_base = o.entry_base;
            L[p].entry_cap = o.entry_cap;
        }
        reinterpret_cast<uint8_t*>(&L[p].flags)[f] = (uint8_t)s_flags;
    }
    int32_t* seg = entries + seg0;
    for (int i = t; i < n; i += NT) {
        int tx0, tx1, ty0, ty1;
        if (!tile_rect(box[i], cfg, o.ntx, o.nty, tx0, tx1, ty0, ty1)) continue;
        for (int ty = ty0; ty <= ty1; ++ty)
            for (int tx = tx0; tx <= tx1; ++tx) seg[atomicAdd(&lh[ty * o.ntx + tx], 1u)] = i;
    }
}

// The home-block order of small pairs in one launch: one workgroup per pair.
template <int NT>
__global__ void __launch_bounds__(NT)
order_small(const synthpix_pair* __restrict__ pairs, const float* __restrict__ x, const float* __restrict__ y,
            RenderConfig cfg, PairLayout* __restrict__ L, uint32_t* __restrict__ tile_count,
            int64_t* __restrict__ tile_offset, int32_t* __restrict__ entries,
            const synthpix_batch_io* __restrict__ iod, const int32_t* __restrict__ live)
{
    extern __shared__ uint32_t lh[];
    __shared__ int64_t s_part[2][NT / 64];
    __shared__ uint32_t s_wave[NT / 64];
    const int p = blockIdx.x, t = (int)threadIdx.x;
    if (iod) {
        x = iod->x1;
        y = iod->y1;
    }
    const synthpix_pair P = pairs[p];
    const PairLayout o = small_layout<NT>(pairs, p, cfg, s_part);
    const int nt = o.ntx * o.nty;
    for (int k = t; k < nt; k += NT) lh[k] = 0u;
    __syncthreads();
    x += P.particle_offset;
    y += P.particle_offset;
    const int n = live ? min(live[p], P.n_max) : P.n_max;
    for (int i = t; i < n; i += NT) atomicAdd(&lh[home_block(x[i], y[i], P.W, P.H, o, cfg)], 1u);
    __syncthreads();
    small_scan<NT>(lh, nt, o.entry_base, tile_count + o.tile_base, tile_offset + o.tile_base, s_wave);
    if (t == 0) L[p] = o;
    int32_t* seg = entries + o.entry_base;
    for (int i = t; i < n; i += NT)
        seg[atomicAdd(&lh[home_block(x[i], y[i], P.W, P.H, o, cfg)], 1u)] = i;
}

// ------------------------------------------------------------------ scans

// Exclusive prefix, in place, of one tile's nc chunk counts (nt apart); their sum.
__device__ __forceinline__ uint32_t scan_column(uint32_t* __restrict__ h, int nt, int nc)
{
    constexpr int U = 8;                 // chunk rows loaded together
    uint32_t run = 0;
    for (int c0 = 0; c0 < nc; c0 += U) {
        uint32_t v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = c0 + k < nc ? h[(int64_t)(c0 + k) * nt] : 0u;
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (c0 + k < nc) h[(int64_t)(c0 + k) * nt] = run;
            run += v[k];
        }
    }
    return run;
}

// Per (pair, frame, tile), one thread each: exclusive prefix of the chunk
// histograms over the chunks, in place (each chunk's first slot inside the
// tile's list), and the tile's total.  Consecutive threads take consecutive
// tiles, so every chunk row is read and written with coalesced accesses.  With
// live counts only the chunks that hold a live slot are scanned (the count and
// scatter passes of the others return at once).
__global__ void __launch_bounds__(256)
scan_chunks(const PairLayout* __restrict__ L, int n_pairs, uint32_t* __restrict__ hist,
            uint32_t* __restrict__ tile_count, int64_t tiles_total, const int32_t* __restrict__ live, int chunk)
{
    const int f = blockIdx.y;
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gt >= tiles_total) return;
    const int p = find_pair_by_tile(L, n_pairs, gt);
    const PairLayout PL = L[p];
    const int nt = PL.ntx * PL.nty;
    const int t = (int)(gt - PL.tile_base);
    const int nc = live ? min(PL.n_chunks, (max(live[p], 0) + chunk - 1) / chunk) : PL.n_chunks;
    const uint32_t run = scan_column(hist + PL.hist_base + (int64_t)f * PL.n_chunks * nt + t, nt, nc);
    tile_count[f * tiles_total + gt] = run;
}

// Exclusive scan over a workgroup of SCAN_THREADS.
constexpr int SCAN_THREADS = 1024;

__device__ __forceinline__ uint32_t block_before(uint32_t v, uint32_t* s_wave, uint32_t& total)
{
    const int wid = threadIdx.x >> 6;
    const uint32_t inc = wave_scan(v);
    if ((threadIdx.x & 63) == 63) s_wave[wid] = inc;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
        const uint32_t sw = s_wave[w];
        if (w < wid) before += sw;
        total += sw;
    }
    __syncthreads();
    return before + inc - v;
}

// Per (pair, frame): exclusive scan of the tile totals -> absolute offsets of
// the tile lists (the pair-frame segment's base plus the prefix).
__global__ void __launch_bounds__(SCAN_THREADS)
scan_tiles(const PairLayout* __restrict__ L, const uint32_t* __restrict__ tile_count,
           int64_t* __restrict__ tile_offset, int64_t tiles_total)
{
    __shared__ uint32_t s_wave[SCAN_THREADS / 64];
    const int p = blockIdx.x;
    const int f = blockIdx.y;
    const PairLayout PL = L[p];
    const int nt = PL.ntx * PL.nty;
    const uint32_t* cnt = tile_count + f * tiles_total + PL.tile_base;
    int64_t* out = tile_offset + f * tiles_total + PL.tile_base;
    int64_t carry = PL.entry_base + (int64_t)f * PL.entry_cap;
    for (int b = 0; b < nt; b += SCAN_THREADS) {
        const int t = b + threadIdx.x;
        uint32_t total;
        const uint32_t before = block_before(t < nt ? cnt[t] : 0u, s_wave, total);
        if (t < nt) out[t] = carry + (int64_t)before;
        carry += total;
    }
}

// Both scans in one launch, one workgroup per (pair, frame): where a pair has few
// chunks the walk over them is short, and the launch it saves is worth more
// (SCAN_FUSED steps of chunks x 1024 tiles, about 0.2 us each).
constexpr int SCAN_FUSED = 64;

__global__ void __launch_bounds__(SCAN_THREADS)
scan_pair(const PairLayout* __restrict__ L, uint32_t* __restrict__ hist, uint32_t* __restrict__ tile_count,
          int64_t* __restrict__ tile_offset, int64_t tiles_total, const int32_t* __restrict__ live, int chunk)
{
    __shared__ uint32_t s_wave[SCAN_THREADS / 64];
    const int p = blockIdx.x;
    const int f = blockIdx.y;
    const PairLayout PL = L[p];
    const int nt = PL.ntx * PL.nty;
    const int nc = live ? min(PL.n_chunks, (max(live[p], 0) + chunk - 1) / chunk) : PL.n_chunks;
    int64_t carry = PL.entry_base + (int64_t)f * PL.entry_cap;
    for (int b = 0; b < nt; b += SCAN_THREADS) {
        const int t = b + threadIdx.x;
        const uint32_t run = t < nt ? scan_column(hist + PL.hist_base + (int64_t)f * PL.n_chunks * nt + t, nt, nc) : 0u;
        uint32_t total;
        const uint32_t before = block_before(run, s_wave, total);
        if (t < nt) {
            tile_count[f * tiles_total + PL.tile_base + t] = run;
            tile_offset[f * tiles_total + PL.tile_base + t] = carry + (int64_t)before;
        }
        carry += total;
    }
}

// ------------------------------------------------------------------ render

// Threads of a renderer workgroup, and particles staged per pass (one per thread):
// 512 for tiles of 4096 pixels, so that the four of them a CU's LDS holds still
// fill its 32 wave slots; one wave for tiles of at most 256, whose lists would leave
// the others idle (16 pairs of 512^2, d about 2.5: 16 x 16 tiles 88 -> 47 us, 8 x 8 265 ->
// 108).
constexpr int render_threads(int tw, int th) { return tw * th >= 4096 ? 512 : tw * th <= 256 ? 64 : 256; }

// Whether a tile's patches may fill most of its rows (`WIDE`): they then lie over one
// another, so lanes that walk them in step add to the same words.  Each lane starts at a
// row of its own, four lanes take a patch's rows in turn, and the columns go in blocks.  16
// pairs of 512^2 with d 4 to 16, 3x3 blur, in step / so, in us: 64 x 64 tiles 234 / 162, 64
// x 32 330 / 200, 32 x 32 464 / 220, 16 x 16 784 / 320, 8 x 8 1933 / 613; one pair with 64 x
// 64, 3x3 / 7x7 blur 54 / 76 -> 39 / 52; d to 9 with 128 x 32 96 / 85.  Where d is about 2.5
// all the same the walk of its own costs 7 %, with registers for both forms in one kernel 6 %.
constexpr bool wide_patches(int th, float d_max) { return 4.5f * d_max > (float)th; }
constexpr int SLACK = 24;       // accumulator words past the region and one more row (zero columns and rows
                                // may overrun it)
constexpr int SIZES = 64;       // patch sizes told apart when a pass is sorted

__device__ __forceinline__ uint32_t pack_box(int c0, int w, int r0, int h)
{
    return (uint32_t)c0 | ((uint32_t)w << 8) | ((uint32_t)r0 << 16) | ((uint32_t)h << 24);
}

// K columns of one particle's patch, from column fx on, over its rows j, j + 2^lp,
// ..: the column factors stay in registers (zero past the patch's pw columns),
// each row's factor is formed as the row is added.  fx, fy: the first column's
// and row j's pixel centres (exact in binary32, so adding small integers to
// them gives every other centre exactly).  TURN: from a row of the lane's own on, back to
// the first behind the last.
template <int K, int RS, bool TURN>
__device__ __forceinline__ void splat_columns(uint32_t* dst, float fx, float x, float kx, int pw, float fy, float y,
                                              float ky, float Af, int j, int h, int lp, int lane)
{
    float gx[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float dx = (fx + (float)k) - x;
        const float g = expneg_lt80(kx * (dx * dx));
        gx[k] = k < pw ? g : 0.0f;
    }
    const int step = 1 << lp;
    const int n = TURN ? (h - j + step - 1) >> lp : 0;      // the lane's rows
    int r = TURN ? (lane * n) >> 6 : 0, left = n;
    if (TURN) {
        dst += r * step * RS;
        fy += (float)(r * step);
    }
#pragma unroll 1
    while (TURN ? left > 0 : j < h) {
        const float dy = fy - y;
        const float rv = Af * expneg_lt80(ky * (dy * dy));
#pragma unroll
        for (int k = 0; k < K; ++k) atomicAdd(dst + k, (uint32_t)(rv * gx[k]));
        int to = step;
        if (TURN) {
            const bool last = ++r == n;
            to = last ? (1 - n) * step : step;
            r = last ? 0 : r;
            --left;
        } else {
            j += step;
        }
        fy += (float)to;
        dst += to * RS;
    }
}

// The same with two lanes per particle, a the lane's place in its pair: lane a adds
// the columns a, a + 2, .. and forms the factors of the rows a, a + 2, .., which
// the pair exchanges.
template <int N>
__device__ __forceinline__ float pair_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), N ? 0xF5 : 0xA0, 0xF, 0xF, false));
}

template <int K, int RS>
__device__ __forceinline__ void splat_pairs(uint32_t* dst, float fx, float x, int pw, float fy, float y, float kappa,
                                            float Af, int a, int h)
{
    float gx[K / 2];
#pragma unroll
    for (int k = 0; k < K / 2; ++k) {
        const float dx = (fx + (float)(2 * k)) - x;
        const float g = expneg_lt80(kappa * (dx * dx));
        gx[k] = 2 * k + a < pw ? g : 0.0f;
    }
#pragma unroll 1
    for (int j = 0; j < h; j += 2) {
        const float dy = fy - y;
        float rv = Af * expneg_lt80(kappa * (dy * dy));
        rv = j + a < h ? rv : 0.0f;
        const float r0 = pair_lane<0>(rv), r1 = pair_lane<1>(rv);
#pragma unroll
        for (int k = 0; k < K / 2; ++k) atomicAdd(dst + 2 * k, (uint32_t)(r0 * gx[k]));
#pragma unroll
        for (int k = 0; k < K / 2; ++k) atomicAdd(dst + RS + 2 * k, (uint32_t)(r1 * gx[k]));
        fy += 2.0f;
        dst += 2 * RS;
    }
}

// Tile renderer, templated on the tile shape and the blur radius (tile-local
// index arithmetic becomes shifts, blur loops unroll).  ANISO: the full model's
// particle images (Eq. 1 with sigma_y = d_y / 4 and rho, from the shape
// records): kappa_x = 8 / (om d^2), kappa_y = 8 / (om d_y^2), om = 1 - rho^2;
// rho = 0 keeps the separable factors (with kappa_y for the rows), rho != 0
// evaluates exp(-q) per pixel, q = dx (kappa_x dx + kappa_xy dy) + kappa_y dy^2,
// kappa_xy = -16 rho / (om d d_y); the patch is |dx| <= 1.5 d, |dy| <= 1.5 d_y.
//
// The tile's particles are staged in LDS up to 64, 256 or 512 at a time, one per thread,
// sorted by patch size (a counting sort on LDS counters), and splatted one
// particle per lane: a lane keeps its patch's column factors in registers and
// walks down the rows, so an exponential is computed once per patch column and
// row and no factor passes through LDS.  The sort makes a wave's 64 patches
// nearly equal, so few lanes idle.  Lists that leave most of a wave empty give
// each particle 2 or 4 lanes, which take its rows in turn.
// Bound by VALU issue (exponentials, products, the epilogue's draws), with the
// LDS adds close behind (7.4 clocks per wave at 64 unrelated addresses, 6.5 at
// eight rows of eight patches: the order of the lanes hardly matters).  Measured
// with 64 x 32 tiles against one patch row per lane with the column factors in an
// LDS table: 64 pairs of 1024^2 at 0.05 ppp, 3x3 blur, noise: 505 -> 385 us; 32
// pairs of 2048^2 at 0.1 ppp, d to 6, 5x5 blur: 2.97 -> 2.31 ms; uneven pairs, ppp
// to 0.1: 940 -> 664 us; with 64 x 64 tiles 340 us, 1.96 ms and 612 us, and with
// wide patches by pairs of lanes 341 us, 1.83 ms and 621 us.  Of the first, the
// epilogue takes about 150 us.  Sorting by width alone or by an
// estimate of the work was slower (397 and 408 us with 64 x 32 tiles).
template <int TW, int TH, int B, bool ANISO, bool PERSIST, bool WIDE>
__global__ void __launch_bounds__(render_threads(TW, TH)) __attribute__((amdgpu_waves_per_eu(PERSIST ? 6 : 8)))
render_tile(const synthpix_pair* __restrict__ pairs, const PairLayout* __restrict__ L, int n_pairs,
            const float4* __restrict__ rec0, const float4* __restrict__ rec1, const uint2* __restrict__ box0,
            const uint2* __restrict__ box1, const float2* __restrict__ shp0,
            const float2* __restrict__ shp1, EpilogueArgs a, int spread,
            const uint32_t* __restrict__ tile_count, const int64_t* __restrict__ tile_offset,
            const int32_t* __restrict__ entries, int64_t tiles_total, uint32_t* __restrict__ status,
            uint32_t* __restrict__ queue)
{
    static_assert(TW % 4 == 0 && (TW & (TW - 1)) == 0 && (TH & (TH - 1)) == 0, "power-of-two tiles");
    static_assert(TW + 6 < 256 && TH + 6 < 256, "patch boxes are packed in bytes");
    static_assert(B >= 0 && B <= 3, "blur radius 0..3");
    constexpr int NT = render_threads(TW, TH), STAGE = NT;
    constexpr int Q4 = TW / 4;
    constexpr int RW = TW + 2 * B;
    constexpr int RH = TH + 2 * B;
    // words from row to row: those of rows that are a whole number of bank cycles long fall
    // on one bank (d 4 to 16, no blur, 16 pairs of 512^2: 369 us, so 152, lanes in step 276)
    constexpr int RS = WIDE && B == 0 ? RW + 2 : RW;
    constexpr int ACC = ((RH + 1) * RS + SLACK + 3) & ~3;
    constexpr int STAGE_BYTES = STAGE * (16 + 4 + (ANISO ? 8 : 0));
    constexpr int BLUR_BYTES = B > 0 ? RH * TW * 4 : 0;
    float wb[2 * B + 1];
#pragma unroll
    for (int q = 0; q <= 2 * B; ++q) wb[q] = a.blur_w[q];
    __shared__ __align__(16) uint32_t acc[ACC];
    __shared__ __align__(16) unsigned char work[STAGE_BYTES > BLUR_BYTES ? STAGE_BYTES : BLUR_BYTES];
    float4* stg = reinterpret_cast<float4*>(work);                  // (x, y, kappa_x, Af)
    float2* stg2 = reinterpret_cast<float2*>(stg + STAGE);          // (kappa_y, kappa_xy), ANISO only
    uint32_t* box = reinterpret_cast<uint32_t*>(work + STAGE * (ANISO ? 24 : 16));   // c0 | w | r0 | h bytes
    float* tmp = reinterpret_cast<float*>(work);                    // blur scratch, reuses the staging
    __shared__ uint32_t s_hist[2][SIZES];       // particles of each patch size, by pass parity
    __shared__ uint32_t s_live[2];              // particles with pixels in the region, by pass parity
    // fixed-point range bound: every term a particle adds to a pixel is at most its
    // integer peak, so the peaks of the particles that touch a band of rows bound
    // its pixel sums.  Only where some band's sum (in units of 256, each peak
    // rounded up) reaches 2^32 are the rows summed one by one.
    constexpr int BAND = 16, BANDS = (RH + BAND - 1) / BAND;
    __shared__ unsigned long long s_band[BANDS];
    __shared__ uint32_t s_over;

    // PERSIST: a persistent work list.  Each workgroup pops (frame, tile) items
    // from the queue of its XCD until the queue is empty; the items of one XCD
    // form a contiguous range (workgroups are dispatched to the 8 XCDs
    // round-robin), so the neighbouring tiles in flight on an XCD share particle
    // records in its L2, and the grid is at most what the chip holds at once.
    // Otherwise one item per workgroup, numbered XCD-contiguously.
    __shared__ unsigned s_pop;
    uint64_t pid_base = 0;
    if (a.iod) {
        a.images = a.iod->images;
        a.seed = a.iod->seed;
        pid_base = a.iod->pair_id_base;
    }
    const unsigned n_items = (unsigned)(2 * tiles_total);
    const bool split = gridDim.x >= 8;
    const unsigned xq = split ? (blockIdx.x & 7u) : 0u;
    const unsigned q8 = n_items >> 3, r8 = n_items & 7u;
    const unsigned lo = split ? (xq < r8 ? xq * (q8 + 1) : r8 * (q8 + 1) + (xq - r8) * q8) : 0u;
    const unsigned len = split ? (xq < r8 ? q8 + 1 : q8) : n_items;
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    for (;;) {
    int64_t item;
    if (PERSIST) {
        if (t == 0) s_pop = atomicAdd(&queue[xq], 1u);
        __syncthreads();
        const unsigned kq = (unsigned)__builtin_amdgcn_readfirstlane((int)s_pop);   // uniform: one scalar value
        if (kq >= len) break;             // the same value in every thread of the workgroup
        item = (int64_t)lo + kq;
    } else {
        item = xcd_contiguous(blockIdx.x, gridDim.x);
    }
    const int f = item >= tiles_total ? 1 : 0;
    const int64_t tile = item - (int64_t)f * tiles_total;
    const int p = find_pair_by_tile(L, n_pairs, tile);
    const int pW = pairs[p].W, pH = pairs[p].H;
    const int64_t p_off = pairs[p].particle_offset, p_img = pairs[p].image_offset;
    const uint64_t pid = pairs[p].pair_id + pid_base;
    const int64_t tile_base = L[p].tile_base;
    const int ntx = L[p].ntx;
    const int tl = (int)(tile - tile_base);
    const int ty = tl / ntx;
    const int tx = tl - ty * ntx;
    const int rx0 = tx * TW - B;          // region origin in image pixels
    const int ry0 = ty * TH - B;
    if (tl == 0 && t == 0) {
        const uint32_t fl = (L[p].flags >> (8 * f)) & 255u;      // raised by the small pairs' binning
        if (fl) atomicOr(status, fl);
    }
    const int cnt = (int)tile_count[item];
    const int32_t* __restrict__ list = entries + tile_offset[item];
    const float4* __restrict__ rec = (f ? rec1 : rec0) + p_off;
    const uint2* __restrict__ bxs = (f ? box1 : box0) + p_off;
    const float2* __restrict__ shp = (f ? shp1 : shp0) + p_off;

    for (int k = t; k < ACC / 4; k += NT) reinterpret_cast<uint4*>(acc)[k] = make_uint4(0u, 0u, 0u, 0u);
    for (int k = t; k < 2 * SIZES; k += NT) (&s_hist[0][0])[k] = 0u;
    if (t < 2) s_live[t] = 0u;
    if (t < BANDS) s_band[t] = 0ull;
    if (t == 0) s_over = 0u;
    __syncthreads();

    // particle e's patch box (image pixels) clipped to the region
    auto clip = [&](int e, int& w, int& h, int& c0, int& r0) {
        const uint2 pb = bxs[e];
        const int a0 = max((int)(pb.x & 0xffffu), rx0), a1 = min((int)(pb.x >> 16), rx0 + RW - 1);
        const int b0 = max((int)(pb.y & 0xffffu), ry0), b1 = min((int)(pb.y >> 16), ry0 + RH - 1);
        if (!box_empty(pb) && a0 <= a1 && b0 <= b1) {
            w = a1 - a0 + 1;
            h = b1 - b0 + 1;
            c0 = a0 - rx0;
            r0 = b0 - ry0;
        }
    };

    for (int base = 0, par = 0; base < cnt; base += STAGE, par ^= 1) {
        // one particle per thread
        float4 r = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float2 rs = make_float2(0.0f, 0.0f);
        int w = 0, h = 0, c0 = 0, r0 = 0, size = 0;
        uint32_t rank = 0;
        const bool some = base + wave * 64 < cnt;        // the wave has particles (uniform)
        if (some) {
            if (base + t < cnt) {
                const int e = list[base + t];
                r = rec[e];
                if (ANISO) rs = shp[e];
                clip(e, w, h, c0, r0);
            }
            size = min(max(w, h), SIZES - 1);
            const uint32_t in_wave = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(w > 0));
            if (lane == 0) atomicAdd(&s_live[par], in_wave);
            if (w > 0) {
                rank = atomicAdd(&s_hist[par][size], 1u);
                const unsigned long long peak = (uint32_t)(r.w * 0x1p-8f) + 1u;
                for (int k = r0 / BAND; k <= (r0 + h - 1) / BAND; ++k)
                    if (atomicAdd(&s_band[k], peak) + peak >= (1ull << 24)) s_over = 1u;
            }
        }
        __syncthreads();
        const int n = __builtin_amdgcn_readfirstlane((int)s_live[par]);
        if (some) {
            // largest patches first: lane l of the wave scans size SIZES - 1 - l
            const uint32_t inc = wave_scan(s_hist[par][SIZES - 1 - lane]);
            const uint32_t above = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * (SIZES - 2 - size), (int)inc);
            if (w > 0) {
                const int slot = (int)((size < SIZES - 1 ? above : 0u) + rank);
                stg[slot] = r;
                if (ANISO) stg2[slot] = rs;
                box[slot] = pack_box(c0, w, r0, h);
            }
        }
        __syncthreads();
        if (t < SIZES) s_hist[par][t] = 0u;      // next used two passes on, past a barrier
        if (t == 0) s_live[par] = 0u;
        // lanes per particle: 1, or 2 or 4 where the particles then still fit in `spread`
        // lanes; 4 for the full model, whose patches (two diameters, an exponential per
        // pixel) the sort leaves uneven (16 pairs of 1024^2: 1 / 4 / 8 lanes 187 / 146 /
        // 155 us, one patch row per lane 177)
        const int lp = ANISO || WIDE || 4 * n <= spread ? 2 : 2 * n <= spread ? 1 : 0;
        for (int s0 = wave * (64 >> lp); s0 < n; s0 += (NT / 64) * (64 >> lp)) {
            const int slot = s0 + (lane >> lp);
            const int step = 1 << lp, j = lane & (step - 1);
            const bool on = slot < n;
            const uint32_t bx = on ? box[slot] : 0u;
            const float4 sf = stg[on ? slot : s0];
            const int pc0 = (int)(bx & 255u), pw = (int)((bx >> 8) & 255u);
            const int pr0 = (int)((bx >> 16) & 255u), ph = (int)(bx >> 24);
            uint32_t* dst = acc + (pr0 + j) * RS + pc0;
            const float fx = (float)(rx0 + pc0) + 0.5f, fy = (float)(ry0 + pr0 + j) + 0.5f;
            float ky = sf.z;
            int hs = ph;
            if (ANISO) {
                const float2 s2 = stg2[on ? slot : s0];
                ky = s2.x;
                if (s2.y != 0.0f) {
                    // rho != 0: one exponential per pixel of the row
                    float fr = fy;
                    for (int jr = j; jr < ph; jr += step) {
                        const float dy = fr - sf.y;
                        const float ra = s2.y * dy, rb = s2.x * (dy * dy);
                        uint32_t* dr = dst + (jr - j) * RS;
                        float fc = fx;
                        for (int c = 0; c < pw; ++c) {
                            const float dx = fc - sf.x;
                            const float q = __builtin_fmaxf(__builtin_fmaf(dx, __builtin_fmaf(sf.z, dx, ra), rb), 0.0f);
                            atomicAdd(dr + c, (uint32_t)(sf.w * expneg(q)));
                            fc += 1.0f;
                        }
                        fr += (float)step;
                    }
                    hs = 0;                       // nothing left for the separable form
                }
                if (__builtin_amdgcn_ballot_w64(hs > 0) == 0) continue;
            }
#define SP_SPLAT(K_) splat_columns<K_, RS, WIDE>(dst, fx, sf.x, sf.z, pw, fy, sf.y, ky, sf.w, j, hs, lp, lane)
            if (!__builtin_amdgcn_ballot_w64(pw > 4)) SP_SPLAT(4);
            else if (!__builtin_amdgcn_ballot_w64(pw > 6)) SP_SPLAT(6);
            else if (!__builtin_amdgcn_ballot_w64(pw > 8)) SP_SPLAT(8);
            else if (!__builtin_amdgcn_ballot_w64(pw > 10)) SP_SPLAT(10);
            else if (!__builtin_amdgcn_ballot_w64(pw > 12)) SP_SPLAT(12);
            else if constexpr (ANISO || WIDE) {
                // blocks of at most 12 columns that a patch as wide as the region fills
                constexpr int NB = (RW + 11) / 12, K = ANISO ? 12 : (RW + NB - 1) / NB;
                for (int cb = 0; __builtin_amdgcn_ballot_w64(pw > cb) != 0; cb += K)
                    splat_columns<K, RS, WIDE>(dst + cb, fx + (float)cb, sf.x, sf.z, pw - cb, fy, sf.y, ky, sf.w, j,
                                               pw > cb ? hs : 0, lp, lane);
            } else {
                // wide patches: two lanes per particle, 32 particles at a time.  The adds of
                // a pair fall on neighbouring banks, and half the columns need half the
                // registers.  From 13 columns on, as narrower patches gain less than the
                // pairs' set-up (32 pairs of 2048^2 with d to 6 / 64 of 1024^2 with d about
                // 2.5: from 7 columns 1.85 ms / 362 us, from 13 1.83 / 341, from 17 1.91 /
                // 343, never 1.96 / 342).
                const int e0 = min(s0 + (64 >> lp), n);
#pragma unroll 1
                for (int s2 = s0 + (lane >> 1); __builtin_amdgcn_ballot_w64(s2 < e0) != 0; s2 += 32) {
                    const bool on2 = s2 < e0;
                    const int a2 = lane & 1;
                    const uint32_t b2 = on2 ? box[s2] : 0u;
                    const float4 f2 = stg[on2 ? s2 : s0];
                    const int qc0 = (int)(b2 & 255u), qw = (int)((b2 >> 8) & 255u);
                    const int qr0 = (int)((b2 >> 16) & 255u), qh = (int)(b2 >> 24);
                    uint32_t* d2 = acc + qr0 * RS + qc0 + a2;
                    const float gx0 = (float)(rx0 + qc0 + a2) + 0.5f, gy0 = (float)(ry0 + qr0 + a2) + 0.5f;
#define SP_PAIRS(K_) splat_pairs<K_, RS>(d2, gx0, f2.x, qw, gy0, f2.y, f2.z, f2.w, a2, qh)
                    if (!__builtin_amdgcn_ballot_w64(qw > 12)) SP_PAIRS(12);
                    else if (!__builtin_amdgcn_ballot_w64(qw > 16)) SP_PAIRS(16);
                    else if (!__builtin_amdgcn_ballot_w64(qw > 20)) SP_PAIRS(20);
                    else
                        for (int cb = 0; __builtin_amdgcn_ballot_w64(qw > cb) != 0; cb += 20)
                            splat_pairs<20, RS>(d2 + cb, gx0 + (float)cb, f2.x, qw - cb, gy0, f2.y, f2.z, f2.w, a2,
                                                qw > cb ? qh : 0);
#undef SP_PAIRS
                }
            }
#undef SP_SPLAT
        }
    }
    __syncthreads();
    if (s_over) {
        // a difference array over the region's rows (each peak added over the rows
        // its patch covers), its prefix sums by wave 0: flag a row whose bound
        // reaches 2^32
        unsigned long long* rows = reinterpret_cast<unsigned long long*>(work);
        static_assert((RH + 1) * 8 <= STAGE_BYTES, "the row sums reuse the staging");
        for (int k = t; k <= RH; k += NT) rows[k] = 0ull;
        __syncthreads();
        for (int k = t; k < cnt; k += NT) {
            const int e = list[k];
            int w = 0, h = 0, c0 = 0, r0 = 0;
            clip(e, w, h, c0, r0);
            if (w > 0) {
                const unsigned long long pk = (unsigned long long)rec[e].w;
                atomicAdd(&rows[r0], pk);
                atomicAdd(&rows[r0 + h], 0ull - pk);
            }
        }
        __syncthreads();
        if (t < 64) {
            unsigned long long carry = 0ull, top = 0ull;
            for (int c = 0; c <= RH; c += 64) {
                unsigned long long v = c + lane <= RH ? rows[c + lane] : 0ull;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const unsigned long long u = __shfl_up(v, o, 64);
                    if (lane >= o) v += u;
                }
                v += carry;
                top = v > top ? v : top;
                carry = __shfl(v, 63, 64);
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                const unsigned long long u = __shfl_xor(top, o, 64);
                top = u > top ? u : top;
            }
            if (lane == 0 && top >= (1ull << 32)) atomicOr(status, SP_STATUS_FIXED_RANGE);
        }
        __syncthreads();
    }

    // fixed point -> float happens as the blur / store passes read the accumulator
    constexpr float FIX = 0x1p-24f;
    if constexpr (B > 0) {
        // horizontal pass over all region rows: four tile columns per work item
#pragma unroll
        for (int k0 = 0; k0 < RH * Q4; k0 += NT) {
            const int k = k0 + t;
            if (k0 + NT > RH * Q4 && k >= RH * Q4) break;
            const int r = k / Q4;
            const int c = (k % Q4) * 4;
            // the fixed-point scale rides on the weights: w (v 2^-24) and (w 2^-24) v
            // are the same binary32 products (exact power-of-two scaling, no underflow)
            const uint32_t* src = acc + r * RS + c;
            float vv[4 + 2 * B];
#pragma unroll
            for (int q = 0; q < 4 + 2 * B; ++q) vv[q] = (float)src[q];
            float o0 = 0.0f, o1 = 0.0f, o2 = 0.0f, o3 = 0.0f;
#pragma unroll
            for (int q = 0; q <= 2 * B; ++q) {
                const float wq = wb[q] * FIX;
                o0 = __builtin_fmaf(wq, vv[q], o0);
                o1 = __builtin_fmaf(wq, vv[q + 1], o1);
                o2 = __builtin_fmaf(wq, vv[q + 2], o2);
                o3 = __builtin_fmaf(wq, vv[q + 3], o3);
            }
            *reinterpret_cast<float4*>(tmp + r * TW + c) = make_float4(o0, o1, o2, o3);
        }
        __syncthreads();
    }

    // vertical pass, noise, codes, store: four consecutive pixels per work item,
    // addressed from the tile's first pixel (offsets fit 32 bits; the stores are
    // whole vectors at any alignment)
    const int Wq = (pW + 3) >> 2;
    const float Lq = a.bits > 0 ? (float)((1u << a.bits) - 1u) : 0.0f;
    const bool noisy = a.noise_sigma > 0.0f;
    typedef __attribute__((address_space(1))) unsigned char gbyte;
    typedef uint32_t codes4 __attribute__((ext_vector_type(2), aligned(2)));
    typedef float pixels4 __attribute__((ext_vector_type(4), aligned(4)));
    const int64_t first = p_img + (int64_t)f * ((int64_t)pH * pW) + (int64_t)(ty * TH) * pW + tx * TW;
    gbyte* img = (gbyte*)a.images + first * (a.bits > 0 ? 2 : 4);
#pragma unroll
    for (int k0 = 0; k0 < TH * Q4; k0 += NT) {
        const int gi = k0 + t;
        if (k0 + NT > TH * Q4 && gi >= TH * Q4) break;
        const int r = gi / Q4, q4 = gi % Q4, c4 = 4 * q4;
        const int left = pW - (tx * TW + c4);                // pixels from here to the image's edge
        if (ty * TH + r >= pH || left <= 0) continue;
        float o[4];
        if constexpr (B > 0) {
            float4 s4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
            for (int q = 0; q <= 2 * B; ++q) {
                const float wq = wb[q];
                const float4 t4 = *reinterpret_cast<const float4*>(tmp + (r + q) * TW + c4);
                s4.x = __builtin_fmaf(wq, t4.x, s4.x);
                s4.y = __builtin_fmaf(wq, t4.y, s4.y);
                s4.z = __builtin_fmaf(wq, t4.z, s4.z);
                s4.w = __builtin_fmaf(wq, t4.w, s4.w);
            }
            o[0] = s4.x; o[1] = s4.y; o[2] = s4.z; o[3] = s4.w;
        } else {
            const uint32_t* src = acc + r * RS + c4;
            o[0] = (float)src[0] * FIX; o[1] = (float)src[1] * FIX;
            o[2] = (float)src[2] * FIX; o[3] = (float)src[3] * FIX;
        }
        if (noisy) {
            const u32x4 w = draw((uint32_t)((ty * TH + r) * Wq + ((tx * TW) >> 2) + q4), STREAM_NOISE0 + f, pid, a.seed);
            const uint32_t wa[2] = {w.a, w.c};
            const uint32_t wb[2] = {w.b, w.d};
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const float u1 = u24_open0(wa[h2]);
                const float u2 = u24(wb[h2]);
                // v_log_f32 is log2 (so -2 ln u = -2 ln2 log2 u); v_sin/v_cos take revolutions
                const float rad = __builtin_amdgcn_sqrtf(-1.38629436111989061883f * __builtin_amdgcn_logf(u1));
                o[2 * h2] = __builtin_fmaf(a.noise_sigma, rad * __builtin_amdgcn_cosf(u2), o[2 * h2]);
                o[2 * h2 + 1] = __builtin_fmaf(a.noise_sigma, rad * __builtin_amdgcn_sinf(u2), o[2 * h2 + 1]);
            }
        }
        const uint32_t at = (uint32_t)r * (uint32_t)pW + (uint32_t)c4;
        if (a.bits > 0) {
            // clamp to [0, L] with one median, then round to even by adding 2^23: the code
            // is the sum's low half (rounding a clamped value clamps the rounded one)
            uint32_t qv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                qv[e] = __float_as_uint(__builtin_amdgcn_fmed3f(o[e] * Lq, 0.0f, Lq) + 8388608.0f);
            gbyte* dst = img + 2 * at;
            if (left >= 4) {
                const codes4 v = {__builtin_amdgcn_perm(qv[1], qv[0], 0x05040100u),
                                  __builtin_amdgcn_perm(qv[3], qv[2], 0x05040100u)};
                *(__attribute__((address_space(1))) codes4*)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < left) *(__attribute__((address_space(1))) uint16_t*)(dst + 2 * e) = (uint16_t)qv[e];
            }
        } else {
            gbyte* dst = img + 4 * at;
            if (left >= 4) {
                const pixels4 v = {o[0], o[1], o[2], o[3]};
                *(__attribute__((address_space(1))) pixels4*)dst = v;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < left) *(__attribute__((address_space(1))) float*)(dst + 4 * e) = o[e];
            }
        }
    }
    if (!PERSIST) break;
    // the next item's accumulator reset and queue pop wait for this epilogue
    __syncthreads();
    }
}

// Tile shapes with a compiled renderer (width x height).
bool render_shape_supported(int tw, int th)
{
    switch (tw * 1000 + th) {
    case 8008: case 16016: case 32016: case 32032: case 64016: case 64032: case 64064: case 128032:
        return true;
    default:
        return false;
    }
}

// ------------------------------------------------------------------ launcher

static void launch_scans(const PairLayout* L, int n_pairs, uint32_t* hist, const BatchTotals& tot,
                         uint32_t* tile_count, int64_t* tile_offset, int frames, hipStream_t s, const int32_t* live,
                         int chunk)
{
    const int64_t tiles = tot.tiles;
    const int64_t steps = ((tot.max_n + chunk - 1) / chunk) * ((tot.max_tiles + SCAN_THREADS - 1) / SCAN_THREADS);
    if (steps <= SCAN_FUSED) {
        hipLaunchKernelGGL(scan_pair, dim3((unsigned)n_pairs, frames), dim3(SCAN_THREADS), 0, s, L, hist, tile_count,
                           tile_offset, tiles, live, chunk);
        return;
    }
    hipLaunchKernelGGL(scan_chunks, dim3((unsigned)((tiles + 255) / 256), frames), dim3(256), 0, s, L, n_pairs, hist,
                       tile_count, tiles, live, chunk);
    hipLaunchKernelGGL(scan_tiles, dim3((unsigned)n_pairs, frames), dim3(SCAN_THREADS), 0, s, L, tile_count,
                       tile_offset, tiles);
}

// Launches one renderer instantiation: one workgroup per item, or (persistent
// kernels) as many workgroups as the device holds at once, from the kernel's
// occupancy (cached per kernel).  The persistent form is compiled for the
// isotropic renderer; anisotropic batches run one workgroup per item.
template <typename K, typename... Args>
static void launch_tile_kernel(K kernel, dim3 grid, int threads, hipStream_t s, bool persistent, Args... args)
{
    if (persistent) {
        static std::mutex mu;
        static std::map<const void*, int> cache;
        int per_cu = 0;
        {
            std::lock_guard<std::mutex> lk(mu);
            const void* key = reinterpret_cast<const void*>(kernel);
            auto it = cache.find(key);
            if (it == cache.end()) {
                if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess)
                    per_cu = 0;
                cache[key] = per_cu;
            } else {
                per_cu = it->second;
            }
        }
        if (per_cu > 0) {
            const unsigned cap = (unsigned)per_cu * (unsigned)device_cu_count();
            if (grid.x > cap) grid.x = cap;
        }
    }
    hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, args...);
}

template <int TW, int TH>
static void launch_render_shape(dim3 grid, hipStream_t s, const RenderArgs& a, const RenderConfig& cfg,
                                const PairLayout* L, const float4* r0, const float4* r1, const uint2* b0,
                                const uint2* b1, const float2* h0, const float2* h1, const uint32_t* tile_count,
                                const int64_t* tile_offset, const int32_t* entries, int64_t tiles, uint32_t* status)
{
    EpilogueArgs ea;
    ea.images = a.images;
    ea.noise_sigma = a.noise_sigma;
    ea.bits = a.bits;
    ea.seed = a.seed;
    ea.iod = a.iod;
    for (int q = 0; q < 7; ++q) ea.blur_w[q] = a.blur_w[q];
    // a grid of under 1024 threads per CU leaves most of the chip idle and spreads a
    // tile's particles over all its waves (a shorter walk), a larger one over as
    // few waves as hold them (less work in all)
    const int threads = render_threads(TW, TH);
    const int spread = (int64_t)grid.x * threads < (int64_t)1024 * device_cu_count() ? threads : 64;
#define SP_TILE(B_, ANISO_, PERSIST_, WIDE_)                                                                         \
    launch_tile_kernel(render_tile<TW, TH, B_, ANISO_, PERSIST_, WIDE_>, grid, threads, s, PERSIST_, a.pairs, L,     \
                       a.n_pairs, r0, r1, b0, b1, h0, h1, ea, spread, tile_count, tile_offset, entries, tiles,      \
                       status, status + 8)
    const bool wide = wide_patches(TH, cfg.d_max);
#define SP_B(B_)                                                                                                    \
    case B_:                                                                                                        \
        if (a.aniso) SP_TILE(B_, true, false, false);                                                               \
        else if (cfg.persistent && wide) SP_TILE(B_, false, true, true);                                            \
        else if (cfg.persistent) SP_TILE(B_, false, true, false);                                                   \
        else if (wide) SP_TILE(B_, false, false, true);                                                             \
        else SP_TILE(B_, false, false, false);                                                                      \
        break;
    switch (cfg.apron) { SP_B(0) SP_B(1) SP_B(2) SP_B(3) default: break; }
#undef SP_B
#undef SP_TILE
}

// Whether one workgroup per pair (and frame) bins a batch.
static bool small_pairs(const BatchTotals& tot, int most)
{
    return tot.max_n <= most && tot.max_tiles <= SMALL_TILES;
}

hipError_t launch_bins(const RenderArgs& a, const RenderConfig& cfg, const BatchTotals& tot, char* ws,
                       const WorkspaceLayout& wl, hipStream_t s)
{
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + wl.status);
    PairLayout* L = reinterpret_cast<PairLayout*>(ws + wl.layout);
    uint32_t* tile_count = reinterpret_cast<uint32_t*>(ws + wl.tile_count);
    int64_t* tile_offset = reinterpret_cast<int64_t*>(ws + wl.tile_offset);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + wl.hist);
    int32_t* entries = reinterpret_cast<int32_t*>(ws + wl.entries);
    float4* rec0 = reinterpret_cast<float4*>(ws + wl.records);
    float4* rec1 = rec0 + tot.n_span;
    uint2* box0 = reinterpret_cast<uint2*>(ws + wl.boxes);
    uint2* box1 = box0 + tot.n_span;
    float2* shp0 = reinterpret_cast<float2*>(ws + wl.shapes);
    float2* shp1 = shp0 + tot.n_span;

    const size_t hist_lds = (size_t)tot.max_tiles * sizeof(uint32_t);
    // the full model's prep writes every slot; live counts only with the isotropic prep
    const int32_t* live = a.model ? nullptr : a.live;
    if (small_pairs(tot, SMALL_BINS)) {
        TimedScope ts("bins", s);
        const int nt = small_threads(2 * (int64_t)a.n_pairs);
#define SP_BINS(MODEL_, NT_)                                                                                        \
    hipLaunchKernelGGL((bins_small<MODEL_, NT_>), dim3((unsigned)a.n_pairs, 2), dim3(NT_), hist_lds, s, a.pairs, a,  \
                       cfg, L, rec0, rec1, box0, box1, shp0, shp1, tile_count, tile_offset, tot.tiles, entries, live, \
                       status)
        if (a.model && nt == 1024) SP_BINS(true, 1024);
        else if (a.model) SP_BINS(true, 256);
        else if (nt == 1024) SP_BINS(false, 1024);
        else SP_BINS(false, 256);
#undef SP_BINS
        return hipGetLastError();
    }
    const bool inl = a.n_pairs <= INLINE_PAIRS && tot.chunks > 0;
    if (!inl) {
        TimedScope ts("bin_layout", s);
        hipLaunchKernelGGL(bin_layout, dim3(1), dim3(256), 0, s, a.pairs, a.n_pairs, cfg, L, status);
    }
    if (tot.chunks > 0) {
        TimedScope ts("bin_count", s);
        const dim3 grid((unsigned)tot.chunks), block(COUNT_THREADS);
        // seven floats per particle above half of the 256 MB last-level cache
        const bool stream = 28 * tot.n_span > (int64_t)128 << 20;
#define SP_COUNT(MODEL_, INLINE_, STREAM_)                                                                        \
    hipLaunchKernelGGL((bin_count<MODEL_, INLINE_, STREAM_>), grid, block, hist_lds, s, a.pairs, L, a.n_pairs, a,   \
                       cfg, rec0, rec1, box0, box1, shp0, shp1, hist, (unsigned)tot.chunks, live, status)
        if (a.model && inl) SP_COUNT(true, true, false);
        else if (a.model) SP_COUNT(true, false, false);
        else if (inl && stream) SP_COUNT(false, true, true);
        else if (inl) SP_COUNT(false, true, false);
        else if (stream) SP_COUNT(false, false, true);
        else SP_COUNT(false, false, false);
#undef SP_COUNT
    }
    if (tot.tiles > 0) {
        TimedScope ts("bin_scan", s);
        launch_scans(L, a.n_pairs, hist, tot, tile_count, tile_offset, 2, s, live, cfg.chunk);
    }
    if (tot.chunks > 0) {
        TimedScope ts("bin_scatter", s);
        hipLaunchKernelGGL(bin_scatter, dim3((unsigned)tot.chunks, 2), dim3(256), hist_lds, s, a.pairs, L, a.n_pairs,
                           box0, box1, cfg, hist, tile_offset, tot.tiles, entries, (unsigned)tot.chunks, live, status);
    }
    return hipGetLastError();
}

hipError_t launch_render(const RenderArgs& a, const RenderConfig& cfg, const BatchTotals& tot, char* ws,
                         const WorkspaceLayout& wl, hipStream_t s)
{
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + wl.status);
    PairLayout* L = reinterpret_cast<PairLayout*>(ws + wl.layout);
    uint32_t* tile_count = reinterpret_cast<uint32_t*>(ws + wl.tile_count);
    int64_t* tile_offset = reinterpret_cast<int64_t*>(ws + wl.tile_offset);
    int32_t* entries = reinterpret_cast<int32_t*>(ws + wl.entries);
    float4* rec0 = reinterpret_cast<float4*>(ws + wl.records);
    float4* rec1 = rec0 + tot.n_span;
    uint2* box0 = reinterpret_cast<uint2*>(ws + wl.boxes);
    uint2* box1 = box0 + tot.n_span;
    float2* shp0 = reinterpret_cast<float2*>(ws + wl.shapes);
    float2* shp1 = shp0 + tot.n_span;
    const hipError_t e = launch_bins(a, cfg, tot, ws, wl, s);
    if (e != hipSuccess) return e;
    if (tot.tiles > 0) {
        TimedScope ts("render_tile", s);
        const dim3 grid((unsigned)(2 * tot.tiles));
#define SP_SHAPE(W_, H_)                                                                                        \
    if (cfg.tile_w == W_ && cfg.tile_h == H_)                                                                   \
        launch_render_shape<W_, H_>(grid, s, a, cfg, L, rec0, rec1, box0, box1, shp0, shp1, tile_count,   \
                                    tile_offset, entries, tot.tiles, status);                                   \
    else
        SP_SHAPE(8, 8) SP_SHAPE(16, 16) SP_SHAPE(32, 16) SP_SHAPE(32, 32) SP_SHAPE(64, 16) SP_SHAPE(64, 32)
        SP_SHAPE(64, 64) SP_SHAPE(128, 32)
        return hipErrorInvalidValue;
#undef SP_SHAPE
    }
    return hipGetLastError();
}

hipError_t launch_order(const synthpix_pair* pairs_dev, int n_pairs, const float* x, const float* y,
                        const RenderConfig& cfg, const BatchTotals& tot, char* ws, const OrderLayout& ol,
                        hipStream_t s, const synthpix_batch_io* iod, const int32_t* live)
{
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + ol.status);
    PairLayout* L = reinterpret_cast<PairLayout*>(ws + ol.layout);
    uint32_t* tile_count = reinterpret_cast<uint32_t*>(ws + ol.tile_count);
    int64_t* tile_offset = reinterpret_cast<int64_t*>(ws + ol.tile_offset);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + ol.hist);
    int32_t* entries = reinterpret_cast<int32_t*>(ws + ol.entries);
    TimedScope ts("order", s);
    const size_t hist_lds = (size_t)tot.max_tiles * sizeof(uint32_t);
    if (small_pairs(tot, SMALL_ORDER)) {
        if (small_threads(n_pairs) == 1024)
            hipLaunchKernelGGL(order_small<1024>, dim3((unsigned)n_pairs), dim3(1024), hist_lds, s, pairs_dev, x, y,
                               cfg, L, tile_count, tile_offset, entries, iod, live);
        else
            hipLaunchKernelGGL(order_small<256>, dim3((unsigned)n_pairs), dim3(256), hist_lds, s, pairs_dev, x, y, cfg,
                               L, tile_count, tile_offset, entries, iod, live);
        return hipGetLastError();
    }
    const bool inl = n_pairs <= INLINE_PAIRS && tot.chunks > 0;
    if (!inl) hipLaunchKernelGGL(bin_layout, dim3(1), dim3(256), 0, s, pairs_dev, n_pairs, cfg, L, status);
    if (tot.chunks == 0) return hipGetLastError();
#define SP_ORDER(SCATTER_, INLINE_)                                                                               \
    hipLaunchKernelGGL((order_pass<SCATTER_, INLINE_>), dim3((unsigned)tot.chunks), dim3(256), hist_lds, s,        \
                       pairs_dev, L, n_pairs, x, y, cfg, hist, tile_offset, entries, (unsigned)tot.chunks, iod, live)
    if (inl) SP_ORDER(false, true);
    else SP_ORDER(false, false);
    launch_scans(L, n_pairs, hist, tot, tile_count, tile_offset, 1, s, live, cfg.chunk);
    SP_ORDER(true, false);
#undef SP_ORDER
    return hipGetLastError();
}

}  // namespace sp
