// Histogram adjustment of the stored images (Section 2, after Remark 2: the
// output may be remapped so that its intensities follow a histogram the user
// chooses), gfx950.
//
// Histogram specification of every stored image (each frame of each pair, its
// integer codes) to one target histogram t[0 .. B - 1], B = 2^bits: with the
// image's cumulative counts S(k) (N pixels) and the target's T(m) (total
// T_tot), code k becomes the smallest m with T(m) N >= S(k) T_tot.  Everything
// is integer arithmetic (T_tot < 2^32 and N < 2^31, so both products fit in 64
// bits), so the result is exact and independent of the launch shape.  bits is
// at most 14: a workgroup holds one image's histogram (64 KB) and both
// cumulative tables (128 KB) in LDS.
//
//   hist_clear : zero the per-image histograms
//   hist_count : per (image, pixel chunk) LDS histogram, flushed with one
//                global atomic per non-empty bin
//   hist_lut   : per image, the prefix sums of its histogram and of the target
//                in LDS and a binary search per code -> look-up table
//   hist_apply : every pixel through its image's table, held in LDS
// The pixel passes are bound by memory: eight codes per load and store, and the
// dark pixels of a wave counted by one vote.  128 images of 512^2 at 12 bits
// (67 MB): count 51 -> 18 us, table 36 -> 13 (1024 threads, DPP scans in place of
// 16 serial additions per thread), apply 32 -> 24 (5.7 TB/s), 127 -> 64 us in all.
#include <hip/hip_runtime.h>

#include "launch.hpp"

namespace sp {
namespace {

// Pixels per applying workgroup.
constexpr int APPLY_CHUNK = 256 * 128;
constexpr int COUNT_THREADS = 1024, LUT_THREADS = 1024;

// Pixels per counting workgroup.  It clears and flushes a histogram of its own, so it takes
// many, but no more than leave every CU one: codes that repeat add to one LDS word, one
// after another, for as long as its workgroup has them.  Images of one code / of all codes
// alike, 12 bits, the whole call in us with 8 / 16 / 32 / 64 k: one pair of 256^2 31 / 37 /
// 49 / 74 and 26 / 27 / 29 / 33, of 1024^2 34 / 39 / 50 / 75 and 32 / 30 / 30 / 35, 16 of
// 512^2 53 / 55 / 54 / 79 and 42 / 37 / 35 / 39, one of 4096^2 137 / 114 / 102 / 95 and 123
// / 84 / 65 / 61.
constexpr int COUNT_CHUNK_MIN = 8192, COUNT_CHUNK_MAX = 65536;
int count_chunk(int64_t max_pixels, int64_t nimg)
{
    int chunk = COUNT_CHUNK_MAX;
    while (chunk > COUNT_CHUNK_MIN && nimg * ((max_pixels + chunk - 1) / chunk) < device_cu_count()) chunk /= 2;
    return chunk;
}

__device__ __forceinline__ void image_of(const synthpix_pair* __restrict__ pairs, int img, int64_t& off, int64_t& n)
{
    const synthpix_pair P = pairs[img >> 1];
    n = (int64_t)P.H * P.W;
    off = P.image_offset + (img & 1) * n;
}

__global__ void __launch_bounds__(256) hist_clear(uint32_t* __restrict__ h, int64_t n, uint32_t* __restrict__ status)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) status[0] = 0u;
    if (i < n) h[i] = 0u;
}

// Runs f(pixel, code) on the codes [c0, c1) of one image and stores its results
// where WRITE, eight codes (16 bytes) per thread and step between an unaligned
// head and tail.
template <int THREADS, bool WRITE, typename F>
__device__ __forceinline__ void each_code(uint16_t* __restrict__ im, int64_t c0, int64_t c1, F f)
{
    const int t = (int)threadIdx.x;
    const int64_t head = min(c1 - c0, (int64_t)((8 - (((uintptr_t)(im + c0) >> 1) & 7)) & 7));
    const int64_t v0 = c0 + head, nv = (c1 - v0) >> 3, v1 = v0 + 8 * nv;
    const int64_t edge = head + (c1 - v1);                  // fewer than 16 codes
    if (t < edge) {
        const int64_t i = t < head ? c0 + t : v1 + (t - head);
        const uint32_t m = f((uint32_t)im[i], true);
        if (WRITE) im[i] = (uint16_t)m;
    }
    uint4* v = reinterpret_cast<uint4*>(im + v0);
    // whole waves run the body together (f may vote): the last step masks lanes
    for (int64_t k = t; k < ((nv + 63) & ~(int64_t)63); k += THREADS) {
        const bool on = k < nv;
        const uint4 q = on ? v[k] : make_uint4(0u, 0u, 0u, 0u);
        uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = f(w[e] & 0xffffu, on), hi = f(w[e] >> 16, on);
            if (WRITE) w[e] = lo | (hi << 16);
        }
        if (WRITE && on) v[k] = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// A wave's zeros, the commonest code of a dark image, are counted by a vote: one
// addition for all of them instead of as many on one LDS word.
__global__ void __launch_bounds__(COUNT_THREADS)
hist_count(const synthpix_pair* __restrict__ pairs, uint16_t* __restrict__ images, int B,
           int chunk, uint32_t* __restrict__ hist, uint32_t* __restrict__ status)
{
    extern __shared__ uint32_t lh[];
    const int img = blockIdx.y;
    int64_t off, n;
    image_of(pairs, img, off, n);
    const int64_t c0 = (int64_t)blockIdx.x * chunk;
    if (c0 >= n) return;
    for (int b = threadIdx.x; b < B; b += COUNT_THREADS) lh[b] = 0u;
    __syncthreads();
    bool wide = false;
    uint32_t zeros = 0u;                                     // the wave's, in every lane
    each_code<COUNT_THREADS, false>(images + off, c0, min(c0 + chunk, n), [&](uint32_t c, bool on) {
        zeros += (uint32_t)__popcll(__ballot(on && c == 0u));
        if (on && c != 0u) {
            wide = wide || c >= (uint32_t)B;
            atomicAdd(&lh[min(c, (uint32_t)B - 1u)], 1u);
        }
        return c;
    });
    if (zeros && (threadIdx.x & 63) == 0) atomicAdd(&lh[0], zeros);
    if (wide) atomicOr(status, SP_STATUS_HIST_CODE);
    __syncthreads();
    uint32_t* g = hist + (int64_t)img * B;
    for (int b = threadIdx.x; b < B; b += COUNT_THREADS)
        if (lh[b]) atomicAdd(&g[b], lh[b]);
}

// In-place inclusive scan of s[0 .. B) over the LUT_THREADS threads.
__device__ void block_scan(uint32_t* s, int B, uint32_t* part)
{
    const int t = (int)threadIdx.x, wid = t >> 6;
    uint32_t carry = 0;
    for (int b = 0; b < B; b += LUT_THREADS) {
        const int k = b + t;
        const uint32_t inc = wave_scan(k < B ? s[k] : 0u);
        if ((t & 63) == 63) part[wid] = inc;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (int w = 0; w < LUT_THREADS / 64; ++w) {
            const uint32_t sw = part[w];
            if (w < wid) before += sw;
            carry += sw;
        }
        if (k < B) s[k] = before + inc;
        __syncthreads();
    }
}

// One workgroup per image.  The target's total is summed in 64 bits first; with
// it below 2^32 every cumulative count fits 32 bits (the image's: N < 2^31).
__global__ void __launch_bounds__(LUT_THREADS)
hist_lut(const synthpix_pair* __restrict__ pairs, const uint32_t* __restrict__ target, int B,
         const uint32_t* __restrict__ hist, uint16_t* __restrict__ lut, uint32_t* __restrict__ status)
{
    extern __shared__ uint32_t ls[];
    uint32_t* S = ls;           // [B] image cumulative counts
    uint32_t* T = ls + B;       // [B] target cumulative counts
    __shared__ uint32_t part[LUT_THREADS / 64];
    __shared__ unsigned long long s_tot;
    const int img = blockIdx.x;
    int64_t off, n;
    image_of(pairs, img, off, n);
    unsigned long long tsum = 0;
    const uint32_t* h = hist + (int64_t)img * B;
    for (int b = threadIdx.x; b < B; b += LUT_THREADS) {
        S[b] = h[b];
        T[b] = target[b];
        tsum += T[b];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) tsum += __shfl_xor(tsum, o, 64);
    if (threadIdx.x == 0) s_tot = 0ull;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicAdd(&s_tot, tsum);
    __syncthreads();
    const unsigned long long Tt = s_tot;
    uint16_t* out = lut + (int64_t)img * B;
    if (Tt == 0ull || Tt >= (1ull << 32)) {
        // no usable target: the images stay as they are
        if (threadIdx.x == 0) atomicOr(status, SP_STATUS_HIST_TARGET);
        for (int b = threadIdx.x; b < B; b += LUT_THREADS) out[b] = (uint16_t)b;
        return;
    }
    block_scan(S, B, part);
    block_scan(T, B, part);
    const unsigned long long N = (unsigned long long)n;
    for (int k = threadIdx.x; k < B; k += LUT_THREADS) {
        const unsigned long long need = (unsigned long long)S[k] * Tt;     // < 2^31 * 2^32
        int lo = 0, hi = B - 1;                                             // T[B - 1] N >= S[k] Tt holds
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((unsigned long long)T[mid] * N >= need) hi = mid; else lo = mid + 1;
        }
        out[k] = (uint16_t)lo;
    }
}

__global__ void __launch_bounds__(256)
hist_apply(const synthpix_pair* __restrict__ pairs, uint16_t* __restrict__ images, int B,
           const uint16_t* __restrict__ lut)
{
    extern __shared__ uint32_t ls[];
    uint16_t* L = reinterpret_cast<uint16_t*>(ls);
    const int img = blockIdx.y;
    int64_t off, n;
    image_of(pairs, img, off, n);
    const int64_t c0 = (int64_t)blockIdx.x * APPLY_CHUNK;
    if (c0 >= n) return;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(lut + (int64_t)img * B);     // B is even
    for (int k = threadIdx.x; k < B / 2; k += 256) ls[k] = src[k];
    __syncthreads();
    each_code<256, true>(images + off, c0, min(c0 + APPLY_CHUNK, n),
                         [&](uint32_t c, bool) { return (uint32_t)L[min(c, (uint32_t)B - 1u)]; });
}

}  // namespace

size_t hist_workspace_bytes(int n_pairs, int bits)
{
    const size_t B = (size_t)1 << bits, nimg = 2 * (size_t)n_pairs;
    return 256 + ((nimg * B * 4 + 255) & ~(size_t)255) + ((nimg * B * 2 + 255) & ~(size_t)255);
}

hipError_t launch_histogram_match(const synthpix_pair* pairs_dev, int n_pairs, int64_t max_pixels, int bits,
                                  const uint32_t* target, uint16_t* images, char* ws, hipStream_t s)
{
    const int B = 1 << bits;
    const int nimg = 2 * n_pairs;
    uint32_t* status = reinterpret_cast<uint32_t*>(ws);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + 256);
    uint16_t* lut = reinterpret_cast<uint16_t*>(ws + 256 + (((size_t)nimg * B * 4 + 255) & ~(size_t)255));
    const int64_t nh = (int64_t)nimg * B;
    const int chunk = count_chunk(max_pixels, nimg);
    const dim3 count_grid((unsigned)((max_pixels + chunk - 1) / chunk), (unsigned)nimg);
    const dim3 apply_grid((unsigned)((max_pixels + APPLY_CHUNK - 1) / APPLY_CHUNK), (unsigned)nimg);
    TimedScope ts("histogram_match", s);
    hipLaunchKernelGGL(hist_clear, dim3((unsigned)((nh + 255) / 256)), dim3(256), 0, s, hist, nh, status);
    hipLaunchKernelGGL(hist_count, count_grid, dim3(COUNT_THREADS), (size_t)B * 4, s, pairs_dev, images, B, chunk, hist,
                       status);
    hipLaunchKernelGGL(hist_lut, dim3((unsigned)nimg), dim3(LUT_THREADS), (size_t)B * 8, s, pairs_dev, target, B, hist,
                       lut, status);
    hipLaunchKernelGGL(hist_apply, apply_grid, dim3(256), (size_t)B * 2, s, pairs_dev, images, B, lut);
    return hipGetLastError();
}

}  // namespace sp
