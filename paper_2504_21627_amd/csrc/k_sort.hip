// Coherence order of a ray batch: the rays sorted by a coarse key --
// direction octant, then the Morton code of the cell (2^b per axis, b <= 6
// chosen per object) of the voxel grid where the ray's segment [ta, tb]
// starts; at b = 7 (128^3 cells) the cell alone, without the octant.  Rays
// that meet the grid close together and head the same way then share waves,
// so their walks and their hash-grid gathers touch the same cache lines.
//
// The sort is a least-significant-digit radix sort with 8-bit digits (three
// passes for the largest keys).  Each pass counts the digit per block of
// kRadixTile consecutive rays of its input (the first pass while forming the
// keys) in LDS, scans the counters digit-major, which gives every (digit,
// block) its output range, then ranks each block's rays stably (a wave
// matches equal digits with one ballot per digit bit and keeps running counts
// per digit in LDS) and writes them there.  No global atomics: a counting
// sort's histogram and scatter take one device-wide atomic per ray, and those
// atomics, not the bytes moved, set its pace.
// Every ray's result is independent of the order the rays are processed in.
#include "lsnif_group.hpp"

namespace lsnif {

// Bits 0..6 of x spread to bits 0, 3, 6, ..., 18 (one axis of a 3-D Morton code).
__device__ __forceinline__ uint32_t spread7(uint32_t x)
{
    x &= 127u;
    x = (x | (x << 8)) & 0x0000f00fu;
    x = (x | (x << 4)) & 0x000c30c3u;
    x = (x | (x << 2)) & 0x00249249u;
    return x;
}


__device__ __forceinline__ uint32_t coherence_key(const Geom &g, float4 r0, float4 r1)
{
    VRay w;
    setup_ray(g, r0, r1, w);
    if (!w.cand) return sort_bins(g.sort_bits) - 1;
    uint32_t cell[3];
    const float cells = (float)(1u << g.sort_bits);
    const float sc = cells / (float)g.V;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float x = (w.o[a] + w.ta * w.d[a]) * sc;
        x = x < 0.0f ? 0.0f : (x > cells - 1.0f ? cells - 1.0f : x);
        cell[a] = (uint32_t)x;
    }
    const uint32_t morton = spread7(cell[0]) | (spread7(cell[1]) << 1) | (spread7(cell[2]) << 2);
    if (g.sort_bits >= 7u) return morton;
    const uint32_t oct = (w.d[0] < 0.0f ? 1u : 0u) | (w.d[1] < 0.0f ? 2u : 0u) | (w.d[2] < 0.0f ? 4u : 0u);
    return (oct << (3u * g.sort_bits)) | morton;
}

__global__ __launch_bounds__(kBlock) void k_fill(uint32_t *p, uint32_t n, uint32_t v)
{
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

constexpr uint32_t kRadixMaxPasses = 3;                 // coherence keys of at most 24 bits

// Block b: the coherence keys of rays [kRadixTile b, kRadixTile (b + 1)), and the
// count of each value of their lowest digit, to hist[digit nblk + b].
__global__ __launch_bounds__(kBlock) void k_radix_keys(Geom g, const float4 *rays, uint32_t n, uint32_t *keys,
                                                       uint32_t *hist, uint32_t nblk)
{
    __shared__ uint32_t cnt[256];
    const uint32_t t = threadIdx.x, b = blockIdx.x;
    cnt[t] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kRadixPer; ++j) {
        const uint32_t i = b * kRadixTile + j * kBlock + t;
        if (i < n) {
            const uint32_t k = coherence_key(g, rays[2 * i], rays[2 * i + 1]);
            keys[i] = k;
            atomicAdd(&cnt[k & 255u], 1u);
        }
    }
    __syncthreads();
    hist[(size_t)t * nblk + b] = cnt[t];
}

// The same with the keys' lowest kGroupBits bits as the digit and the counts block-major, a
// thread per digit (more threads than items of a thread: the keys' chain is what takes time).
__global__ __launch_bounds__(kGroupDigits) void k_group_keys(Geom g, const float4 *rays, uint32_t n, uint32_t *keys,
                                                       uint32_t *hist)
{
    __shared__ uint32_t cnt[kGroupDigits];
    const uint32_t t = threadIdx.x, b = blockIdx.x;
    cnt[t] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kRadixTile / kGroupDigits; ++j) {
        const uint32_t i = b * kRadixTile + j * kGroupDigits + t;
        if (i < n) {
            const uint32_t k = coherence_key(g, rays[2 * i], rays[2 * i + 1]);
            keys[i] = k;
            atomicAdd(&cnt[k & (kGroupDigits - 1u)], 1u);
        }
    }
    __syncthreads();
    hist[(size_t)b * kGroupDigits + t] = cnt[t];
}

__global__ __launch_bounds__(kBlock) void k_digit_count(const uint32_t *sk, uint32_t n, uint32_t *hist, uint32_t shift,
                                                        uint32_t digits)
{
    __shared__ uint32_t cnt[kGroupDigits];
    const uint32_t t = threadIdx.x, b = blockIdx.x;
    for (uint32_t d = t; d < group_row(digits); d += kBlock) cnt[d] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kRadixPer; ++j) {
        const uint32_t i = b * kRadixTile + j * kBlock + t;
        if (i < n) atomicAdd(&cnt[sk[i] >> shift], 1u);
    }
    __syncthreads();
    for (uint32_t d = t; d < group_row(digits); d += kBlock) hist[(size_t)b * group_row(digits) + d] = cnt[d];
}

// One grouping pass (group_pass): (sk, sv) to (dk, dv); NULLs as k_radix_scatter.
__global__ __launch_bounds__(kBlock) void k_group_scatter(const uint32_t *sk, const uint32_t *sv, uint32_t *dk,
                                                          uint32_t *dv, uint32_t n, const uint32_t *hist,
                                                          uint32_t digits, uint32_t shift)
{
    __shared__ GroupShared S;
    uint32_t key[kRadixPer], pos[kRadixPer];
    group_pass<kRadixPer>(sk, n, hist, digits, shift, S, key, pos);
    const uint32_t w = threadIdx.x >> 6;
#pragma unroll
    for (uint32_t j = 0; j < kRadixPer; ++j) {
        const uint32_t i = group_item<kRadixPer>(j);
        const uint32_t dst = S.run[w][(key[j] >> shift) & (kGroupDigits - 1u)] + pos[j];
        if (i < n && dst < n) {
            if (dk) dk[dst] = key[j];
            dv[dst] = sv ? sv[i] : i;
        }
    }
}

hipError_t launch_digit_count(const uint32_t *sk, uint32_t n, uint32_t *hist, uint32_t shift, uint32_t digits,
                              hipStream_t s)
{
    hipLaunchKernelGGL(k_digit_count, dim3((n + kRadixTile - 1) / kRadixTile), dim3(kBlock), 0, s, sk, n, hist, shift,
                       digits);
    return hipGetLastError();
}

// Block b: the count of each value of the digit at `shift` among keys
// [kRadixTile b, kRadixTile (b + 1)), to hist[digit nblk + b].
__global__ __launch_bounds__(kBlock) void k_radix_count(const uint32_t *sk, uint32_t n, uint32_t *hist,
                                                        uint32_t nblk, uint32_t shift)
{
    __shared__ uint32_t cnt[256];
    const uint32_t t = threadIdx.x, b = blockIdx.x;
    cnt[t] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kRadixPer; ++j) {
        const uint32_t i = b * kRadixTile + j * kBlock + t;
        if (i < n) atomicAdd(&cnt[(sk[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(size_t)t * nblk + b] = cnt[t];
}

// One pass: block b moves rays [kRadixTile b, kRadixTile (b + 1)) of (sk, sv) to
// their places in (dk, dv) by the digit at `shift`, keeping their order within a
// digit.  off: the exclusive scan of this pass's counters (digit-major), less
// `base`.  sv NULL: the indices are the positions;
// dk NULL: the keys are not needed after this pass.  Wave w takes rays
// 512 w .. 512 w + 511 of the block, 64 at a time, so (wave, step, lane) is
// the rays' order.
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const uint32_t *sk, const uint32_t *sv, uint32_t *dk,
                                                          uint32_t *dv, uint32_t n, const uint32_t *off,
                                                          uint32_t nblk, uint32_t shift, uint32_t base)
{
    __shared__ uint32_t run[kBlock / 64][256];   // per wave: rays of each digit so far, then the wave's start
    const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6, b = blockIdx.x;
    for (uint32_t i = t; i < (kBlock / 64) * 256u; i += kBlock) (&run[0][0])[i] = 0u;
    __syncthreads();
    uint32_t key[kRadixPer], pos[kRadixPer];
    rank_digits<kRadixPer, 256>(sk, n, shift, 255u, 8u, run, key, pos);
    __syncthreads();
    {   // thread t = digit t: the start of each wave's rays of that digit
        uint32_t at = off[(size_t)t * nblk + b] - base;
#pragma unroll
        for (uint32_t q = 0; q < kBlock / 64; ++q) {
            const uint32_t c = run[q][t];
            run[q][t] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t j = 0; j < kRadixPer; ++j) {
        const uint32_t i = b * kRadixTile + w * (kRadixTile / 4u) + j * 64u + lane;
        const uint32_t dst = run[w][(key[j] >> shift) & 255u] + pos[j];
        if (i < n && dst < n) {
            if (dk) dk[dst] = key[j];
            dv[dst] = sv ? sv[i] : i;
        }
    }
}

// Exclusive scan of n counters in two passes: block b first sums counters
// [1024 b, 1024 b + 1024), then rescans them with the sum of the blocks before
// it as the carry-in.
constexpr uint32_t kScanChunk = 1024;

__global__ __launch_bounds__(kBlock) void k_scan_partial(const uint32_t *hist, uint32_t nbins, uint32_t *part)
{
    __shared__ uint32_t tmp[kBlock];
    const uint32_t b0 = blockIdx.x * kScanChunk;
    uint32_t v = 0;
#pragma unroll
    for (uint32_t q = 0; q < kScanChunk / kBlock; ++q) {
        const uint32_t i = b0 + q * kBlock + threadIdx.x;
        if (i < nbins) v += hist[i];
    }
    uint32_t total;
    (void)block_exclusive_scan(v, tmp, total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(kBlock) void k_scan_final(uint32_t *hist, uint32_t nbins, const uint32_t *part)
{
    __shared__ uint32_t tmp[kBlock];
    const uint32_t t = threadIdx.x;
    // carry-in: sum of the partial sums of the blocks before this one
    uint32_t c = 0;
    for (uint32_t j = t; j < blockIdx.x; j += kBlock) c += part[j];
    uint32_t carry;
    (void)block_exclusive_scan(c, tmp, carry);
    // each thread scans 4 consecutive counters
    const uint32_t i0 = blockIdx.x * kScanChunk + 4 * t;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[q] = i0 + q < nbins ? hist[i0 + q] : 0u;
        sum += v[q];
    }
    uint32_t total;
    uint32_t run = carry + block_exclusive_scan(sum, tmp, total);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (i0 + q < nbins) hist[i0 + q] = run;
        run += v[q];
    }
}

hipError_t launch_exclusive_scan(uint32_t *v, uint32_t n, uint32_t *part, hipStream_t s, bool summed)
{
    const uint32_t nblocks = (n + kScanChunk - 1) / kScanChunk;
    if (!nblocks) return hipSuccess;
    if (!summed) hipLaunchKernelGGL(k_scan_partial, dim3(nblocks), dim3(kBlock), 0, s, v, n, part);
    hipLaunchKernelGGL(k_scan_final, dim3(nblocks), dim3(kBlock), 0, s, v, n, part);
    return hipGetLastError();
}

hipError_t launch_radix_pass(const uint32_t *sk, const uint32_t *sv, uint32_t *dk, uint32_t *dv, uint32_t n,
                             uint32_t *hist, uint32_t shift, bool counted, hipStream_t s)
{
    static_assert(kRadixTile == 4u * 512u && kBlock == 256u, "a block of the passes is 4 waves of 8 x 64 items");
    const uint32_t nblk = (n + kRadixTile - 1) / kRadixTile, counters = 256u * nblk;
    if (!nblk) return hipSuccess;
    if (!counted) hipLaunchKernelGGL(k_radix_count, dim3(nblk), dim3(kBlock), 0, s, sk, n, hist, nblk, shift);
    const hipError_t e = launch_exclusive_scan(hist, counters, hist + counters, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_radix_scatter, dim3(nblk), dim3(kBlock), 0, s, sk, sv, dk, dv, n, hist, nblk, shift, 0u);
    return hipGetLastError();
}

hipError_t launch_group_scatter(const uint32_t *sk, const uint32_t *sv, uint32_t *dk, uint32_t *dv, uint32_t n,
                                const uint32_t *hist, uint32_t digits, uint32_t shift, hipStream_t s)
{
    hipLaunchKernelGGL(k_group_scatter, dim3((n + kRadixTile - 1) / kRadixTile), dim3(kBlock), 0, s, sk, sv, dk, dv, n,
                       hist, digits, shift);
    return hipGetLastError();
}

hipError_t launch_coherence_sort(const Geom &g, const float4 *rays, uint32_t n, uint32_t *ws, uint32_t **order,
                                 hipStream_t s)
{
    const uint32_t passes = radix_passes(g.sort_bits), nblk = (n + kRadixTile - 1) / kRadixTile;
    if (passes > kRadixMaxPasses) return hipErrorInvalidValue;
    uint32_t *k0 = ws, *v0 = k0 + n, *k1 = v0 + n, *v1 = k1 + n, *hist = v1 + n;
    // Two passes of 10-bit digits: 4 launches where three passes of 8 bits take 12 (40,000 rays
    // 62 -> 36 us, 262,144 69 -> 49).  The first pass's counters lie in v0 (group_counts_at) and the
    // second's in k0, both free then (at most n / 2 + 1,024 words each).
    const uint32_t top = sort_bins(g.sort_bits) - 1u;
    if (n >= 2u * kRadixTile && n <= kGroupMax && top < kGroupDigits * kGroupDigits) {
        uint32_t *c0 = ws + group_counts_at(n);
        hipLaunchKernelGGL(k_group_keys, dim3(nblk), dim3(kGroupDigits), 0, s, g, rays, n, k0, c0);
        hipLaunchKernelGGL(k_group_scatter, dim3(nblk), dim3(kBlock), 0, s, k0, nullptr, k1, v1, n, c0, kGroupDigits, 0u);
        const uint32_t digits = (top >> kGroupBits) + 1u;
        const hipError_t e = launch_digit_count(k1, n, k0, kGroupBits, digits, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_group_scatter, dim3(nblk), dim3(kBlock), 0, s, k1, v1, nullptr, v0, n, k0, digits,
                           kGroupBits);
        *order = v0;
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_radix_keys, dim3(nblk), dim3(kBlock), 0, s, g, rays, n, k0, hist, nblk);
    const uint32_t *sk = k0, *sv = nullptr;
    for (uint32_t p = 0; p < passes; ++p) {
        uint32_t *dk = (p & 1u) ? k0 : k1, *dv = (p & 1u) ? v0 : v1;
        const hipError_t e = launch_radix_pass(sk, sv, p + 1 < passes ? dk : nullptr, dv, n, hist, 8u * p, p == 0, s);
        if (e != hipSuccess) return e;
        sk = dk;
        sv = dv;
    }
    *order = const_cast<uint32_t *>(sv);
    return hipGetLastError();
}

}  // namespace lsnif
