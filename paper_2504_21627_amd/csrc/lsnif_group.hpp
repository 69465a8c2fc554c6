// One stable grouping pass over at most kGroupMax items, shared by the coherence sort and
// the pair preparation.
#pragma once
#include "lsnif_kernels.hpp"
#include "lsnif_launch.hpp"

namespace lsnif {

constexpr uint32_t kRadixPer = kRadixTile / kBlock;   // items per thread in a block of the passes

// Exclusive scan of one value per thread of a block (Hillis-Steele in LDS).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *tmp, uint32_t &total)
{
    const uint32_t t = threadIdx.x;
    tmp[t] = v;
    __syncthreads();
    for (uint32_t off = 1; off < kBlock; off <<= 1) {
        const uint32_t u = t >= off ? tmp[t - off] : 0u;
        __syncthreads();
        tmp[t] += u;
        __syncthreads();
    }
    total = tmp[kBlock - 1];
    const uint32_t incl = tmp[t];
    __syncthreads();
    return incl - v;
}

// Item j of this thread: a block takes 256 PER items, wave w of it 64 PER of those in a row, 64
// at a time, so (wave, step, lane) is the items' order.
template <uint32_t PER> __device__ __forceinline__ uint32_t group_item(uint32_t j)
{
    return blockIdx.x * (kBlock * PER) + (threadIdx.x >> 6) * (64u * PER) + j * 64u + (threadIdx.x & 63u);
}

// Ranks of a block's items within their digits: item j of a thread is number pos[j] of its
// digit in its wave, and run[w][d] counts wave w's items of digit d.
// A wave matches equal digits with one ballot per digit bit.
template <uint32_t PER, uint32_t STRIDE>
__device__ __forceinline__ void rank_digits(const uint32_t *sk, uint32_t n, uint32_t shift, uint32_t mask, uint32_t bits,
                                            uint32_t (*run)[STRIDE], uint32_t key[PER], uint32_t pos[PER])
{
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    const uint64_t below = lane ? (~0ull >> (64u - lane)) : 0ull;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t i = group_item<PER>(j);
        key[j] = i < n ? sk[i] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t i = group_item<PER>(j);
        const bool live = i < n;
        const uint32_t d = (key[j] >> shift) & mask;
        uint64_t same = __ballot(live);
        for (uint32_t q = 0; q < bits; ++q) {
            const uint64_t ones = __ballot((d >> q) & 1u);
            same &= ((d >> q) & 1u) ? ones : ~ones;
        }
        const uint32_t before = run[w][d];
        pos[j] = before + (uint32_t)__builtin_popcountll(same & below);
        if (live && (same & below) == 0ull) run[w][d] = before + (uint32_t)__builtin_popcountll(same);
    }
}

// Words from one block's counters to the next's (rows of whole 16-byte words; the spare
// counters are 0).
__host__ __device__ inline uint32_t group_row(uint32_t digits) { return (digits + 3u) / 4u * 4u; }

// The LDS of a grouping pass.
struct GroupShared {
    uint32_t run[kBlock / 64][kGroupDigits];   // per wave: items of each digit, then the wave's start
    uint32_t first[kGroupDigits + 4];          // first position of each digit, and the end of the last
    uint32_t tmp[kBlock];
};

// Ranks the block's items by the digit at `shift` (below `digits`, at most kGroupDigits)
// and leaves every wave's start of every digit in S.run and the digits' first positions in
// S.first.  hist: the counts of all blocks, block-major; each block sums them itself, which
// for up to 128 blocks is cheaper than launches that scan them (4.5 us each).
template <uint32_t PER>
__device__ __forceinline__ void group_pass(const uint32_t *sk, uint32_t n, const uint32_t *hist, uint32_t digits,
                                           uint32_t shift, GroupShared &S, uint32_t key[PER], uint32_t pos[PER])
{
    const uint32_t t = threadIdx.x, b = blockIdx.x, nblk = (n + kBlock * PER - 1u) / (kBlock * PER);
    for (uint32_t i = t; i < (kBlock / 64) * kGroupDigits; i += kBlock) (&S.run[0][0])[i] = 0u;
    // thread t: digits 4 t .. 4 t + 3, their items in the blocks before this one and in all
    uint32_t before[4] = {}, all[4] = {};
    const uint32_t row = group_row(digits);
    if (4u * t < digits) {
        const uint4 *col = reinterpret_cast<const uint4 *>(hist + 4u * t);
        for (uint32_t c0 = 0; c0 < nblk; c0 += 16u) {
            uint4 v[16];
#pragma unroll
            for (uint32_t q = 0; q < 16u; ++q) v[q] = col[(size_t)min(c0 + q, nblk - 1u) * (row / 4u)];
#pragma unroll
            for (uint32_t q = 0; q < 16u; ++q) {
                const uint32_t in = c0 + q < nblk ? ~0u : 0u, bf = c0 + q < b ? ~0u : 0u;
                const uint32_t x[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    all[k] += x[k] & in;
                    before[k] += x[k] & bf;
                }
            }
        }
    }
    uint32_t total;
    uint32_t at = block_exclusive_scan((all[0] + all[1]) + (all[2] + all[3]), S.tmp, total);   // its barriers cover S.run
    rank_digits<PER, kGroupDigits>(sk, n, shift, kGroupDigits - 1u, 32u - (uint32_t)__builtin_clz(digits - 1u | 1u), S.run,
                              key, pos);
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t d = 4u * t + q;
        S.first[d] = at;
        uint32_t start = at + before[q];
#pragma unroll
        for (uint32_t w = 0; w < kBlock / 64; ++w) {
            const uint32_t c = S.run[w][d];
            S.run[w][d] = start;
            start += c;
        }
        at += all[q];
    }
    if (t == kBlock - 1u) S.first[kGroupDigits] = at;
    __syncthreads();
}

}  // namespace lsnif
