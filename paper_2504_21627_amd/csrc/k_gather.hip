// The gather-ceiling kernel: the query's gathers alone, for measurement.
#include "lsnif_query.hpp"

namespace lsnif {

// The query kernel without its MLP: the same tiles, packed points, batches of levels and LDS budget, but
// a point's interpolated features are summed, a float per point and batch, and a ray's points'
// sums go to sums[r].  Without the accumulators and the products the gathers run as fast
// as this split of them can (ms, the query kernel, this, and a ray per lane as it was: 2,097,152
// FP16 rays of 16 levels 1.64, 1.36, 1.51; 300,000 0.43, 0.39, 0.62; 1,048,576 of 2 levels with 3
// features 0.44, 0.26, 0.47).
template <typename TF, int F, int R>
__global__ __launch_bounds__(kBlock, 4) void k_gather_only(QueryArgs A, float *sums, uint32_t lds_bytes)
{
    constexpr int NL = PointT<_Float16, F>::NLB;
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    __shared__ QueryShared<R> S;
    const Geom &g = A.g;
    const TF *__restrict__ tab = reinterpret_cast<const TF *>(A.tables);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slot0 = block_subtile<R>(A.tile0) * R;
    uint32_t r = 0, pair, nv = 0;
    bool live = false;
    if (tid == 0) S.most[0] = 0u;
    __syncthreads();
    if (tid < (uint32_t)R) {
        VRay w;
        slot_ray<false>(A, g, slot0 + tid, r, pair, live, w);
        nv = live ? A.nvox[slot0 + tid] : 0u;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            S.ray[a][tid] = w.o[a];
            S.ray[3 + a][tid] = w.d[a];
            S.ray[6 + a][tid] = w.inv[a];
        }
        S.mov[tid] = (uint8_t)w.mov;
        S.nvox[tid] = (uint8_t)nv;
        atomicMax(&S.most[0], nv);
    }
    __syncthreads();
    const uint32_t most = __builtin_amdgcn_readfirstlane(S.most[0]), nbat = level_batches<_Float16, F>(g.L);
    const uint32_t vox = min(most, (lds_bytes - 64u) / (2u * R * (18u + 4u * nbat))), zero = 2u * R * vox;
    float4 *pts = reinterpret_cast<float4 *>(s_dyn);
    float *part = reinterpret_cast<float *>(pts + zero);
    uint16_t *smap = reinterpret_cast<uint16_t *>(part + zero * nbat);
    float total = 0.0f, here = 0.0f;
    for (uint32_t j0 = 0; j0 < most; j0 += vox) {
        const uint32_t nj = min(vox, most - j0);
        pack_points<R>(A, slot0, j0, nj, zero, S, pts, smap);
        const uint32_t npts = __builtin_amdgcn_readfirstlane(S.npts);
        const uint32_t tasks = (npts + 63u) / 64u * nbat;
        for (uint32_t t = wave; t < tasks; t += kBlock / 64) {
            const uint32_t grp = t / nbat, b = t - grp * nbat, s = grp * 64u + lane;
            if (s >= npts) continue;
            const float4 p4 = pts[s];
            const float p[3] = {p4.x, p4.y, p4.z};
            const int l0 = (int)b * NL;
            float v[NL][F], sum = 0.0f;
            bool aligned = false;
            if constexpr (F == 3) {
                const uint32_t all = ((1u << NL) - 1u) & ((uint32_t)(2u << (g.L - 1 - l0)) - 1u);
                aligned = (~(g.aligned_mask >> l0) & all) == 0u;
            }
            if (aligned) encode_aligned<TF, F, NL, false>(g, tab, l0, p, __float_as_int(p4.w), v);
            else encode_levels<TF, F, NL>(g, tab, l0, p, __float_as_int(p4.w), v);
#pragma unroll
            for (int lv = 0; lv < NL; ++lv)
#pragma unroll
                for (int f = 0; f < F; ++f) sum += v[lv][f];
            part[s * nbat + b] = sum;
        }
        __syncthreads();
        if (tid < (uint32_t)R)
            for (uint32_t hh = 0; hh < 2u * nj && 2u * j0 + hh < 2u * nv; ++hh) {
                const uint32_t s = smap[hh * R + tid];
                if (s != kSameSlot) {
                    here = 0.0f;
                    for (uint32_t b = 0; b < nbat; ++b) here += part[s * nbat + b];
                }
                total += here;
            }
        __syncthreads();
    }
    if (live) sums[r] = total;
}

template <typename TF, int F, int R> static void go(QueryArgs A, uint32_t nbat, float *sums, uint32_t grid, hipStream_t s)
{
    uint32_t vox = (uint32_t)A.g.H / 2u;
    auto need = [&]() { return 2u * R * vox * (18u + 4u * nbat) + 64u; };
    while (vox > 1u && need() > kQueryLds) --vox;
    for (uint32_t left = grid, most = tiles_per_launch(kBlock / R * kBlock); left;) {
        const uint32_t now = left < most ? left : most;
        hipLaunchKernelGGL((k_gather_only<TF, F, R>), dim3(now * (kBlock / R)), dim3(kBlock), need(), s, A, sums, need());
        A.tile0 += now;
        left -= now;
    }
}

template <typename TF, int F> static void rays(const QueryArgs &A, bool f32, float *sums, uint32_t grid, hipStream_t s)
{
    const uint32_t nbat = level_batches<_Float16, F>(A.g.L);
    const int R = rays_per_block(grid * kBlock, nbat, f32);
    if (R == 16) go<TF, F, 16>(A, nbat, sums, grid, s);
    else if (R == 32) go<TF, F, 32>(A, nbat, sums, grid, s);
    else go<TF, F, 64>(A, nbat, sums, grid, s);
}

hipError_t launch_gather_only(const QueryArgs &A, int feat_dtype, int F, bool f32, float *sums, uint32_t grid,
                              hipStream_t s)
{
    if (feat_dtype == LSNIF_FP32) {
        if (F == 2) rays<float, 2>(A, f32, sums, grid, s); else rays<float, 3>(A, f32, sums, grid, s);
    } else if (feat_dtype == LSNIF_FP16) {
        if (F == 2) rays<_Float16, 2>(A, f32, sums, grid, s); else rays<_Float16, 3>(A, f32, sums, grid, s);
    } else {
        if (F == 2) rays<__bf16, 2>(A, f32, sums, grid, s); else rays<__bf16, 3>(A, f32, sums, grid, s);
    }
    return hipGetLastError();
}

}  // namespace lsnif
