// The voxel-walk kernels.
#include "lsnif_kernels.hpp"
#include "lsnif_launch.hpp"

namespace lsnif {

// The walk with G lanes per ray (find_voxels), then the first H / 2 voxels found, in
// order of their place.  A wave's serial walk is one dependent chain of up to 3V
// divergent steps, 0.3 us and more each while few waves share a SIMD, however few
// the rays; here the chain is a few rounds of crossings.  Walks measured (us, one
// lane per ray, then this): 4,096 rays at V = 32 40 and 16, 32,000 at V = 128 66
// and 48, 2,500 pairs at V up to 256 105 and 23.
constexpr uint32_t kFoundRoom = 63;   // voxels of a ray kept; with more, one lane walks it

// Orders the LDS accesses of a wave's lanes (a ray's lanes are in one wave).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <bool PAIRS, bool RECHECK, int G, bool CELLS>
__global__ __launch_bounds__(kBlock) void k_walk_wide(QueryArgs A)
{
    constexpr uint32_t per = kBlock / G;   // rays of the block
    __shared__ uint32_t s_found[per][kFoundRoom + 2];   // per ray: their number, then the entries
    const uint32_t tid = threadIdx.x, lane = tid % G, ray = tid / G;
    const uint32_t slot = A.tile0 * kBlock + blockIdx.x * per + ray;
    uint32_t *count = &s_found[ray][0], *found = &s_found[ray][1];
    const auto walk = [&](const Geom &g) {
        const uint32_t cap = (uint32_t)g.H >> 1;
        uint32_t r, pair;
        bool live;
        VRay w;
        slot_ray<PAIRS>(A, g, slot, r, pair, live, w);
        const bool cand = live && w.cand;
        if (lane == 0) *count = 0u;
        wave_sync();
        WalkStart S;
        if (cand) find_voxels<RECHECK, G, CELLS>(g, w, (int)lane, g.coarse, count, found, kFoundRoom, S);
        wave_sync();
        uint32_t n = *count;
        if (cand && n > kFoundRoom) {   // the first voxels may be among those dropped
            if (lane == 0) n = (uint32_t)walk_cells<RECHECK>(g, w, S, A.lists + slot, A.n, (int)cap);
        } else if (cand) {
            for (uint32_t e = lane; e < n; e += G) {
                const uint32_t v = found[e];
                uint32_t at = 0;
                for (uint32_t q = 0; q < n; ++q) at += found[q] < v ? 1u : 0u;
                if (at >= cap) continue;
                const int k0 = (int)((v >> 10) & 1023u), k1 = (int)(v & 1023u), k2 = (int)(v >> 20) - k0 - k1;
                const int c[3] = {S.c0[0] + (S.up[0] ? k0 : -k0), S.c0[1] + (S.up[1] ? k1 : -k1),
                                  S.c0[2] + (S.up[2] ? k2 : -k2)};
                A.lists[(size_t)at * A.n + slot] = pack_ijk(c);
            }
        }
        if (lane == 0 && slot < A.n) A.nvox[slot] = (uint8_t)(n < cap ? n : cap);
    };
    if constexpr (PAIRS) {
        const int o = tile_object(A.pr, A.tile0 + blockIdx.x * per / kBlock);
        if (o < 0) return;   // the whole block; the query kernel skips such a tile too
        walk(((const cObjDev *)A.pr.objs)[o].g);
    } else {
        walk(A.g);
    }
}

// By the launch's slots n and its largest grid V.  64 lanes per ray and a plane per lane up to 8,192 slots (4,096 rays:
// 16 us at V = 32, 19 at 128; 8 lanes and bricks: 24 and 42; 16,000 rays at V = 128: 48 and
// 40), then a brick boundary per lane: 16 lanes up to 32,768 where V is 128 or more (16,000 rays at
// V = 128 40 and, 16 lanes, 32, at V = 32 24 and 29; 40,000 at 128 42 and 47; 16,000 pairs at V up
// to 256 58 and 40), 8 up to 57,344, one lane beyond: its chain (40 us at
// V = 32, 66 at 128, 105 at 256) takes as long for few rays as for a chip full (us, 8 lanes and
// one: V = 32, 40,000 slots 36 and 38, 80,000 59 and 41; V = 128, 64,000 62 and 66, 128,000 93 and
// 68; pairs at V up to 256, 24,000 78 and 103, 154,000 170 and 112).
template <bool PAIRS, bool RECHECK>
static void go(const QueryArgs &A, uint32_t max_V, uint32_t grid, hipStream_t s)
{
    const uint32_t n = grid * kBlock;
    if (n <= 8192u)
        hipLaunchKernelGGL((k_walk_wide<PAIRS, RECHECK, 64, true>), dim3(grid * 64u), dim3(kBlock), 0, s, A);
    else if (n <= 32768u && max_V >= 128u)
        hipLaunchKernelGGL((k_walk_wide<PAIRS, RECHECK, 16, false>), dim3(grid * 16u), dim3(kBlock), 0, s, A);
    else if (n <= 57344u)
        hipLaunchKernelGGL((k_walk_wide<PAIRS, RECHECK, 8, false>), dim3(grid * 8u), dim3(kBlock), 0, s, A);
    else
        hipLaunchKernelGGL((k_walk<PAIRS, RECHECK>), dim3(grid), dim3(kBlock), 0, s, A);
}

hipError_t launch_walk(const QueryArgs &A, bool pairs, bool recheck, uint32_t max_V, uint32_t grid, hipStream_t s)
{
    if (pairs) {
        if (recheck) go<true, true>(A, max_V, grid, s);
        else go<true, false>(A, max_V, grid, s);
    } else {
        if (recheck) go<false, true>(A, max_V, grid, s);
        else go<false, false>(A, max_V, grid, s);
    }
    return hipGetLastError();
}

}  // namespace lsnif
