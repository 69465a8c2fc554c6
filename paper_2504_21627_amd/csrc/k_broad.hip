// Broad phase of instanced queries: which instances each ray may hit.
//
// Pair (r, i) exists when ray r, mapped into instance i's object space, meets
// the object's voxel grid on [max(ta, tmin), tb] with positive length and
// that segment starts no later than tmax: the same mapping and slab test the
// pair query's narrow phase starts with (to_object_space, setup_ray), and a
// hit's t lies in [ta, tb] and must not exceed tmax, so no pair that can hit
// is left out.
// The instance and its object's constants are wave-uniform, read through the scalar path.
// With at most 256 instances a thread tests a ray against 8 of them and leaves a byte of
// bits, so that a few rays against many instances are as many threads as tests / 8 (2,500
// rays and 64 instances 11 us, 262,144 rays 36; one lane per ray testing all 64: 67 and 73); a counting pass,
// the scan of the counts and a writing pass then list the pairs by ray, then instance, from the
// bytes.  With more instances one lane per ray tests them all, once to count and once to write.
#include "lsnif_kernels.hpp"
#include "lsnif_launch.hpp"

namespace lsnif {

typedef const __attribute__((address_space(4))) lsnif_instance cinst;

__device__ __forceinline__ bool meets(const BroadArgs &B, uint32_t i, float4 a, float4 b)
{
    const uint32_t o = ((cinst *)B.inst)[i].object_id;
    if (o >= B.n_objs || !((const cObjDev *)B.objs)[o].live) return false;   // no such object: no pair
    const cObjDev &O = ((const cObjDev *)B.objs)[o];
    lsnif_instance I;
    I.object_id = o;
#pragma unroll
    for (int k = 0; k < 12; ++k) I.world_to_object[k] = ((cinst *)B.inst)[i].world_to_object[k];
    to_object_space(I, a, b);
    VRay w;
    setup_ray(O.g, a, b, w);
    return w.cand && w.ta <= w.tmax;
}

// Block (x, y): rays 256 x .. against instances 8 y ..
__global__ __launch_bounds__(kBlock) void k_broad_masks(BroadArgs B)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x, i0 = 8u * blockIdx.y;
    const bool live = r < B.n_rays;
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
    if (live) {
        a = B.rays[2 * r];
        b = B.rays[2 * r + 1];
    }
    uint32_t bits = 0;
    for (uint32_t q = 0; q < 8u && i0 + q < B.n_inst; ++q) bits |= meets(B, i0 + q, a, b) ? 1u << q : 0u;
    if (live) B.masks[(size_t)blockIdx.y * B.n_rays + r] = (uint8_t)bits;
}

// Block b: the pairs of rays 1024 b .., and their sum for the scan.
constexpr uint32_t kCountRays = 1024;   // the scan's chunk
__global__ __launch_bounds__(kCountRays) void k_broad_count(BroadArgs B)
{
    __shared__ uint32_t sum;
    if (threadIdx.x == 0) sum = 0u;
    __syncthreads();
    const uint32_t r = blockIdx.x * kCountRays + threadIdx.x;
    uint32_t n = 0;
    if (r < B.n_rays)
        for (uint32_t k = 0; 8u * k < B.n_inst; ++k) n += (uint32_t)__builtin_popcount(B.masks[(size_t)k * B.n_rays + r]);
    if (r <= B.n_rays) B.offsets[r] = n;   // 0 at n_rays: the scan leaves the total there
    if (n) atomicAdd(&sum, n);
    __syncthreads();
    if (threadIdx.x == 0) B.part[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kBlock) void k_broad_list(BroadArgs B)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= B.n_rays) return;
    uint32_t at = B.offsets[r];
    for (uint32_t k = 0; 8u * k < B.n_inst; ++k) {
        uint32_t m = B.masks[(size_t)k * B.n_rays + r];
        while (m) {
            B.pair_ray[at] = r;
            B.pair_inst[at] = 8u * k + (uint32_t)__builtin_ctz(m);
            ++at;
            m &= m - 1u;
        }
    }
}

// More instances than the masks hold.
template <bool WRITE>
__global__ __launch_bounds__(kBlock) void k_broad(BroadArgs B)
{
    const uint32_t r = blockIdx.x * kBlock + threadIdx.x;
    const bool live = r < B.n_rays;
    if (!WRITE && r == B.n_rays) B.offsets[r] = 0u;   // the exclusive scan leaves the total here
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
    if (live) {
        a = B.rays[2 * r];
        b = B.rays[2 * r + 1];
    }
    uint32_t n = 0, at = WRITE && live ? B.offsets[r] : 0u;
    for (uint32_t i = 0; i < B.n_inst; ++i) {
        if (!(live && meets(B, i, a, b))) continue;
        if constexpr (WRITE) {
            B.pair_ray[at] = r;
            B.pair_inst[at] = i;
            ++at;
        } else {
            ++n;
        }
    }
    if (!WRITE && live) B.offsets[r] = n;
}

hipError_t launch_broad_count(const BroadArgs &B, hipStream_t s)
{
    const uint32_t n1 = B.n_rays + 1u;
    if (!B.masks) {
        hipLaunchKernelGGL(k_broad<false>, dim3(B.n_rays / kBlock + 1), dim3(kBlock), 0, s, B);
        return launch_exclusive_scan(B.offsets, n1, B.part, s);
    }
    if (B.n_rays && B.n_inst)
        hipLaunchKernelGGL(k_broad_masks, dim3((B.n_rays + kBlock - 1) / kBlock, (B.n_inst + 7) / 8), dim3(kBlock), 0, s,
                           B);
    hipLaunchKernelGGL(k_broad_count, dim3((n1 + kCountRays - 1) / kCountRays), dim3(kCountRays), 0, s, B);
    return launch_exclusive_scan(B.offsets, n1, B.part, s, true);
}

hipError_t launch_broad_write(const BroadArgs &B, hipStream_t s)
{
    if (!B.n_rays) return hipSuccess;
    const dim3 grid((B.n_rays + kBlock - 1) / kBlock);
    if (B.masks) hipLaunchKernelGGL(k_broad_list, grid, dim3(kBlock), 0, s, B);
    else hipLaunchKernelGGL(k_broad<true>, grid, dim3(kBlock), 0, s, B);
    return hipGetLastError();
}

}  // namespace lsnif
