// Training: the order of a batch's rays, and one kernel for the encoding, the layers' forward
// and backward products, the losses and the encoding's gradient.
#include "lsnif_group.hpp"
#include "lsnif_train.hpp"

namespace lsnif {

// ------------------------------------------------------------------- ray order
// Block b: keys of rays [kRadixTile b, kRadixTile (b + 1)), `most` less the ray's voxels, and
// their counts: block-major in rows of `row` (row 0: digit-major over nblk blocks).
__global__ __launch_bounds__(1024) void k_train_keys(const uint8_t *nvox, uint32_t n, uint32_t most, uint32_t *keys,
                                                     uint32_t *hist, uint32_t row, uint32_t nblk, uint32_t *n_live)
{
    __shared__ uint32_t cnt[256];
    const uint32_t t = threadIdx.x, b = blockIdx.x;
    if (t < 256u) cnt[t] = 0u;
    __syncthreads();
    for (uint32_t j = 0; j < kRadixTile / 1024u; ++j) {
        const uint32_t i = b * kRadixTile + j * 1024u + t;
        if (i >= n) continue;
        const uint32_t k = most - nvox[i];
        keys[i] = k;
        atomicAdd(&cnt[k], 1u);
    }
    __syncthreads();
    if (t < 256u && (!row || t < row)) hist[row ? (size_t)b * row + t : (size_t)t * nblk + b] = cnt[t];
    if (t == 0) atomicAdd(n_live, min(kRadixTile, n - b * kRadixTile) - cnt[most]);
}

// Longest lists first: tiles of like lists, dealt to the blocks in turn, multiply little padding
// and end together.  Up to kGroupMax rays, two launches.
hipError_t launch_train_order(const uint8_t *nvox, uint32_t n, uint32_t most, uint32_t *ws, uint32_t **order,
                              uint32_t *n_live, hipStream_t s)
{
    const uint32_t nblk = (n + kRadixTile - 1) / kRadixTile, digits = most + 1u;
    const uint32_t row = n <= kGroupMax ? group_row(digits) : 0u;
    uint32_t *hist = ws, *keys = ws + (radix_hist_words(n) + 3u) / 4u * 4u, *out = keys + n;
    hipLaunchKernelGGL(k_train_keys, dim3(nblk), dim3(1024), 0, s, nvox, n, most, keys, hist, row, nblk, n_live);
    *order = out;
    return row ? launch_group_scatter(keys, nullptr, nullptr, out, n, hist, digits, 0u, s)
               : launch_radix_pass(keys, nullptr, nullptr, out, n, hist, 0u, true, s);
}

// ------------------------------------------------------------------ fused step
// W^T of each layer, units in rows of 32 j floats (layer 0) or the width: thread = entry.
__global__ __launch_bounds__(kBlock) void k_train_transpose(TrainStepArgs A, uint32_t in0, uint32_t width)
{
    const uint32_t k = blockIdx.y, in = k ? width : in0, ldT = k ? width : A.ldT0;
    const uint32_t ld = k == A.n_hidden ? (uint32_t)kMaxOut : width;
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x, c = i / ldT, u = i - c * ldT;
    if (c < ld) A.WT[A.offT[k] + i] = u < in ? A.W[A.off[k] + u * ld + c] : 0.0f;
}

// 32 x 32 products of a row-major weight matrix (lane's column at w, rows ld apart, lane half
// q starting at row q) and 32 rows in LDS (lane's row at `in`): acc += w[k] in[k] over its `rows`
// rows, ascending.  a: the first 8 weights, loaded before the barrier ahead of the product; the
// next 8 travel while 8 are multiplied.  TAIL: `rows` need not be a multiple of 16; the last
// ones are multiplied with weights of 0 after them (step_weight_row).
__device__ __forceinline__ void first_weights(const float *w, uint32_t ld, float a[8])
{
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) a[j] = w[2u * j * ld];
}

__device__ __forceinline__ void multiply8(f16_t &acc, const float a[8], const float *in, uint32_t q)
{
#pragma unroll
    for (uint32_t j = 0; j < 8; j += 2) {
        const float4 b = *reinterpret_cast<const float4 *>(in + 2u * j);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], q ? b.y : b.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j + 1], q ? b.w : b.z, acc, 0, 0, 0);
    }
}

template <bool TAIL>
__device__ __forceinline__ f16_t product(const float *w, uint32_t ld, const float *in, uint32_t rows, uint32_t q, float a[8])
{
    const uint32_t K = TAIL ? rows / 16u * 16u : rows;
    f16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    for (uint32_t c = 0; c < K; c += 16u) {
        float next[8];
        first_weights(w + (size_t)(c + 16u < K ? c + 16u : 0u) * ld, ld, next);
        multiply8(acc, a, in + c, q);
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) a[j] = next[j];
    }
    if (TAIL && K < rows) {
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t row = K + 2u * j + q;
            const float x = w[(int)(step_weight_row(row, rows) - q) * (int)ld];
            a[j] = row < rows ? x : 0.0f;
        }
        multiply8(acc, a, in + K, q);
    }
    return acc;
}

// One block takes tiles of 32 rows (rays), dealt in turn from the longest lists to the shortest.
// A tile's encoding, activations and gradients stay in LDS, row-major with strides of 4 modulo
// 32 floats; the weight gradients stay in the waves' accumulators (32 x 32 blocks, block id to
// wave id % 4) over all of the block's tiles.  All products are v_mfma_f32_32x32x2f32 (the
// head's forward one 16x16x4), the forward ones in ascending K, so the outputs are what
// layer-by-layer products give, bit for bit.  Of the encoding only the points of the tile's
// longest list are formed, multiplied and given gradients, and rays that list nothing are not
// in the order.  (A first-layer weight that is not finite therefore spoils the tiles that reach its
// point, not every gradient at once.)
//
// Separate launches moved every activation and gradient through HBM and multiplied the zeros:
// at 262,144 rays of the paper's default object (173,070 list voxels) 916 us of products, 57 of
// partial sums, 126 + 398 of encodings and 20 of losses, against 787 here, 17 and 20 for the
// order.  Of the 787 the matrix cores work 220; the table atomics, which
// overlap with other blocks' products, add 220 (at 505 + 433 as a launch of their own), and
// the rest is the waves' serial phases (rays, encoding, head, losses: 32 k of 110 k cycles a
// tile) at the two waves per SIMD that the accumulators leave room for.  Tiles in coherence order
// instead: 589 for 505, the blocks' padding and ends being less even.
template <int F, int WIDTH, int MAXB>
__global__ __launch_bounds__(kBlock, 2) void k_train_fused(TrainStepArgs A, uint32_t SX)
{
    constexpr uint32_t R = kStepRows, MB = WIDTH / 32, SA = WIDTH + 4;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ float s_ray[9][R];
    __shared__ uint32_t s_mov[R], s_nv[R], s_row[R], s_most;
    const Geom &g = A.L.g;
    const uint32_t nh = A.n_hidden, LF = (uint32_t)g.L * F, in0 = (uint32_t)g.H * LF;
    float *X = lds, *Act = X + R * SX, *Z = Act + nh * R * SA, *Gz = Z + R * kStepZ;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t li = lane & 31u, lq = lane >> 5;
    const uint32_t rows = *A.n_live, tiles = (rows + R - 1u) / R;
    f16_t dw[MAXB];
#pragma unroll
    for (int i = 0; i < MAXB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) dw[i][e] = 0.0f;
    float loss = 0.0f;
    const float inv_n = 1.0f / (float)A.L.n;
    auto act_of = [&](uint32_t k) { return Act + (k - 1u) * R * SA; };
    auto point = [&](uint32_t rr, uint32_t h, float p[3]) {   // boundary point h of row rr: its face
        VRay w;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            w.o[a] = s_ray[a][rr];
            w.d[a] = s_ray[3 + a][rr];
            w.inv[a] = s_ray[6 + a][rr];
        }
        w.mov = s_mov[rr];
        return (uint32_t)boundary_point(w, A.lists[(size_t)(h >> 1) * A.L.n + s_row[rr]], (h & 1u) != 0u, p);
    };
    float *gcopy = A.gtab + (size_t)(blockIdx.x % A.replicas) * A.n_tab;   // the copy of this XCD's blocks
    auto ld_of = [&](uint32_t k) { return k == nh ? (uint32_t)kMaxOut : (uint32_t)WIDTH; };

    for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        // ---- rays
        if (tid == 0) s_most = 0u;
        __syncthreads();
        float ta = 0.0f, tb = 0.0f;
        uint32_t ray = 0;
        const bool live = tid < R && tile * R + tid < rows;
        if (tid < R) {
            uint32_t nv = 0;
            VRay w;
            w.mov = 0;
            if (live) {
                ray = A.order[tile * R + tid];
                nv = A.L.nvox[ray];
                setup_ray(g, A.L.rays[2 * ray], A.L.rays[2 * ray + 1], w);
                ta = w.ta;
                tb = w.tb;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    s_ray[a][tid] = w.o[a];
                    s_ray[3 + a][tid] = w.d[a];
                    s_ray[6 + a][tid] = w.inv[a];
                }
            }
            s_mov[tid] = w.mov;
            s_nv[tid] = nv;
            s_row[tid] = ray;
            atomicMax(&s_most, nv);
        }
        __syncthreads();
        const uint32_t most = __builtin_amdgcn_readfirstlane(s_most);
        const uint32_t K1 = 2u * most * LF, K1r = (K1 + 31u) / 32u * 32u;   // inputs in use

        // ---- encoding, thread per (ray, point, level)
        for (uint32_t i = tid; i < R * 2u * most * (uint32_t)g.L; i += kBlock) {
            const uint32_t rr = i % R, hl = i / R, h = hl / (uint32_t)g.L, l = hl - h * (uint32_t)g.L;
            float acc[F];
#pragma unroll
            for (int f = 0; f < F; ++f) acc[f] = 0.0f;
            if (h < 2u * s_nv[rr]) {
                float p[3], wt[3];
                uint32_t c3[3];
                const uint32_t face = point(rr, h, p);
                level_cell(g, (int)l, p, c3, wt);
                const bool al = (g.aligned_mask >> l) & 1u;
                const float wf = face == 0u ? wt[0] : (face == 1u ? wt[1] : wt[2]);
                const uint32_t fb = wf != 0.0f ? 1u : 0u, low = (1u << face) - 1u;
                const char *base = reinterpret_cast<const char *>(A.tab + ((size_t)l << g.log2_T) * F);
                // 4 corners at a time: the face's on an aligned level, else the lower and upper z
                for (uint32_t half = 0; half < (al ? 1u : 2u); ++half) {
                    Entry<float, F> en[4];
                    float wc[4];
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        const uint32_t c = al ? ((q & low) | (fb << face) | ((q & ~low) << 1)) : 4u * half + q;
                        const uint32_t bx = c & 1u, by = (c >> 1) & 1u, bz = (c >> 2) & 1u;
                        wc[q] = ((bx ? wt[0] : 1.0f - wt[0]) * (by ? wt[1] : 1.0f - wt[1])) * (bz ? wt[2] : 1.0f - wt[2]);
                        en[q].load(base, vertex_slot(g, (int)l, c3[0] + bx, c3[1] + by, c3[2] + bz) * (uint32_t)(F * 4));
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q)
#pragma unroll
                        for (int f = 0; f < F; ++f) acc[f] = __builtin_fmaf(wc[q], en[q].get(f), acc[f]);
                }
            }
#pragma unroll
            for (int f = 0; f < F; ++f) X[rr * SX + hl * F + f] = acc[f];
        }
        for (uint32_t i = tid; i < R * (K1r - K1); i += kBlock) X[(i % R) * SX + K1 + i / R] = 0.0f;

        // ---- forward: layer k from its input to act_of(k + 1)
        for (uint32_t k = 0; k < nh; ++k) {
            const float *Wk = A.W + A.off[k] + lq * WIDTH + 32u * (wave % MB) + li;
            float wa[8];
            first_weights(Wk, WIDTH, wa);
            __syncthreads();
            if (wave < MB) {
                const f16_t acc = product<true>(Wk, WIDTH, k ? act_of(k) + li * SA : X + li * SX, k ? (uint32_t)WIDTH : K1, lq, wa);
                float *O = act_of(k + 1u) + li * SA + 32u * wave + 4u * lq;
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    float v[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = acc[e + t] > 0.0f ? acc[e + t] : acc[e + t] * A.slope;
                    *reinterpret_cast<float4 *>(O + 2 * e) = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        }
        __syncthreads();
        if (wave < R / 16u) {
            typedef float f4_t __attribute__((ext_vector_type(4)));
            const uint32_t i16 = lane & 15u, q4 = lane >> 4;
            const float *I = act_of(nh) + (16u * wave + i16) * SA + q4;
            const float *Wk = A.W + A.off[nh] + q4 * kMaxOut + i16;
            f4_t o4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
            for (uint32_t c = 0; c < WIDTH; c += 4u)
                o4 = __builtin_amdgcn_mfma_f32_16x16x4f32(Wk[c * kMaxOut], I[c], o4, 0, 0, 0);
            *reinterpret_cast<float4 *>(Z + (16u * wave + i16) * kStepZ + 4u * q4) = make_float4(o4[0], o4[1], o4[2], o4[3]);
        }
        __syncthreads();

        // ---- losses and their gradients
        if (tid < R) {
            float *d = Gz + tid * kStepZ;
#pragma unroll
            for (uint32_t k = 0; k < kMaxOut; ++k) d[k] = 0.0f;
            float l = 0.0f;
            if (live) {
                const lsnif_train_target y = A.L.gt[ray];
                l = ray_loss(A.L, y, ta, tb, Z + tid * kStepZ, d);
#pragma unroll
                for (uint32_t k = 0; k < kMaxOut; ++k) d[k] *= inv_n;
            }
            for (int o = 16; o >= 1; o >>= 1) l += __shfl_xor(l, o, 32);
            loss += l;
        }
        __syncthreads();

        // ---- backward, from the head down
        for (int k = (int)nh; k >= 0; --k) {
            const uint32_t ku = (uint32_t)k, ld = ld_of(ku);
            float *I = k ? act_of(ku) : X;
            const uint32_t SI = k ? SA : SX;
            const float *G = ku == nh ? Gz : act_of(ku + 1u);
            const uint32_t SG = ku == nh ? kStepZ : SA, nN = ku == nh ? 1u : MB;
            // weight gradient: input^T x G over the rows
#pragma unroll
            for (int i = 0; i < MAXB; ++i) {
                const uint32_t id = 4u * i + wave;
                if (id >= A.first[k] && id < A.first[k + 1]) {
                    const uint32_t b = id - A.first[k], mi = b / nN, ni = b - mi * nN;
                    if (k || 32u * mi < K1) {
                        const float *pa = I + lq * SI + 32u * mi + li, *pb = G + lq * SG + 32u * ni + li;
                        f16_t sum;   // the tile's: its rounding is that of 32 terms, not of all the block's
#pragma unroll
                        for (int e = 0; e < 16; ++e) sum[e] = 0.0f;
#pragma unroll
                        for (uint32_t s = 0; s < R / 2u; ++s)
                            sum = __builtin_amdgcn_mfma_f32_32x32x2f32(pa[2u * s * SI], pb[2u * s * SG], sum, 0, 0, 0);
#pragma unroll
                        for (int e = 0; e < 16; ++e) dw[i][e] += sum[e];
                    }
                }
            }
            // input gradient: G x W^T, times the derivative
            const uint32_t units = k ? (uint32_t)WIDTH : K1r, ldT = k ? (uint32_t)WIDTH : A.ldT0;
            f16_t acc;
            for (uint32_t m = wave; m < (units / 32u + 3u) / 4u * 4u; m += kBlock / 64) {
                const bool mine = 32u * m < units;
                if (mine) {
                    const float *Wt = A.WT + A.offT[k] + lq * ldT + 32u * m + li;
                    float wa[8];
                    first_weights(Wt, ldT, wa);
                    acc = product<false>(Wt, ldT, G + li * SG, ld, lq, wa);
                }
                __syncthreads();   // the weight gradients have read the layer's input
                if (!mine) continue;
#pragma unroll
                for (int e = 0; e < 16; e += 4) {
                    float4 *o = reinterpret_cast<float4 *>(I + li * SI + 32u * m + 2u * e + 4u * lq);
                    if (k) {
                        const float4 y = *o;
                        *o = make_float4(y.x > 0.0f ? acc[e] : acc[e] * A.slope, y.y > 0.0f ? acc[e + 1] : acc[e + 1] * A.slope,
                                         y.z > 0.0f ? acc[e + 2] : acc[e + 2] * A.slope,
                                         y.w > 0.0f ? acc[e + 3] : acc[e + 3] * A.slope);
                    } else {
                        *o = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
                    }
                }
            }
            __syncthreads();
        }

        // ---- tables: the points again (over the activations), then a thread per (point, level,
        // feature), the F features of a corner in adjacent lanes of one atomic instruction
        float4 *P = reinterpret_cast<float4 *>(Act);
        for (uint32_t i = tid; i < R * 2u * most; i += kBlock) {
            const uint32_t rr = i % R, h = i / R;
            if (h >= 2u * s_nv[rr]) continue;
            float p[3];
            const uint32_t face = point(rr, h, p);
            P[i] = make_float4(p[0], p[1], p[2], __uint_as_float(face));
        }
        __syncthreads();
        for (uint32_t i = tid; i < R * K1; i += kBlock) {
            const uint32_t j = i / F, f = i - j * F, rr = j % R, hl = j / R, h = hl / (uint32_t)g.L, l = hl - h * (uint32_t)g.L;
            const uint32_t points = 2u * s_nv[rr];
            if (h >= points) continue;
            const float4 v = P[h * R + rr];
            auto same = [&](uint32_t o) {
                const float4 u = P[o * R + rr];
                return u.x == v.x && u.y == v.y && u.z == v.z;
            };
            if (!(h & 1u) && h && same(h - 1u)) continue;   // added by the previous exit point
            float dx = X[rr * SX + hl * F + f];
            if ((h & 1u) && h + 1u < points && same(h + 1u)) dx += X[rr * SX + hl * F + LF + f];
            if (dx == 0.0f) continue;
            const float p[3] = {v.x, v.y, v.z};
            float wt[3];
            uint32_t c3[3];
            level_cell(g, (int)l, p, c3, wt);
            const uint32_t face = __float_as_uint(v.w);
            const bool al = (g.aligned_mask >> l) & 1u;
            const float wf = face == 0u ? wt[0] : (face == 1u ? wt[1] : wt[2]);
            const uint32_t fb = wf != 0.0f ? 1u : 0u, low = (1u << face) - 1u;
            float *dst = gcopy + ((size_t)l << g.log2_T) * F + f;
            for (uint32_t half = 0; half < (al ? 1u : 2u); ++half)
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const uint32_t c = al ? ((q & low) | (fb << face) | ((q & ~low) << 1)) : 4u * half + q;
                    const uint32_t bx = c & 1u, by = (c >> 1) & 1u, bz = (c >> 2) & 1u;
                    const float wc = ((bx ? wt[0] : 1.0f - wt[0]) * (by ? wt[1] : 1.0f - wt[1])) * (bz ? wt[2] : 1.0f - wt[2]);
                    if (wc != 0.0f)
                        unsafeAtomicAdd(dst + (size_t)vertex_slot(g, (int)l, c3[0] + bx, c3[1] + by, c3[2] + bz) * F, wc * dx);
                }
        }
    }
    // ---- this block's weight gradients and loss
    float *part = A.part + (size_t)blockIdx.x * A.n_w;
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        const uint32_t id = 4u * i + wave;
        if (id >= A.first[nh + 1u]) continue;
        uint32_t k = 0;
        while (id >= A.first[k + 1u]) ++k;
        const uint32_t nN = k == nh ? 1u : MB, b = id - A.first[k], mi = b / nN, ni = b - mi * nN;
        const uint32_t in = k ? (uint32_t)WIDTH : in0, ld = ld_of(k);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t row = 32u * mi + 8u * (e / 4) + 4u * lq + e % 4, col = 32u * ni + li;
            if (row < in && col < ld) part[A.off[k] + row * ld + col] = dw[i][e];
        }
    }
    if (tid == 0) A.loss_part[blockIdx.x] = loss;
}

template <int F, int WIDTH>
static hipError_t step_go(const TrainStepArgs &A, uint32_t in0, hipStream_t s)
{
    const uint32_t nb = A.first[A.n_hidden + 1], lds = (uint32_t)step_lds_bytes(in0, A.n_hidden, WIDTH), SX = step_x_stride(in0);
    const dim3 grid(step_blocks(A.L.n));
    if (nb <= 4u * 5u) hipLaunchKernelGGL((k_train_fused<F, WIDTH, 5>), grid, dim3(kBlock), lds, s, A, SX);
    else hipLaunchKernelGGL((k_train_fused<F, WIDTH, 9>), grid, dim3(kBlock), lds, s, A, SX);
    return hipGetLastError();
}

hipError_t launch_train_step(const TrainStepArgs &A, uint32_t F, uint32_t width, hipStream_t s)
{
    const uint32_t in0 = (uint32_t)A.L.g.H * (uint32_t)A.L.g.L * F;
    const uint32_t most = width * (A.ldT0 > width ? A.ldT0 : width);
    hipLaunchKernelGGL(k_train_transpose, dim3((most + kBlock - 1) / kBlock, A.n_hidden + 1u), dim3(kBlock), 0, s, A, in0, width);
    if (width == 128) return F == 2 ? step_go<2, 128>(A, in0, s) : step_go<3, 128>(A, in0, s);
    return F == 2 ? step_go<2, 64>(A, in0, s) : step_go<3, 64>(A, in0, s);
}

}  // namespace lsnif
