// Arguments of the training kernels (one training step of Sec. 5.2, 5.3).
#pragma once
#include "lsnif_kernels.hpp"

namespace lsnif {

// Encoding of a batch (forward: features into x0) and its transpose
// (backward: dx0 scattered onto the table gradients).  Thread = (ray, point).
struct TrainEncArgs {
    Geom g;
    const float4 *rays;
    uint32_t n;
    const uint32_t *lists;    // walk output, entry j of ray r at lists[j n + r]
    const uint8_t *nvox;
    const float *tab;         // [L][T][F] parameters
    float *gtab;              // backward: `replicas` gradient copies of [L][T][F], back to back
    uint32_t replicas;        // block b adds into copy b % replicas (blocks alternate over the XCDs)
    uint64_t n_tab;           // floats of one copy
    float *x;                 // [n][H L F]: x0 (forward) or dx0 (backward)
};

// C(i, j) = sum_k A(i, k) B(k, j) over i < M, j < N, k < K, the operands read
// through strides; gridDim.z splits K in chunks of kchunk (partial epilogue).
struct GemmArgs {
    const float *A;
    int64_t sai, sak;
    const float *B;
    int64_t sbk, sbj;
    float *C;
    int64_t ldc;
    const float *aux;         // post-activation values for the derivative epilogue, ld = ldc
    uint32_t M, N, K, kchunk;
    float slope;              // activation slope below 0 (0 for ReLU)
};

// Output tile of a block (rows x columns) and the K slice staged per step.
constexpr uint32_t kGM = 64, kGN = 64, kGK = 32;

// kEpiPartial: K chunk z stores its partial product at C + z M ldc (summed afterwards).
enum GemmEpi : int { kEpiStore = 0, kEpiAct = 1, kEpiActGrad = 2, kEpiPartial = 3 };

struct TrainLossArgs {
    Geom g;
    const float4 *rays;
    const lsnif_train_target *gt;
    uint32_t n;
    const uint8_t *nvox;
    const float *z;           // [n][ldz] raw outputs
    float *dz;                // [n][ldz] d loss / d z
    uint32_t ldz, out_dim, n_mat, has_albedo;
    float *loss_part;         // per-block sums of the per-ray losses, one float per block
};

__device__ __forceinline__ float sigmoidf(float z) { return 1.0f / (1.0f + expf(-z)); }

// Loss of one ray with outputs z over its interval [ta, tb], and d loss / d z into d (zero on entry).
__device__ __forceinline__ float ray_loss(const TrainLossArgs &A, const lsnif_train_target &y, float ta, float tb,
                                          const float *z, float d[kMaxOut])
{
    const float yh = y.hit ? 1.0f : 0.0f;
    // occlusion: softplus(z0) - y z0, the stable form
    const float z0 = z[0];
    float l = (fmaxf(z0, 0.0f) + log1pf(expf(-fabsf(z0)))) - yh * z0;
    d[0] = sigmoidf(z0) - yh;
    if (y.hit) {
        // local hit distance
        float tau = (y.t - ta) / (tb - ta);
        tau = fminf(fmaxf(tau, 0.0f), 1.0f);
        const float s1 = sigmoidf(z[1]), e1 = s1 - tau;
        l += fabsf(e1);
        d[1] = (e1 > 0.0f ? 1.0f : (e1 < 0.0f ? -1.0f : 0.0f)) * (s1 * (1.0f - s1));
        // normal: 1 - cosine similarity
        const float nn = sqrtf((z[2] * z[2] + z[3] * z[3]) + z[4] * z[4]);
        const float dot = (z[2] * y.n[0] + z[3] * y.n[1]) + z[4] * y.n[2];
        const float den = fmaxf(nn, 1e-8f);
        const float cs = dot / den;
        l += 1.0f - cs;
        for (int b = 0; b < 3; ++b)
            d[2 + b] = nn > 1e-8f ? -(y.n[b] / nn - cs * (z[2 + b] / nn) / nn) : -(y.n[b] / 1e-8f);
        uint32_t m0 = 5;
        if (A.has_albedo) {
            for (int c = 0; c < 3; ++c) {
                const float a = sigmoidf(z[5 + c]), e = a - y.albedo[c];
                const float q = (a + 0.01f) * (a + 0.01f);
                l += (e * e / q) / 3.0f;
                d[5 + c] = ((2.0f * e / q) / 3.0f) * (a * (1.0f - a));
            }
            m0 = 8;
        }
        if (y.material >= 0 && (uint32_t)y.material < A.n_mat) {
            float mx = z[m0];
            for (uint32_t k = 1; k < A.n_mat; ++k) mx = fmaxf(mx, z[m0 + k]);
            float sum = 0.0f;
            for (uint32_t k = 0; k < A.n_mat; ++k) sum += expf(z[m0 + k] - mx);
            l += (mx + logf(sum)) - z[m0 + y.material];
            for (uint32_t k = 0; k < A.n_mat; ++k)
                d[m0 + k] = expf(z[m0 + k] - mx) / sum - ((int32_t)k == y.material ? 1.0f : 0.0f);
        }
    }
    return l;
}

struct AdamArgs {
    float *p, *m, *v;
    const float *g;
    uint64_t count;
    float lr, b1, b2, eps, c1, c2;   // c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t)
    uint32_t *odd;                   // set if one of the first n_odd parameters leaves the finite numbers (for good)
    uint64_t n_odd;
};

// One training step's forward and backward passes after the walk, in one kernel.
struct TrainStepArgs {
    TrainLossArgs L;          // geometry, rays, targets, n, nvox, outputs; z, dz and loss_part unused
    const uint32_t *lists;
    const uint32_t *order, *n_live;   // rays that list voxels, and their number
    const float *tab;
    const float *W;           // packed weights
    int32_t off[8];
    float *WT;                // transposed weights, layer k at offT[k], rows of ldT0 (layer 0) or width
    uint32_t offT[8], ldT0;
    uint32_t n_hidden;
    float slope;              // activation slope below 0
    float *gtab;              // [replicas][n_tab] gradient copies
    uint32_t replicas;
    uint64_t n_tab;
    uint32_t first[9];        // first 32 x 32 block of each layer's weight gradient, and their number
    float *part;              // [blocks of the launch][n_w] weight gradients, laid out like W
    uint32_t n_w;
    float *loss_part;         // one float per block of the launch
};
// Rows a block takes at once; blocks of a launch over n rays (two to a CU).
constexpr uint32_t kStepRows = 32;
inline uint32_t step_blocks(uint32_t n) { return (n + kStepRows - 1) / kStepRows < 512u ? (n + kStepRows - 1) / kStepRows : 512u; }
// Floats of a tile's row of inputs, and of outputs or their gradients (16 used); the kernel's dynamic
// LDS for an object with in0 inputs, nh hidden layers of `width`.
constexpr uint32_t kStepZ = 20;
inline uint32_t step_x_stride(uint32_t in0) { return (in0 + 31u) / 32u * 32u + 4u; }
inline size_t step_lds_bytes(uint32_t in0, uint32_t nh, uint32_t width)
{
    return 4u * (size_t)(kStepRows * (step_x_stride(in0) + nh * (width + 4u) + 2u * kStepZ) + 32u);
}
// Blocks of 32 x 32 of layer k's weight gradient.
inline uint32_t step_grad_blocks(uint32_t in0, uint32_t nh, uint32_t width, uint32_t k)
{
    const uint32_t mb = width / 32u;
    return (k ? mb : (in0 + 31u) / 32u) * (k == nh ? 1u : mb);
}
// Whether one kernel takes a step of n rays: the weight gradients fit 9 accumulator blocks per
// wave beside two blocks to a CU, the activations the LDS; and, as a tile's encoding and
// scatter are serial work in proportion to the inputs, batches of an object with many are
// large (us, separate launches and this: 288 inputs, 2,000 rays 303 and 344, 4,096 373 and 344,
// 65,536 2,250 and 1,410; 108 inputs, 32 rays 169 and 153).  12 blocks per wave (576 inputs, one
// block to a CU): 2,000 rays 784 and 1,095, 16,384 1,100 and 1,165, 131,072 3,806 and 3,270.
inline bool step_takes(uint32_t in0, uint32_t H, uint32_t nh, uint32_t width, uint32_t n)
{
    uint32_t blocks = 0;
    for (uint32_t k = 0; k <= nh; ++k) blocks += step_grad_blocks(in0, nh, width, k);
    return blocks <= 36u && (in0 <= 128u || n >= 4096u) && 4u * H <= nh * (width + 4u) &&
           step_lds_bytes(in0, nh, width) <= (78u << 10);
}
// The row that a lane reads for row `row` of a matrix of `rows` rows.  The first layer's product runs
// over the inputs in use, padded to 32, and the packed weights end with the head's 16 rows: with one
// hidden layer the rows past the inputs would lie past the allocation.
__host__ __device__ inline uint32_t step_weight_row(uint32_t row, uint32_t rows) { return row < rows ? row : rows - 1u; }
hipError_t launch_train_step(const TrainStepArgs &A, uint32_t F, uint32_t width, hipStream_t s);
// Order of the rays that list voxels (at most `most`), longest lists first, in ws
// (order_ws_words(n) words, 16-byte aligned); *n_live (0 before) receives their number.
inline size_t order_ws_words(uint32_t n) { return radix_hist_words(n) + 3u + 2u * (size_t)n; }
hipError_t launch_train_order(const uint8_t *nvox, uint32_t n, uint32_t most, uint32_t *ws, uint32_t **order,
                              uint32_t *n_live, hipStream_t s);

// Zeroes a and b, and *live unless NULL.
hipError_t launch_train_fill(float *a, uint64_t na, float *b, uint64_t nb, uint32_t *live, hipStream_t s);
hipError_t launch_train_encode(const TrainEncArgs &A, bool backward, hipStream_t s);
hipError_t launch_train_gemm(const GemmArgs &G, int epi, hipStream_t s);
// dst[i ld + j] = sum over z < nz of part[(z M + i) N + j], i < M, j < N; part2 holds
// kSumGroups x M x N floats of scratch.
constexpr uint32_t kSumGroups = 16;
hipError_t launch_sum_partials(const float *part, uint32_t nz, uint32_t M, uint32_t N, float *part2, float *dst,
                               uint32_t ld, hipStream_t s);
// a[i] += sum over r = 1 .. copies-1 of a[r n + i], i < n.
hipError_t launch_sum_copies(float *a, uint64_t n, uint32_t copies, hipStream_t s);
hipError_t launch_train_loss(const TrainLossArgs &A, hipStream_t s);
hipError_t launch_train_loss_final(const float *part, uint32_t nparts, uint32_t n, float *loss, hipStream_t s);
hipError_t launch_adam(const AdamArgs &A, hipStream_t s);

}  // namespace lsnif
