// Types and device functions the kernels share (gfx950): kernel arguments, the
// hash-grid encoding, matrix-core operand types, decode, and the walk kernel.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>
#include <stdint.h>

#include "lsnif_device.hpp"
#include "lsnif_launch.hpp"
#include "../../include/lsnif.h"

namespace lsnif {

constexpr int kBlock = 256;
constexpr int kMaxOut = 16;

// MLP description for the kernels.
struct Mlp {
    const void *W;            // packed weights (layout depends on the kernel)
    int32_t off[8];           // element offset of each layer in W
    int32_t n_hidden;
    int32_t out_dim;
    int32_t act;              // LSNIF_RELU / LSNIF_LEAKY_RELU
    float slope;
    int32_t n_mat, has_albedo;
    int32_t kb_point;         // matrix-core path: K blocks (16 wide) per boundary point
    uint32_t odd;             // matrix-core path: not 0 if some first-layer weight is not finite
    uint32_t *odd_at;         // float32 path: the same, kept after the weights, which training moves
    const float *odd_w;       // then: the first layer as [inputs][width], read for those weights
    int32_t woff[8];          // matrix-core path: dword offset of each layer's fragments
    float qs[8];              // FP8: 1 / activation scale of each layer's input (1 otherwise)
    float dq[8];              // FP8: weight scale x activation scale of each layer (1 otherwise)
};

struct Dbg {
    int32_t *count;
    float *tatb;
    float *out;
    float *enc;
    float *act_amax;          // float32 path: largest |input| of each layer, for FP8 scales
};

// Result of one (ray, instance) pair, kept until the nearest hit is known.
struct PairRes {
    float t;                  // +inf on a miss
    float n[3];               // object-space normal
    int32_t material;
};

// A built object as the pair kernels see it (device object table, indexed by id).
struct ObjDev {
    Geom g;
    Mlp m;
    const void *tables;
    int32_t live;
};

struct PairArgs {
    const uint32_t *pair_ray;
    const uint32_t *pair_inst;
    const lsnif_instance *inst;
    const ObjDev *objs;
    const int32_t *tile_obj;      // object id of each 256-slot tile, -1 for none
    const uint32_t *slot_pair;    // pair index of each sorted slot, 0xffffffff for padding
    unsigned long long *minkey;   // per ray: (ordered t << 32) | instance of the nearest hit
    PairRes *res;                 // per pair
};

struct QueryArgs {
    Geom g;
    Mlp m;
    const void *tables;       // [L][T][F] in the feature type
    const float4 *rays;
    lsnif_hit *hits;
    uint32_t n;               // rays (single object) or sorted pair slots (pairs)
    const uint32_t *order;    // processing order of the rays (coherence sort), or NULL
    uint32_t *lists;          // voxel lists by slot: entry j of slot i at lists[j n + i]
    uint8_t *nvox;            // listed voxels of each slot
    uint32_t tile0;           // first tile of the launch (a launch may cover a range of the tiles)
    uint32_t width;           // hidden width of the launch's objects (64 or 128), picks the kernel
    Dbg dbg;
    PairArgs pr;
};

// Order-preserving map of a float to 32 unsigned bits.
__device__ __forceinline__ uint32_t ordered_bits(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Instance transform x_obj = A x + b (row-major 3x4), evaluated in the order
// ((m0 x + m1 y) + m2 z) + m3; directions are not renormalised, so t is
// shared by both spaces.  An invalid world ray stays invalid.
__device__ __forceinline__ void to_object_space(const lsnif_instance &I, float4 &r0, float4 &r1)
{
    const float in[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 6; ++i) ok = ok && (__builtin_fabsf(in[i]) <= 3.402823466e38f);
    ok = ok && (in[6] == in[6]) && (in[7] == in[7]);
    ok = ok && !(in[3] == 0.0f && in[4] == 0.0f && in[5] == 0.0f) && !(in[6] > in[7]);
    float o[3], d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float *m = I.world_to_object + 4 * a;
        o[a] = ((m[0] * in[0] + m[1] * in[1]) + m[2] * in[2]) + m[3];
        d[a] = (m[0] * in[3] + m[1] * in[4]) + m[2] * in[5];
    }
    r0 = make_float4(ok ? o[0] : __builtin_nanf(""), o[1], o[2], d[0]);
    r1 = make_float4(d[1], d[2], in[6], in[7]);
}

template <typename TF> __device__ __forceinline__ float to_f32(TF v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<_Float16>(_Float16 v) { return (float)v; }
template <> __device__ __forceinline__ float to_f32<__bf16>(__bf16 v) { return (float)v; }

template <typename TF> __device__ __forceinline__ float lo16(uint32_t x)
{
    uint16_t u = (uint16_t)(x & 0xffffu);
    TF v;
    __builtin_memcpy(&v, &u, 2);
    return to_f32<TF>(v);
}
template <typename TF> __device__ __forceinline__ float hi16(uint32_t x)
{
    uint16_t u = (uint16_t)(x >> 16);
    TF v;
    __builtin_memcpy(&v, &u, 2);
    return to_f32<TF>(v);
}

// Raw bytes of one table entry (F features of type TF) at byte offset `off`.
template <typename TF, int F> struct Entry {
    static constexpr int W = (F * (int)sizeof(TF) + 3) / 4;   // dwords
    uint32_t d[W];
    __device__ __forceinline__ void load(const char *base, uint32_t off)
    {
        if constexpr (F * sizeof(TF) == 4) {
            d[0] = *reinterpret_cast<const uint32_t *>(base + off);
        } else if constexpr (F * sizeof(TF) == 8) {
            uint2 x = *reinterpret_cast<const uint2 *>(base + off);
            d[0] = x.x;
            d[1] = x.y;
        } else if constexpr (F * sizeof(TF) == 16) {
            uint4 x = *reinterpret_cast<const uint4 *>(base + off);
            d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w;
        } else if constexpr (F == 3 && sizeof(TF) == 2) {
            // one 8-byte load from a 2-byte boundary: the 6 bytes and 2 that nothing reads (after
            // the last entry, spare ones)
            typedef uint32_t u32x2a2 __attribute__((ext_vector_type(2), aligned(2)));
            const u32x2a2 x = *reinterpret_cast<const u32x2a2 *>(base + off);
            d[0] = x.x;
            d[1] = x.y;
        } else {
            static_assert(F == 3 && sizeof(TF) == 4, "2 or 3 features");
            const uint32_t *x = reinterpret_cast<const uint32_t *>(base + off);
            d[0] = x[0]; d[1] = x[1]; d[2] = x[2];
        }
    }
    // An opaque use of the loaded dwords: nothing that reads them can be
    // moved above this point, so a batch of gathers is issued in full first.
    __device__ __forceinline__ void pin()
    {
#pragma unroll
        for (int k = 0; k < W; ++k) asm volatile("" : "+v"(d[k]));
    }
    __device__ __forceinline__ float get(int f) const
    {
        if constexpr (sizeof(TF) == 4) return __uint_as_float(d[f]);
        else return (f & 1) ? hi16<TF>(d[f >> 1]) : lo16<TF>(d[f >> 1]);
    }
};

// Cell of point p on level l and the weights inside it, as level_cell, with the
// clamps as min/max (the debug path keeps level_cell itself).
__device__ __forceinline__ void level_cell_mm(const Geom &g, int l, const float p[3], uint32_t i[3], float wt[3])
{
    const float Rf = (float)g.R[l], sc = g.lsc[l];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const float x = __builtin_amdgcn_fmed3f(p[b] * sc, 0.0f, Rf);   // clamp to [0, R]
        const float k = __builtin_fminf(__builtin_floorf(x), Rf - 1.0f);
        i[b] = (uint32_t)k;
        wt[b] = x - k;
    }
}

// The last multiply-add of a sum that is rounded to FP16 next.  In one instruction the two
// are one rounding; the compiler finds it only where both lie in one basic block, so a
// caller with several ways to the rounding takes it here (the result is exact in float).
__device__ __forceinline__ float fma_f16(float a, float b, float c)
{
    const _Float16 h = (_Float16)__builtin_fmaf(a, b, c);
    uint16_t u;
    __builtin_memcpy(&u, &h, 2);
    uint32_t x = u;
    asm volatile("" : "+v"(x));   // keeps both halves here
    return lo16<_Float16>(x);
}

// Interpolated features of NL consecutive levels l0 .. l0 + NL - 1 at the
// boundary point p (voxel units) whose crossing axis is `face`; levels at or
// beyond L give zeros.  All slots are formed first and all gathers issued
// before any is consumed.  On a level aligned with the voxel faces the
// crossing-axis weight is exactly 0 or 1, and the 4 zero-weight corners do
// not touch their own entries (they read the level's first entry).
// H16: the features are rounded to FP16 (fma_f16).
template <typename TF, int F, int NL, bool H16 = false>
__device__ __forceinline__ void encode_levels(const Geom &g, const TF *__restrict__ tab, int l0, const float p[3],
                                              int face, float out[NL][F])
{
    const char *base[NL];
    uint32_t off[NL][8];
    float wx[NL][2], wy[NL][2], wz[NL][2];
    constexpr uint32_t esz = F * sizeof(TF);
#pragma unroll
    for (int lv = 0; lv < NL; ++lv) {
        const int l = l0 + lv < g.L ? l0 + lv : g.L - 1;
        uint32_t i[3];
        float wt[3];
        level_cell_mm(g, l, p, i, wt);
        // With a power-of-two entry size the byte offset is formed directly: scaling
        // x, y my and z mz by esz commutes with the sum and, as a shift, with the xor
        // and the mask.
        constexpr uint32_t sh = esz == 4 ? 2u : (esz == 8 ? 3u : (esz == 16 ? 4u : 0u));
        constexpr bool scaled = sh != 0u;
        const uint32_t my = g.my[l] << sh, mz = g.mz[l] << sh;
        const uint32_t x0 = i[0] << sh;
        uint32_t t[3][2] = {{x0, x0 + (1u << sh)}, {i[1] * my, i[1] * my + my}, {i[2] * mz, i[2] * mz + mz}};
        // vertex slot: x + y + z on a directly indexed level, (x ^ y ^ z) & (T - 1) on a
        // hashed one (y, z already times their multipliers); the level kind is wave-uniform
        constexpr uint32_t m = scaled ? 1u : esz;
        if ((g.dense_mask >> l) & 1u) {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                off[lv][c] = (t[0][c & 1] + t[1][(c >> 1) & 1] + t[2][c >> 2]) * m;
        } else {
            const uint32_t hm = g.hmask[l] << sh;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t yz = t[1][q & 1] ^ t[2][q >> 1];
                off[lv][2 * q] = ((t[0][0] ^ yz) & hm) * m;
                off[lv][2 * q + 1] = ((t[0][1] ^ yz) & hm) * m;
            }
        }
        if ((g.aligned_mask >> l) & 1u) {
            // On a face-aligned level the crossing axis' weight is exactly 0 or 1, so the 4
            // corners on the other side weigh 0.  They read the level's first entry: one
            // line for every lane, where their own slots would cost the addresser a line
            // per lane.  Weight 0 times a finite entry adds nothing (the sum is never -0).
            const float wf = face == 0 ? wt[0] : (face == 1 ? wt[1] : wt[2]);
            const uint32_t fb = 1u << face, keep = wf != 0.0f ? fb : 0u;
#pragma unroll
            for (int c = 0; c < 8; ++c) off[lv][c] = ((uint32_t)c & fb) == keep ? off[lv][c] : 0u;
        }
        wx[lv][0] = 1.0f - wt[0]; wx[lv][1] = wt[0];
        wy[lv][0] = 1.0f - wt[1]; wy[lv][1] = wt[1];
        wz[lv][0] = 1.0f - wt[2]; wz[lv][1] = wt[2];
        base[lv] = reinterpret_cast<const char *>(tab + ((size_t)l << g.log2_T) * F);
    }
    Entry<TF, F> e[NL][8];
    typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
    for (int lv = 0; lv < NL; ++lv) {
        const int l = l0 + lv < g.L ? l0 + lv : g.L - 1;
        const bool pairx = F * sizeof(TF) == 4 && ((g.dense_mask & ~g.aligned_mask) >> l) & 1u;
        if (pairx) {
            // directly indexed level: the two x-vertices of an edge are adjacent entries
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const u32x2a4 v = *reinterpret_cast<const u32x2a4 *>(base[lv] + off[lv][2 * q]);
                e[lv][2 * q].d[0] = v.x;
                e[lv][2 * q + 1].d[0] = v.y;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) e[lv][c].load(base[lv], off[lv][c]);
        }
    }
    // keep every gather of the batch in flight before the first is consumed
    asm volatile("" ::: "memory");
#pragma unroll
    for (int lv = 0; lv < NL; ++lv)
#pragma unroll
        for (int c = 0; c < 8; ++c) e[lv][c].pin();
#pragma unroll
    for (int lv = 0; lv < NL; ++lv) {
#pragma unroll
        for (int f = 0; f < F; ++f) out[lv][f] = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float wyz = wy[lv][q & 1] * wz[lv][q >> 1];
#pragma unroll
            for (int xb = 0; xb < 2; ++xb) {
                const float w = wx[lv][xb] * wyz;
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const float x = e[lv][2 * q + xb].get(f);
                    out[lv][f] = H16 && q == 3 && xb == 1 ? fma_f16(w, x, out[lv][f]) : __builtin_fmaf(w, x, out[lv][f]);
                }
            }
        }
        if (l0 + lv >= g.L) {
#pragma unroll
            for (int f = 0; f < F; ++f) out[lv][f] = 0.0f;
        }
    }
}

// encode_levels for levels that are all aligned with the voxel faces: the crossing-axis
// weight of a boundary point is exactly 0 or 1 there, so the features are sums over the
// 4 corners of its face.  encode_levels' 4 other corners weigh 0 and leave its sum as it
// is; its last addition (corner 7) may be rounded together with the conversion of the sum,
// so the last addition here is the fourth corner's where that is corner 7, and one of 0
// where it is not.
template <typename TF, int F, int NL, bool H16>
__device__ __forceinline__ void encode_aligned(const Geom &g, const TF *__restrict__ tab, int l0, const float p[3],
                                               int face, float out[NL][F])
{
    constexpr uint32_t esz = F * sizeof(TF);
    constexpr uint32_t sh = esz == 4 ? 2u : (esz == 8 ? 3u : (esz == 16 ? 4u : 0u));
    constexpr uint32_t m = sh ? 1u : esz;
    Entry<TF, F> e[NL][4];
    float wu[NL], wv[NL];
    bool up[NL];
#pragma unroll
    for (int lv = 0; lv < NL; ++lv) {
        const int l = l0 + lv < g.L ? l0 + lv : g.L - 1;
        uint32_t i[3];
        float wt[3];
        level_cell_mm(g, l, p, i, wt);
        const uint32_t my = g.my[l] << sh, mz = g.mz[l] << sh;
        const uint32_t x0 = i[0] << sh, x1 = x0 + (1u << sh), y0 = i[1] * my, y1 = y0 + my, z0 = i[2] * mz, z1 = z0 + mz;
        // u, v: the axes of the face, in order; f: the face's vertex on the crossing axis
        up[lv] = (face == 0 ? wt[0] : (face == 1 ? wt[1] : wt[2])) != 0.0f;
        const uint32_t f0 = face == 0 ? x0 : (face == 1 ? y0 : z0), f1 = face == 0 ? x1 : (face == 1 ? y1 : z1);
        const uint32_t f = up[lv] ? f1 : f0;
        const uint32_t u[2] = {face == 0 ? y0 : x0, face == 0 ? y1 : x1};
        const uint32_t v[2] = {face == 2 ? y0 : z0, face == 2 ? y1 : z1};
        wu[lv] = face == 0 ? wt[1] : wt[0];
        wv[lv] = face == 2 ? wt[1] : wt[2];
        const char *base = reinterpret_cast<const char *>(tab + ((size_t)l << g.log2_T) * F);
        uint32_t off[4];
        if ((g.dense_mask >> l) & 1u) {
#pragma unroll
            for (int q = 0; q < 4; ++q) off[q] = (f + u[q & 1] + v[q >> 1]) * m;
        } else {
            const uint32_t hm = g.hmask[l] << sh;
#pragma unroll
            for (int q = 0; q < 4; ++q) off[q] = ((f ^ u[q & 1] ^ v[q >> 1]) & hm) * m;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) e[lv][q].load(base, off[q]);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int lv = 0; lv < NL; ++lv)
#pragma unroll
        for (int q = 0; q < 4; ++q) e[lv][q].pin();
#pragma unroll
    for (int lv = 0; lv < NL; ++lv) {
        const float u0 = 1.0f - wu[lv], u1 = wu[lv], v0 = 1.0f - wv[lv], v1 = wv[lv];
        const float w3 = u1 * v1;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            float s = __builtin_fmaf(u0 * v0, e[lv][0].get(f), 0.0f);
            s = __builtin_fmaf(u1 * v0, e[lv][1].get(f), s);
            s = __builtin_fmaf(u0 * v1, e[lv][2].get(f), s);
            const float x3 = e[lv][3].get(f), a = up[lv] ? s : __builtin_fmaf(w3, x3, s);
            const float xl = up[lv] ? x3 : 0.0f;   // not a weight of 0: x3 may be infinite
            out[lv][f] = H16 ? fma_f16(w3, xl, a) : __builtin_fmaf(w3, xl, a);
        }
        if (l0 + lv >= g.L) {
#pragma unroll
            for (int f = 0; f < F; ++f) out[lv][f] = 0.0f;
        }
    }
}

__device__ __forceinline__ float act_f(float x, int act, float slope)
{
    return x > 0.0f ? x : (act == LSNIF_LEAKY_RELU ? x * slope : 0.0f);
}

// Largest non-negative value of the wave folded into *dst (float bits of
// non-negative numbers order like unsigned integers).
__device__ __forceinline__ void fold_max(float *dst, float v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax2(v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63u) == 0) atomicMax(reinterpret_cast<unsigned int *>(dst), __float_as_uint(v));
}

// Output heads (Sec. 5.1, 5.3): occlusion logit > 0 is a hit, the hit
// distance is the sigmoid of its logit over [ta, tb], the normal is the
// normalised linear head, the material the arg-max logit.
template <bool PAIRS>
__device__ __forceinline__ void decode_store(const QueryArgs &A, const Mlp &mm, uint32_t r, uint32_t pair,
                                             const VRay &w, int count, const float *o)
{
    lsnif_hit h;
    h.hit = 0;
    h.t = __builtin_inff();
    h.n[0] = h.n[1] = h.n[2] = 0.0f;
    h.material = -1;
    if (count > 0) {
        const float sig = 1.0f / (1.0f + expf(-o[1]));
        const float th = w.ta + sig * (w.tb - w.ta);
        if (o[0] > 0.0f && th <= w.tmax) {
            h.hit = 1;
            h.t = th;
            const float nn = o[2] * o[2] + o[3] * o[3] + o[4] * o[4];
            if (nn > 0.0f) {
                const float inv = 1.0f / __builtin_sqrtf(nn);
                h.n[0] = o[2] * inv;
                h.n[1] = o[3] * inv;
                h.n[2] = o[4] * inv;
            }
            // argmax over the material logits o[m0 .. m0 + n_mat), ties to the lowest index;
            // written over the static slots of o so that o stays in registers
            const int m0 = 5 + 3 * mm.has_albedo;
            int best = 0;
            float bv = 0.0f;
#pragma unroll
            for (int k = 5; k < kMaxOut; ++k) {
                const int mk = k - m0;
                if (mk >= 0 && mk < mm.n_mat && (mk == 0 || o[k] > bv)) {
                    bv = o[k];
                    best = mk;
                }
            }
            h.material = best;
        }
    }
    if constexpr (!PAIRS) {
        A.hits[r] = h;
    } else {
        PairRes pr;
        pr.t = h.t;
        pr.n[0] = h.n[0];
        pr.n[1] = h.n[1];
        pr.n[2] = h.n[2];
        pr.material = h.material;
        A.pr.res[pair] = pr;
        if (h.hit) {
            const unsigned long long key =
                ((unsigned long long)ordered_bits(h.t) << 32) | (unsigned long long)A.pr.pair_inst[pair];
            atomicMin(&A.pr.minkey[r], key);
        }
    }
}

// Tile of rays (or pairs) this block works on.  The dispatcher deals
// workgroups to the 8 XCDs in turn (block b runs on XCD b mod 8), each XCD with
// an L2 of its own, and tiles follow the coherence order of the rays.  Runs of
// C consecutive tiles go to one XCD, so the rays an XCD has in flight lie in
// fewer regions of the object and share more of its L2; short runs keep the
// work of the XCDs even where the cost per tile drifts along the order.  Any
// grid size maps one to one (the last partial round keeps b itself).  A launch
// covers tiles tile0 .. tile0 + gridDim.x - 1.
__device__ __forceinline__ uint32_t block_tile(uint32_t tile0)
{
    constexpr uint32_t C = 8;
    const uint32_t b = blockIdx.x, nb = gridDim.x;
    const uint32_t full = nb / (8u * C) * (8u * C);
    if (b >= full) return tile0 + b;
    const uint32_t x = b & 7u, k = b >> 3;
    return tile0 + ((k / C) * 8u + x) * C + k % C;
}

template <bool PAIRS>
__device__ __forceinline__ void slot_ray(const QueryArgs &A, const Geom &g, uint32_t slot, uint32_t &r,
                                         uint32_t &pair, bool &live, VRay &w)
{
    r = 0u;
    pair = 0xffffffffu;
    if constexpr (PAIRS) {
        pair = slot < A.n ? A.pr.slot_pair[slot] : 0xffffffffu;
        live = pair != 0xffffffffu;
        if (live) r = A.pr.pair_ray[pair];
    } else {
        live = slot < A.n;
        if (live) r = A.order ? A.order[slot] : slot;
    }
    w.valid = w.cand = false;
    w.ta = w.tb = w.tmax = w.tmin = 0.0f;
    w.mov = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) w.o[a] = w.d[a] = w.inv[a] = 0.0f;
    if (live) {
        float4 ra = A.rays[2 * r], rb = A.rays[2 * r + 1];
        if constexpr (PAIRS) to_object_space(A.pr.inst[A.pr.pair_inst[pair]], ra, rb);
        setup_ray(g, ra, rb, w);
    }
}

// The voxel walk of every slot, in a kernel of its own: it needs few registers,
// so many waves per SIMD hide the latency of its dependent brick-mask loads,
// which the query kernels (four waves per SIMD, each with gathers of its own to wait for) could not.
template <bool PAIRS, bool RECHECK>
__device__ __forceinline__ void walk_body(const QueryArgs &A, const Geom &g, uint32_t *coarse)
{
    const uint32_t tid = threadIdx.x;
    const bool lds_coarse = g.coarse_words <= kCoarseLdsWords;
    if (lds_coarse)
        for (int i = tid; i < g.coarse_words; i += kBlock) coarse[i] = g.coarse[i];
    __syncthreads();
    const uint32_t slot = block_tile(A.tile0) * kBlock + tid;
    uint32_t r, pair;
    bool live;
    VRay w;
    slot_ray<PAIRS>(A, g, slot, r, pair, live, w);
    int nvox = 0;
    if (live) {
        uint32_t *list = A.lists + slot;
        nvox = lds_coarse ? walk_voxels<RECHECK>(g, w, coarse, list, A.n, g.H >> 1)
                          : walk_voxels<RECHECK>(g, w, g.coarse, list, A.n, g.H >> 1);
    }
    if (slot < A.n) A.nvox[slot] = (uint8_t)nvox;
}

// Object of this block's tile: one value for the whole block, read through the
// scalar path so that everything derived from it (tables, weights) stays uniform.
__device__ __forceinline__ int tile_object(const PairArgs &P, uint32_t tile)
{
    typedef const __attribute__((address_space(4))) int32_t cint;
    return __builtin_amdgcn_readfirstlane(((cint *)P.tile_obj)[tile]);
}
// The object table, read through the constant address space in the device pass (the
// host pass only type-checks kernel bodies and has no such address space).
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) ObjDev cObjDev;
#else
typedef const ObjDev cObjDev;
#endif

// ------------------------------------------------------------ matrix-core types
//
// Layer k computes D = W_k * X with the weights as the A operand (M = output
// units, 32 per block) and the activations as the B operand (N = rays, 32 per
// block), v_mfma_f32_32x32x16.  Operand layout per lane l (i = l % 32, half
// q = l / 32): A holds W[i][8q .. 8q+7] of the K block, B holds X[8q .. 8q+7][i],
// and the 16 accumulators hold D[8(r/4) + 4q + r%4][i], r = 0..15.  Hidden
// layers take the accumulators as they lie: K slot 8q + e of 16-block s of
// output block m stands for unit 32m + 16s + (e < 4 ? 4q + e : 8 + 4q + e - 4);
// the host packs the weights of later layers in that order.
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef float f16_t __attribute__((ext_vector_type(16)));

// MLP types of the matrix-core path.  Every fragment holds 8 values per
// lane (DW dwords); FP8 values are OCP e4m3 with a per-layer scale.
struct fp8e4m3 {};
typedef long f8x8_t;

template <typename TM> struct MmaT;
template <> struct MmaT<_Float16> {
    typedef h8_t vec;
    static constexpr int DW = 4;
    static constexpr bool scaled = false;
    static __device__ __forceinline__ f16_t mma(vec a, vec b, f16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct MmaT<__bf16> {
    typedef b8_t vec;
    static constexpr int DW = 4;
    static constexpr bool scaled = false;
    static __device__ __forceinline__ f16_t mma(vec a, vec b, f16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct MmaT<fp8e4m3> {
    typedef f8x8_t vec;
    static constexpr int DW = 2;
    static constexpr bool scaled = true;
    static __device__ __forceinline__ f16_t mma(vec a, vec b, f16_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a, b, c, 0, 0, 0);
    }
};

// Two 16-bit TM values in one dword.
template <typename TM> __device__ __forceinline__ uint32_t pack2(float a, float b)
{
    TM x = (TM)a, y = (TM)b;
    uint16_t u, v;
    __builtin_memcpy(&u, &x, 2);
    __builtin_memcpy(&v, &y, 2);
    return (uint32_t)u | ((uint32_t)v << 16);
}

// Eight values, times `scale`, rounded to TM and packed into DW dwords.
template <typename TM>
__device__ __forceinline__ void pack8(const float *v, float scale, uint32_t *d)
{
    if constexpr (MmaT<TM>::scaled) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = v[e] * scale;
            x[e] = y < -448.0f ? -448.0f : (y > 448.0f ? 448.0f : y);   // saturate to the e4m3 range
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(x[4 * q], x[4 * q + 1], 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(x[4 * q + 2], x[4 * q + 3], w, true);
            d[q] = (uint32_t)w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q] = pack2<TM>(v[2 * q], v[2 * q + 1]);
    }
}

template <typename V8, int DW> __device__ __forceinline__ V8 as_vec(const uint32_t *d)
{
    V8 v;
    __builtin_memcpy(&v, d, 4 * DW);
    return v;
}

// One weight fragment (DW dwords of this lane).
template <int DW> __device__ __forceinline__ void load_frag(const uint32_t *p, uint32_t *d)
{
    if constexpr (DW == 4) {
        const uint4 x = *reinterpret_cast<const uint4 *>(p);
        d[0] = x.x; d[1] = x.y; d[2] = x.z; d[3] = x.w;
    } else {
        const uint2 x = *reinterpret_cast<const uint2 *>(p);
        d[0] = x.x; d[1] = x.y;
    }
}

// ------------------------------------------------------------------ broad phase
struct BroadArgs {
    const float4 *rays;
    uint32_t n_rays;
    const lsnif_instance *inst;
    uint32_t n_inst;
    const ObjDev *objs;       // object table by id
    uint32_t n_objs;
    uint32_t *offsets;        // [n_rays + 1]: pairs per ray, then their exclusive scan
    uint32_t *pair_ray, *pair_inst;
    // With at most kBroadMaskInst instances a first pass records which of them each ray meets,
    // a byte for every 8 (bit i % 8 of masks[(i / 8) n_rays + r]); the counting and the
    // writing pass read those bytes.
    uint8_t *masks;           // NULL: more instances
    uint32_t *part;           // partial sums of the scan of the counts
};
constexpr uint32_t kBroadMaskInst = 256;

// ------------------------------------------------------------ merged serving
// One member of a merged serving launch: its own buffers and where its rays and
// pairs start in the staged arrays.
struct MergeMember {
    const float4 *rays;           // [2 n_rays] (a ray is two float4)
    lsnif_hit *out;               // [n_rays]
    const uint32_t *pair_ray, *pair_inst;   // [n_pairs] (pair requests)
    uint32_t ray0, pair0, n_rays, n_pairs;
};
constexpr uint32_t kMergeMax = 32;   // members of one merged launch (the kernel argument holds them)
struct MergeArgs {
    MergeMember m[kMergeMax];
    uint32_t n_members, n_rays, n_pairs;
    float4 *rays;                 // staged rays [2 n_rays]
    uint32_t *pair_ray, *pair_inst;   // staged pairs [n_pairs]
    lsnif_hit *out;               // staged answers [n_rays]
};
static_assert(sizeof(MergeArgs) <= 4096, "merged-launch arguments must fit a kernel's argument space");

// ------------------------------------------------------------------ bounce rays
struct BounceArgs {
    const float4 *rays;       // the rays just answered (world space)
    const lsnif_hit *hits;    // their nearest hits
    uint32_t n;
    uint32_t seed, bounce;
    float eps;                // offset of the new origin along the facing normal
    uint32_t *offsets;        // [n + 1]: 1 per hit, then their exclusive scan
    float4 *next;             // new rays, compacted in the order of their parents
    uint32_t *parent;         // index of each new ray's parent
};

// PCG hash (Jarzynski and Olano 2020, "Hash Functions for GPU Rendering"): a
// 32-bit counter-based generator, one permuted congruential step of the input.
__device__ __forceinline__ uint32_t pcg_hash(uint32_t v)
{
    const uint32_t state = v * 747796405u + 2891336453u;
    const uint32_t word = ((state >> ((state >> 28u) + 4u)) ^ state) * 277803737u;
    return (word >> 22u) ^ word;
}

// ------------------------------------------------------------------ voxel walk
// RECHECK: some object of the launch asks for the float64 re-decision of grazing voxels.
template <bool PAIRS, bool RECHECK>
__global__ __launch_bounds__(kBlock) void k_walk(QueryArgs A)
{
    __shared__ uint32_t coarse[kCoarseLdsWords];
    if constexpr (PAIRS) {
        const int o = tile_object(A.pr, block_tile(A.tile0));
        if (o < 0) return;   // the query kernel skips such a tile too
        const cObjDev &O = ((const cObjDev *)A.pr.objs)[o];
        walk_body<true, RECHECK>(A, O.g, coarse);
    } else {
        walk_body<false, RECHECK>(A, A.g, coarse);
    }
}

// ------------------------------------------------------------------ debug path
struct DebugArgs {
    Geom g;
    const float4 *rays;
    uint32_t n;
    lsnif_debug_bufs b;
};

}  // namespace lsnif
