// The query kernel: boundary points, encoding, every MLP layer on the matrix cores, decode.
#pragma once
#include "lsnif_kernels.hpp"
#include "lsnif_launch.hpp"

namespace lsnif {

// How a point's features lie in LDS, and the matrix-core steps that read them, for
// an MLP type.  16- and 8-bit types: v_mfma_f32_32x32x16, a batch of levels
// fills one unit of 8 K slots (features padded to FP per level); lane (i, q) of a
// step reads unit 2 kb + q.  float: v_mfma_f32_32x32x2f32, whose result is the chain
// of fused multiply-adds in ascending K bit for bit; lane (i, q) takes feature
// 2 s + q in step s, so the even features of a point lie together, then the odd ones.
template <typename TM, int F> struct PointT {
    static constexpr bool f32 = false;
    static constexpr int FP = F == 3 ? 4 : F;
    static constexpr int NLB = 8 / FP;            // levels per batch
    static constexpr uint32_t UB = 4u * MmaT<TM>::DW;   // bytes of a unit
};
template <int F> struct PointT<float, F> {
    static constexpr bool f32 = true;
    static constexpr int FP = F;
    static constexpr int NLB = F == 3 ? 2 : 4;
    static constexpr uint32_t UB = 16u;
};

template <typename TM, int F> __host__ __device__ inline uint32_t level_batches(int L)
{
    return ((uint32_t)L + PointT<TM, F>::NLB - 1u) / PointT<TM, F>::NLB;
}
// LDS bytes of one point's features.
template <typename TM, int F> __host__ __device__ inline uint32_t point_bytes(int L)
{
    if constexpr (PointT<TM, F>::f32) {
        const uint32_t half = (level_batches<TM, F>(L) * PointT<TM, F>::NLB * F + 1u) / 2u;
        return 2u * ((half + 3u) / 4u * 16u);
    } else {
        return (level_batches<TM, F>(L) + 1u) / 2u * 2u * PointT<TM, F>::UB;
    }
}
// LDS bytes of the activations handed from layer to layer, and of the outputs.
template <typename TM, int WIDTH, int R> constexpr uint32_t exchange_bytes()
{
    constexpr uint32_t cols = R < 32 ? 32 : R;
    constexpr uint32_t x = PointT<TM, 2>::f32 ? cols * (WIDTH + 4) * 4u : cols * WIDTH / 8u * PointT<TM, 2>::UB;
    return x + cols * (kMaxOut + 1) * 4u;
}
// Dynamic LDS of a launch: room for the points of `vox` voxels of every ray of a tile.
template <typename TM, int F, int WIDTH, int R> inline uint32_t query_lds_bytes(int L, uint32_t vox)
{
    const uint32_t pts = 2u * R * vox, pb = point_bytes<TM, F>(L);
    const uint32_t need = (pts + 1u) * pb + pts * 16u + pts * 2u + 64u;
    const uint32_t x = exchange_bytes<TM, WIDTH, R>();
    return ((need > x ? need : x) + 15u) / 16u * 16u;
}

constexpr uint32_t kSameSlot = 0xffffu;   // the point repeats the one before it

template <int R> struct QueryShared {
    float ray[9][R];          // o, d, inv
    uint8_t mov[R], nvox[R];
    uint32_t npts;
    uint32_t most[R > 32 ? R / 32 : 1];   // largest voxel count of each 32 rays
};

// Tile of R slots of this block: as block_tile, runs of 2,048 slots to an XCD.
template <int R> __device__ __forceinline__ uint32_t block_subtile(uint32_t tile0)
{
    constexpr uint32_t C = 8u * kBlock / R;
    const uint32_t b = blockIdx.x, nb = gridDim.x, first = tile0 * (kBlock / R);
    const uint32_t full = nb / (8u * C) * (8u * C);
    if (b >= full) return first + b;
    const uint32_t x = b & 7u, k = b >> 3;
    return first + ((k / C) * 8u + x) * C + k % C;
}

// The boundary points of voxels j0 .. j0 + nj - 1 of a tile's rays, by all of a block: the distinct ones,
// packed, into pts (their number into S.npts), and for point h of ray i its place there into
// smap[h R + i]: `zero` past the ray's list, kSameSlot where it repeats the point before it.
template <int R>
__device__ __forceinline__ void pack_points(const QueryArgs &A, uint32_t slot0, uint32_t j0, uint32_t nj, uint32_t zero,
                                            QueryShared<R> &S, float4 *pts, uint16_t *smap)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) S.npts = 0u;
    __syncthreads();
    for (uint32_t i0 = wave * 64u; i0 < nj * R; i0 += kBlock) {
        const uint32_t jj = (i0 + lane) / R, j = j0 + jj, ray = (i0 + lane) % R;
        const bool has = jj < nj && j < S.nvox[ray];
        float p0[3] = {}, p1[3] = {};
        int f0 = 0, f1 = 0;
        bool dup = false;
        if (has) {
            VRay v;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                v.o[a] = S.ray[a][ray];
                v.d[a] = S.ray[3 + a][ray];
                v.inv[a] = S.ray[6 + a][ray];
            }
            v.mov = S.mov[ray];
            const uint32_t *list = A.lists + slot0 + ray;
            const uint32_t c = list[(size_t)j * A.n];
            f0 = boundary_point(v, c, false, p0);
            f1 = boundary_point(v, c, true, p1);
            if (jj > 0u) {
                // the entry point is often the exit point of the voxel before it
                float q[3];
                const int fq = boundary_point(v, list[(size_t)(j - 1u) * A.n], true, q);
                dup = fq == f0 && __float_as_uint(q[0]) == __float_as_uint(p0[0]) &&
                      __float_as_uint(q[1]) == __float_as_uint(p0[1]) &&
                      __float_as_uint(q[2]) == __float_as_uint(p0[2]);
            }
        }
        const uint64_t m_in = __ballot(has && !dup), m_out = __ballot(has);
        const uint32_t n_in = (uint32_t)__builtin_popcountll(m_in);
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&S.npts, n_in + (uint32_t)__builtin_popcountll(m_out));
        base = __builtin_amdgcn_readfirstlane(base);
        const uint64_t below = (1ull << lane) - 1ull;
        const uint32_t s0 = base + (uint32_t)__builtin_popcountll(m_in & below);
        const uint32_t s1 = base + n_in + (uint32_t)__builtin_popcountll(m_out & below);
        if (jj < nj) {
            smap[(2u * jj) * R + ray] = (uint16_t)(has ? (dup ? kSameSlot : s0) : zero);
            smap[(2u * jj + 1u) * R + ray] = (uint16_t)(has ? s1 : zero);
        }
        if (has && !dup) pts[s0] = make_float4(p0[0], p0[1], p0[2], __int_as_float(f0));
        if (has) pts[s1] = make_float4(p1[0], p1[1], p1[2], __int_as_float(f1));
    }
    __syncthreads();
}

// One block answers a tile of R slots whose voxel lists the walk has written.
//
// The encoding's gathers bound the kernel, so what matters is that every lane of every
// gather has a point of its own: the entry and exit points of the tile's voxels, without
// those that repeat the exit before them, are packed into LDS, and a wave takes 64 of them
// and one batch of levels at a time, leaving the features in LDS as the first layer's B
// operand.  With a ray per lane instead, 62 % of the lanes of a gather carried such a point
// (rays differ in length) and a wave held 64 accumulators while it gathered; here a wave
// holds the 16 or 32 of its own output block, and a ray's points are encoded side by side
// rather than one after another, which is what small launches wait for.  Every feature,
// product and sum is what a ray alone would get, in the same order, whatever its tile.
// Points are taken `vox` voxels of every ray at a time, as many as the LDS holds.
// Measured (ms, a ray per lane before / now): 2,097,152 rays FP16 1.90 / 1.71, 1,000,003 FP8
// 0.99 / 0.66, 39,999 0.204 / 0.115, 256 0.046 / 0.018; float32 MLPs, then on the vector ALU
// with weights from scalar loads: 524,288 rays of width 64 2.40 / 1.16, 262,144 of width 128
// 2.09 / 0.25.
template <typename TF, typename TM, int F, int WIDTH, bool PAIRS, int R>
__device__ __forceinline__ void query_body(const QueryArgs &A, const Geom &g, const Mlp &mm, const TF *__restrict__ tab,
                                          QueryShared<R> &S, char *lds, uint32_t lds_bytes, uint32_t tile)
{
    typedef PointT<TM, F> P;
    typedef const __attribute__((address_space(4))) uint32_t cword;
    constexpr bool f32 = P::f32;
    constexpr int DW = f32 ? 4 : (int)P::UB / 4;      // dwords of a unit / fragment
    constexpr int MB = WIDTH / 32, NB = R > 32 ? R / 32 : 1;
    constexpr int NT = kBlock, NW = NT / 64;
    // A wave's output blocks: one of 32 units, and CW of 32 rays -- all of the tile's where there
    // are as many of the units' blocks as waves, so that a weight is loaded by one wave only: the
    // texture addresser is 74 % busy, a third of it with weights (width 128, the loads of an
    // absent batch's zeros left out too, us: 1,048,576 FP16 rays 461 -> 421, 262,144 float32 275 -> 258).
    constexpr bool all = MB >= NW;
    constexpr int CW = all ? NB : 1;
    static_assert(MB <= NW && MB * NB <= NW * CW, "every output block has a wave");
    constexpr uint32_t kCols = 32u * NB;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slot0 = tile * R;
    const uint32_t li = lane & 31u, lq = lane >> 5;
    const uint32_t nb = all ? 0u : wave % NB, m0 = all ? wave : wave / NB;
    const bool mma_wave = m0 < (uint32_t)MB;

    // ---- rays
    uint32_t r = 0, pair = 0xffffffffu;
    bool live = false;
    VRay w;
    int count = 0;
    if (tid < (uint32_t)NB) S.most[tid] = 0u;
    __syncthreads();
    if (tid < (uint32_t)R) {
        slot_ray<PAIRS>(A, g, slot0 + tid, r, pair, live, w);
        const uint32_t nv = live ? A.nvox[slot0 + tid] : 0u;
        count = 2 * (int)nv;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            S.ray[a][tid] = w.o[a];
            S.ray[3 + a][tid] = w.d[a];
            S.ray[6 + a][tid] = w.inv[a];
        }
        S.mov[tid] = (uint8_t)w.mov;
        S.nvox[tid] = (uint8_t)nv;
        atomicMax(&S.most[tid >> 5], nv);
    }
    __syncthreads();
    uint32_t most = S.most[0];
#pragma unroll
    for (int b = 1; b < NB; ++b) most = max(most, S.most[b]);
    most = __builtin_amdgcn_readfirstlane(most);
    const uint32_t my_most = all ? most : __builtin_amdgcn_readfirstlane(S.most[nb]);

    // ---- LDS: features of the points of `vox` voxels per ray and a zero point, the points, their slots
    const uint32_t pb = point_bytes<TM, F>(g.L), nbat = level_batches<TM, F>(g.L);
    const uint32_t vox = min(most, (lds_bytes - pb - 64u) / (2u * R * (pb + 18u)));
    const uint32_t zero = 2u * R * vox;
    float4 *pts = reinterpret_cast<float4 *>(lds + (zero + 1u) * pb);
    uint16_t *smap = reinterpret_cast<uint16_t *>(pts + zero);
    const uint32_t *__restrict__ Wv = reinterpret_cast<const uint32_t *>(mm.W);
    const float *__restrict__ Wf = reinterpret_cast<const float *>(mm.W);
    const int LF = g.L * F;
    const uint32_t half = pb / 8u;   // float: features of each parity
    // swizzle of a point's 16-byte units, so that points side by side use different banks
    const uint32_t units = pb / P::UB;
    const bool pow2 = (units & (units - 1u)) == 0u && units <= 16u && P::UB == 16u;
    const uint32_t swz = pow2 ? units - 1u : 0u, sws = (uint32_t)__builtin_ctz(16u / (pow2 ? units : 16u));
    auto unit_at = [&](uint32_t s, uint32_t u) { return lds + s * pb + ((u ^ ((s >> sws) & swz)) * P::UB); };
    auto feature_at = [&](uint32_t s, uint32_t k) -> float {   // feature k of point s, as stored
        if constexpr (f32) {
            const uint32_t x = k / 2u + (k & 1u) * half;
            return reinterpret_cast<const float *>(lds + s * pb)[(((x >> 2) ^ ((s >> sws) & swz)) << 2) | (x & 3u)];
        } else {
            const uint32_t ks = k / F * P::FP + k % F;
            const uint32_t *d = reinterpret_cast<const uint32_t *>(unit_at(s, ks >> 3));
            if constexpr (DW == 4) {
                const uint32_t x = d[(ks & 7u) >> 1];
                return (ks & 1u) ? hi16<TM>(x) : lo16<TM>(x);
            } else {
                return __builtin_amdgcn_cvt_f32_fp8((int)(d[(ks & 7u) >> 2] >> (8u * (ks & 3u))), 0);
            }
        }
    };

    f16_t acc[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[c][e] = 0.0f;
    float amax = 0.0f;

    if (most > 0u) {
        for (uint32_t i = tid; i < pb / 4u; i += NT) reinterpret_cast<uint32_t *>(lds + zero * pb)[i] = 0u;
        if constexpr (!f32) {
            if (nbat & 1u)   // the last unit holds no level
                for (uint32_t s = tid; s < zero; s += NT) {
                    uint32_t *d = reinterpret_cast<uint32_t *>(unit_at(s, nbat));
#pragma unroll
                    for (int q = 0; q < DW; ++q) d[q] = 0u;
                }
        }
    }
    for (uint32_t j0 = 0; j0 < most; j0 += vox) {
        const uint32_t nj = min(vox, most - j0);
        // ---- points of voxels j0 .. j0 + nj - 1: the distinct ones, packed
        pack_points<R>(A, slot0, j0, nj, zero, S, pts, smap);
        // whether some first-layer weight is not finite; training moves those of FP32 on the device
        uint32_t odd = mm.odd;
        if constexpr (f32) odd = *(cword *)mm.odd_at;   // through the scalar path, needed after the features
        // ---- features: a wave takes 64 points and one batch of levels at a time
        const uint32_t npts = __builtin_amdgcn_readfirstlane(S.npts);
        const uint32_t tasks = (npts + 63u) / 64u * nbat;
        for (uint32_t t = wave; t < tasks; t += NW) {
            const uint32_t grp = t / nbat, b = t - grp * nbat;
            const uint32_t s = grp * 64u + lane;
            if (s < npts) {
                const float4 p4 = pts[s];
                const float p[3] = {p4.x, p4.y, p4.z};
                const int l0 = (int)(b * P::NLB);
                float v[P::NLB][F];
                bool aligned = false;
                if constexpr (F == 3) {
                    const uint32_t all = ((1u << P::NLB) - 1u) & ((uint32_t)(2u << (g.L - 1 - l0)) - 1u);
                    aligned = (~(g.aligned_mask >> l0) & all) == 0u;
                }
                // two ways to the rounding (F = 3): see fma_f16
                constexpr bool H16 = F == 3 && __is_same(TM, _Float16);
                if (aligned) encode_aligned<TF, F, P::NLB, H16>(g, tab, l0, p, __float_as_int(p4.w), v);
                else encode_levels<TF, F, P::NLB, H16>(g, tab, l0, p, __float_as_int(p4.w), v);
                if constexpr (f32) {
                    float *d = reinterpret_cast<float *>(lds + s * pb);
#pragma unroll
                    for (int k = 0; k < P::NLB * F; ++k) {
                        const uint32_t x = b * (P::NLB * F / 2) + k / 2 + (k & 1) * half;   // unit x / 4
                        const float y = v[k / F][k % F];
                        amax = fmax2(amax, __builtin_fabsf(y));
                        d[(((x >> 2) ^ ((s >> sws) & swz)) << 2) | (x & 3u)] = y;
                    }
                } else {
                    float e[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) e[k] = k % P::FP < F ? v[k / P::FP][k % P::FP < F ? k % P::FP : 0] : 0.0f;
                    uint32_t d[DW];
                    pack8<TM>(e, mm.qs[0], d);
                    uint32_t *dst = reinterpret_cast<uint32_t *>(unit_at(s, b));
                    if constexpr (DW == 4) *reinterpret_cast<uint4 *>(dst) = make_uint4(d[0], d[1], d[2], d[3]);
                    else *reinterpret_cast<uint2 *>(dst) = make_uint2(d[0], d[1]);
                }
            }
        }
        __syncthreads();
        if (!PAIRS && A.dbg.enc) {
            for (uint32_t i = tid; i < 2u * nj * R; i += NT) {
                const uint32_t ray = i % R, hh = i / R, h = 2u * j0 + hh, rr = slot0 + ray;
                if (h >= 2u * S.nvox[ray]) continue;
                uint32_t s = smap[i];
                if (s == kSameSlot) s = smap[i - R];
                const uint32_t dst = A.order ? A.order[rr] : rr;
                for (int k = 0; k < LF; ++k) {
                    float v = feature_at(s, (uint32_t)k);
                    if constexpr (!f32 && DW == 2) v /= mm.qs[0];
                    A.dbg.enc[((size_t)dst * g.H + h) * LF + k] = v;
                }
            }
        }
        // ---- first layer: this wave's output blocks of its 32 rays
        if (mma_wave && my_most > j0) {
            const uint32_t nh = 2u * (min(my_most, j0 + nj) - j0);
            const uint16_t *sm[CW];
            uint32_t at[CW];
            bool none[CW];
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const uint32_t col = (nb + c) * 32u + li;
                none[c] = col >= (uint32_t)R;
                sm[c] = smap + (none[c] ? 0u : col);
                at[c] = zero;
            }
            auto next_point = [&](uint32_t hh) {
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const uint32_t ns = none[c] ? zero : sm[c][hh * R];
                    at[c] = ns == kSameSlot ? at[c] : ns;
                }
            };
            if constexpr (f32) {
                const uint32_t steps4 = ((uint32_t)LF + 7u) / 8u;   // groups of 4 matrix-core steps
                const uint32_t nx = nh * steps4;
                const float *Wk = Wf + mm.off[0] + (size_t)(2u * j0) * LF * WIDTH + 32u * m0 + li;
                // A small launch's few waves wait for every weight: two groups' are requested ahead
                // (4,096 rays at 8 levels 33 -> 31 us with the registers below; no gain with more waves).
                constexpr bool ahead = R == 16;
                constexpr int D = ahead ? 2 : 1;
                float nxt[D][4];
                uint32_t ru = 0;
                auto request = [&]() {   // the next D groups (one past the last is in the next layer's weights)
#pragma unroll
                    for (int g4 = 0; g4 < D; ++g4) {
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const uint32_t k = 8u * ru + 2u * t + lq;
                            nxt[g4][t] = k < (uint32_t)LF ? Wk[k * WIDTH] : 0.0f;
                        }
                        if (++ru == steps4) {
                            ru = 0;
                            Wk += LF * WIDTH;
                        }
                    }
                };
                if (ahead) request();
                uint32_t hh = 0, u = 0;
                for (uint32_t x0 = 0; x0 < nx; x0 += D) {
                    if (!ahead) request();
                    float a[D][4];
#pragma unroll
                    for (int g4 = 0; g4 < D; ++g4)
#pragma unroll
                        for (int t = 0; t < 4; ++t) a[g4][t] = nxt[g4][t];
                    if (__builtin_expect(odd != 0u, 0)) {   // made finite, see below
#pragma unroll
                        for (int g4 = 0; g4 < D; ++g4)
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                a[g4][t] = __builtin_amdgcn_fmed3f(a[g4][t], -3.402823466e38f, 3.402823466e38f);
                    }
                    if (ahead && x0 + D < nx) request();
#pragma unroll
                    for (int g4 = 0; g4 < D; ++g4) {
                        if (x0 + g4 >= nx) break;
                        if (u == 0) next_point(hh);
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            const uint32_t s = at[c];
                            const float4 bv = *reinterpret_cast<const float4 *>(
                                lds + s * pb + (((u + lq * (half >> 2)) ^ ((s >> sws) & swz)) << 4));
                            const float b4[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                if (8u * u + 2u * t < (uint32_t)LF)
                                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[g4][t], b4[t], acc[c], 0, 0, 0);
                        }
                        if (++u == steps4) {
                            u = 0;
                            ++hh;
                        }
                    }
                }
            } else {
                typedef typename MmaT<TM>::vec vec_t;
                const int KB = mm.kb_point;
                const uint32_t *Wk = Wv + mm.woff[0] + ((size_t)(2u * j0) * KB * MB + m0) * 64u * DW + lane * DW;
                const uint32_t nx = nh * (uint32_t)KB;
                const bool pad = nbat == 1u && lq != 0u;   // these lanes' weights are the zeros of an absent batch
                constexpr int D = 4;   // fragments requested ahead
                uint32_t nxt[D][DW] = {};
                auto request = [&](uint32_t x0) {
                    if (pad) return;
#pragma unroll
                    for (int t = 0; t < D; ++t) load_frag<DW>(Wk + (size_t)min(x0 + t, nx - 1u) * MB * 64u * DW, nxt[t]);
                };
                request(0);
                uint32_t hh = 0, kb = 0;
                for (uint32_t x0 = 0; x0 < nx; x0 += D) {
                    uint32_t cur[D][DW];
#pragma unroll
                    for (int t = 0; t < D; ++t)
#pragma unroll
                        for (int q = 0; q < DW; ++q) cur[t][q] = nxt[t][q];
                    if (x0 + D < nx) request(x0 + D);
#pragma unroll
                    for (int t = 0; t < D; ++t) {
                        if (x0 + t < nx) {
                            if (kb == 0) next_point(hh);
#pragma unroll
                            for (int c = 0; c < CW; ++c) {
                                uint32_t bd[DW];
                                __builtin_memcpy(bd, __builtin_assume_aligned(unit_at(at[c], 2u * kb + lq), 4 * DW), 4 * DW);
                                acc[c] = MmaT<TM>::mma(as_vec<vec_t, DW>(cur[t]), as_vec<vec_t, DW>(bd), acc[c]);
                            }
                            if (++kb == (uint32_t)KB) {
                                kb = 0;
                                ++hh;
                            }
                        }
                    }
                }
            }
            // Rays whose points have run out took the zero point, and 0 times a weight that is not finite
            // is not 0: the weights above are finite, and where the object has others (rarely),
            // the rays' own points meet those here.
            if (__builtin_expect(odd != 0u, 0)) {
                uint32_t q4 = 4u * lq;
                asm volatile("" : "+v"(q4));   // nothing of this is kept in registers for the common way
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const float *Wo = mm.odd_w + (size_t)(2u * j0) * LF * WIDTH + 32u * m0 + q4;
                    const uint32_t col = (nb + c) * 32u + li;
                    uint32_t s = zero;
#pragma unroll 1
                    for (uint32_t i = 0; i < nh * (uint32_t)LF; ++i, Wo += WIDTH) {
                        const uint32_t hh = i / (uint32_t)LF, k = i - hh * (uint32_t)LF;
                        const uint32_t ns = col < (uint32_t)R ? smap[hh * R + col] : zero;
                        s = ns == kSameSlot ? s : ns;
                        const float x = feature_at(s, k);
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            if (__builtin_amdgcn_ballot_w64(inf_or_nan(Wo[8 * (e / 4) + e % 4])) == 0ull) continue;
                            const float w = Wo[8 * (e / 4) + e % 4];
                            acc[c][e] = inf_or_nan(w) && s != zero ? __builtin_fmaf(x, w, acc[c][e]) : acc[c][e];
                            asm volatile("" ::: "memory");
                        }
                    }
                }
            }
        }
        __syncthreads();
    }

    // ---- hidden layers 2..n_hidden, then the head; activations pass through LDS
    float *outs = reinterpret_cast<float *>(lds + exchange_bytes<TM, WIDTH, R>() - kCols * (kMaxOut + 1) * 4u);
    constexpr uint32_t XS = WIDTH + 4;   // floats of a ray's activations (float)
    if (A.dbg.act_amax) fold_max(A.dbg.act_amax + 0, amax);
    if (most > 0u) {
        for (int k = 1; k <= mm.n_hidden; ++k) {
            const bool head = k == mm.n_hidden;
            if (mma_wave) {
                if constexpr (f32) {
                    amax = 0.0f;
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        float *X = reinterpret_cast<float *>(lds) + ((nb + c) * 32u + li) * XS;
#pragma unroll
                        for (int e = 0; e < 16; e += 4) {
                            float x[4];
#pragma unroll
                            for (int t = 0; t < 4; ++t) {
                                x[t] = act_f(acc[c][e + t], mm.act, mm.slope);
                                amax = fmax2(amax, __builtin_fabsf(x[t]));
                            }
                            const uint32_t at = 16u * m0 + e + 2u * lq;   // (unit 32 m + 2 e + 4 q) / 2
                            *reinterpret_cast<float2 *>(X + at) = make_float2(x[0], x[2]);
                            *reinterpret_cast<float2 *>(X + WIDTH / 2 + at) = make_float2(x[1], x[3]);
                        }
                    }
                    if (A.dbg.act_amax) fold_max(A.dbg.act_amax + k, amax);
                } else {
                    const float dqi = mm.dq[k - 1], qsi = mm.qs[k];
#pragma unroll
                    for (int c = 0; c < CW; ++c)
#pragma unroll
                        for (int s2 = 0; s2 < 2; ++s2) {
                            float v[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float y = MmaT<TM>::scaled ? acc[c][8 * s2 + e] * dqi : acc[c][8 * s2 + e];
                                v[e] = act_f(y, mm.act, mm.slope);
                            }
                            uint32_t d[DW];
                            pack8<TM>(v, qsi, d);
                            uint32_t *dst = reinterpret_cast<uint32_t *>(lds) +
                                            ((((nb + c) * MB + m0) * 2u + s2) * 64u + lane) * DW;
#pragma unroll
                            for (int q = 0; q < DW; ++q) dst[q] = d[q];
                        }
                }
            }
#pragma unroll
            for (int c = 0; c < CW; ++c)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[c][e] = 0.0f;
            __syncthreads();
            if constexpr (f32) {
                if (!head && mma_wave) {
                    const float *X = reinterpret_cast<const float *>(lds) + (nb * 32u + li) * XS + lq * (WIDTH / 2);
                    const float *Wk = Wf + mm.off[k] + lq * WIDTH + 32u * m0 + li;
#pragma unroll 2
                    for (uint32_t u = 0; u < WIDTH / 8; ++u) {
                        float a[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) a[t] = Wk[(8u * u + 2u * t) * WIDTH];
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            const float4 bv = *reinterpret_cast<const float4 *>(X + c * 32u * XS + 4u * u);
                            const float b4[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b4[t], acc[c], 0, 0, 0);
                        }
                    }
                } else if (head) {
                    // 16 outputs of 16 rays at a time: v_mfma_f32_16x16x4f32, the same ascending chain
                    typedef float f4_t __attribute__((ext_vector_type(4)));
                    const uint32_t i16 = lane & 15u, q4 = lane >> 4;
                    const float *Wk = Wf + mm.off[k] + q4 * kMaxOut + i16;
                    for (uint32_t c0 = wave * 16u; c0 < kCols; c0 += 16u * NW) {
                        const float *X = reinterpret_cast<const float *>(lds) + (c0 + i16) * XS +
                                         (q4 & 1u) * (WIDTH / 2) + (q4 >> 1);
                        f4_t o4 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
                        for (uint32_t u = 0; u < WIDTH / 4; ++u)
                            o4 = __builtin_amdgcn_mfma_f32_16x16x4f32(Wk[4u * u * kMaxOut], X[2u * u], o4, 0, 0, 0);
#pragma unroll
                        for (int t = 0; t < 4; ++t) outs[(c0 + i16) * (kMaxOut + 1) + 4u * q4 + t] = o4[t];
                    }
                }
            } else {
                typedef typename MmaT<TM>::vec vec_t;
                const uint32_t *Wk = Wv + mm.woff[k] + (size_t)lane * DW;
                const uint32_t *X = reinterpret_cast<const uint32_t *>(lds) + (size_t)lane * DW;
                if (!head && mma_wave) {
#pragma unroll
                    for (int x = 0; x < 2 * MB; ++x) {
                        uint32_t wd[DW];
                        load_frag<DW>(Wk + (size_t)(m0 * MB * 2 + x) * 64 * DW, wd);
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            uint32_t xd[DW];
                            load_frag<DW>(X + (size_t)((nb + c) * MB * 2 + x) * 64 * DW, xd);
                            acc[c] = MmaT<TM>::mma(as_vec<vec_t, DW>(wd), as_vec<vec_t, DW>(xd), acc[c]);
                        }
                    }
                } else if (head && wave < (uint32_t)NB) {   // 32 rays to a wave
#pragma unroll
                    for (int x = 0; x < 2 * MB; ++x) {
                        uint32_t wd[DW], xd[DW];
                        load_frag<DW>(Wk + (size_t)x * 64 * DW, wd);
                        load_frag<DW>(X + (size_t)(wave * MB * 2 + x) * 64 * DW, xd);
                        acc[0] = MmaT<TM>::mma(as_vec<vec_t, DW>(wd), as_vec<vec_t, DW>(xd), acc[0]);
                    }
                    const float dqo = MmaT<TM>::scaled ? mm.dq[mm.n_hidden] : 1.0f;
                    float *o = outs + (wave * 32u + li) * (kMaxOut + 1) + 4u * lq;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[8 * (e / 4) + e % 4] = acc[0][e] * dqo;
                }
            }
            __syncthreads();
        }
    }
    if (tid >= (uint32_t)R || !live) return;
    float o[kMaxOut];
#pragma unroll
    for (int k = 0; k < kMaxOut; ++k) o[k] = most > 0u ? outs[tid * (kMaxOut + 1) + k] : 0.0f;
    if (A.dbg.count) A.dbg.count[r] = w.valid ? count : -1;
    if (A.dbg.tatb) {
        A.dbg.tatb[2 * r] = w.ta;
        A.dbg.tatb[2 * r + 1] = w.tb;
    }
    if (A.dbg.out) {
#pragma unroll
        for (int k = 0; k < kMaxOut; ++k)
            if (k < mm.out_dim) A.dbg.out[(size_t)r * mm.out_dim + k] = count > 0 ? o[k] : 0.0f;
    }
    decode_store<PAIRS>(A, mm, r, pair, w, count, o);
}

// Waves per SIMD that the registers leave room for.  float32 features of 2 need 145 registers;
// held to 128 they spill, which costs large launches less than a fourth block gives
// (524,288 rays 1,311 us for 1,362) and small ones 2 us.
template <typename TF, int F, int R> constexpr int query_waves() { return sizeof(TF) == 4 && F == 2 && R == 16 ? 3 : 4; }
template <typename TF, typename TM, int F, int WIDTH, bool PAIRS, int R>
__global__ __launch_bounds__(kBlock, (query_waves<TF, F, R>())) void k_query(QueryArgs A, uint32_t lds_bytes)
{
    extern __shared__ __attribute__((aligned(16))) char s_dyn[];
    __shared__ QueryShared<R> S;
    const uint32_t tile = block_subtile<R>(A.tile0);
    if constexpr (PAIRS) {
        const int o = tile_object(A.pr, tile / (kBlock / R));
        if (o < 0) return;
        const cObjDev &O = ((const cObjDev *)A.pr.objs)[o];
        query_body<TF, TM, F, WIDTH, true, R>(A, O.g, O.m, (const TF *)O.tables, S, s_dyn, lds_bytes, tile);
    } else {
        query_body<TF, TM, F, WIDTH, false, R>(A, A.g, A.m, reinterpret_cast<const TF *>(A.tables), S, s_dyn, lds_bytes,
                                              tile);
    }
}

// LDS of a block: four blocks share a CU's 160 KiB, as many as the registers of most variants
// allow.  More voxels per pass leave fewer, fuller groups of points but fewer blocks (2,097,152
// FP16 rays at 31, 42, 53 and 94 KiB: 1.71, 1.80, 2.09 and 3.12 ms).
constexpr uint32_t kQueryLds = 37u << 10;

template <typename TF, typename TM, int F, int WIDTH, int R>
inline void query_go(QueryArgs A, int max_L, bool pairs, uint32_t grid, hipStream_t s)
{
    uint32_t vox = (uint32_t)A.g.H / 2u;
    while (vox > 1u && query_lds_bytes<TM, F, WIDTH, R>(max_L, vox) > kQueryLds) --vox;
    const uint32_t lds = query_lds_bytes<TM, F, WIDTH, R>(max_L, vox);
    // with R = 64 four threads to a slot: from 2^30 slots on more than one launch
    for (uint32_t left = grid, most = tiles_per_launch(kBlock / R * kBlock); left;) {
        const uint32_t now = left < most ? left : most;
        const dim3 blocks(now * (kBlock / R));
        if (pairs) hipLaunchKernelGGL((k_query<TF, TM, F, WIDTH, true, R>), blocks, dim3(kBlock), lds, s, A, lds);
        else hipLaunchKernelGGL((k_query<TF, TM, F, WIDTH, false, R>), blocks, dim3(kBlock), lds, s, A, lds);
        A.tile0 += now;
        left -= now;
    }
}

// Rays per block by the launch's slots n.  Fewer rays give more blocks, which fills the chip
// and shortens the last ones; more rays leave fewer lanes idle in the last group of a batch
// and read the first layer's weights less often.  Measured (us for 16 / 32 / 64 rays):
// 256 rays 20 / 27 / 36, 6,000 42 / 43 / 65, 39,999 102 / 115 / 133, 600,000 826 / 750 / 807,
// 2,097,152 2,250 / 1,887 / 1,706 (16 levels, FP16); 60,000 rays with 8 levels of 64 KiB
// 72 / 55 / 50; 60,000 and 524,288 in float32 356 / 297 / 329 and 1,934 / 1,338 / 1,236.
inline int rays_per_block(uint32_t n, uint32_t batches, bool f32)
{
    const uint32_t mid = batches <= 2u ? 32768u : (f32 ? 393216u : 786432u);
    return n <= 8192u ? 16 : (n <= mid ? 32 : 64);
}

template <typename TF, typename TM, int F, int WIDTH>
inline void query_rays(const QueryArgs &A, int max_L, bool pairs, uint32_t grid, hipStream_t s)
{
    const int R = rays_per_block(grid * kBlock, level_batches<TM, F>(max_L), PointT<TM, F>::f32);
    if (R == 16) query_go<TF, TM, F, WIDTH, 16>(A, max_L, pairs, grid, s);
    else if (R == 32) query_go<TF, TM, F, WIDTH, 32>(A, max_L, pairs, grid, s);
    else query_go<TF, TM, F, WIDTH, 64>(A, max_L, pairs, grid, s);
}

template <typename TF, typename TM, int F>
inline void query_shape(const QueryArgs &A, int max_L, bool pairs, uint32_t grid, hipStream_t s)
{
    if (A.width == 128) query_rays<TF, TM, F, 128>(A, max_L, pairs, grid, s);
    else query_rays<TF, TM, F, 64>(A, max_L, pairs, grid, s);
}

template <typename TM>
inline hipError_t launch_query(const QueryArgs &A, int feat_dtype, int F, int max_L, bool pairs, uint32_t grid,
                              hipStream_t s)
{
    if (feat_dtype == LSNIF_FP32) {
        if (F == 2) query_shape<float, TM, 2>(A, max_L, pairs, grid, s); else query_shape<float, TM, 3>(A, max_L, pairs, grid, s);
    } else if (feat_dtype == LSNIF_FP16) {
        if (F == 2) query_shape<_Float16, TM, 2>(A, max_L, pairs, grid, s); else query_shape<_Float16, TM, 3>(A, max_L, pairs, grid, s);
    } else {
        if (F == 2) query_shape<__bf16, TM, 2>(A, max_L, pairs, grid, s); else query_shape<__bf16, TM, 3>(A, max_L, pairs, grid, s);
    }
    return hipGetLastError();
}

}  // namespace lsnif
