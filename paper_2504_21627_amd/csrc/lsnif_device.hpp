// Device-side steps of an LSNIF query: ray setup, AABB slab test, the voxel
// walk, boundary points and grid-vertex slots (paper Sec. 3.1, 3.2).
//
// Every float32 operation here is written out in the order it is evaluated
// and compiled without contraction into fused multiply-adds, so that the
// voxel list, the points and the table slots are a deterministic function of
// the ray: the same ray gives the same list in every kernel of the library.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lsnif {

constexpr int kMaxLevels = 32;
constexpr int kMaxList = 32;          // H/2 <= 32
constexpr int kCoarseLdsWords = 2048; // brick bits staged in LDS when the grid has <= 65536 bricks
constexpr uint32_t kHotLdsBudget = 40 << 10;  // largest hot_lds_bytes a tuning may name
constexpr uint32_t kTablePad = 16;     // spare bytes after an object's tables (a paired gather may read one entry past the slot it needs)
constexpr uint32_t kPrimeY = 2654435761u;   // spatial hash of Mueller et al. 2022, Eq. 4
constexpr uint32_t kPrimeZ = 805459861u;

// Object geometry and grid description shared by every query kernel.
//
// Occupancy is held as 4x4x4 bricks: `fine` has one 64-bit mask per brick
// (bit (x&3) + 4 (y&3) + 16 (z&3)), brick (x>>2) + NB ((y>>2) + NB (z>>2)),
// and `coarse` one bit per brick telling whether its mask is non-zero.
//
// A level's table slot of vertex v is (vx + my vy + mz vz) & dmask when the
// level is indexed directly (my = R+1, mz = (R+1)^2, dmask = ~0, hmask = 0)
// and (vx ^ my vy ^ mz vz) & hmask when it is hashed (my, mz = the primes,
// dmask = 0, hmask = T-1); the kernels combine both forms without branching.
struct Geom {
    float bmin[3];
    float s[3];               // voxels per object-space unit, (float)V / (bmax - bmin)
    int32_t V;
    int32_t NB;               // bricks per axis, ceil(V / 4)
    const uint64_t *fine;
    const uint32_t *coarse;
    int32_t coarse_words;     // uint32 words of `coarse`
    int32_t L, F, log2_T, H;
    uint32_t dense_mask;      // bit l: level l indexed directly ((R+1)^3 <= T)
    uint32_t aligned_mask;    // bit l: R % V == 0, the crossing-axis weight is 0 or 1
    uint32_t recheck;         // 1: grazing voxels of the walk are re-decided in float64
    uint32_t sort_bits;       // coherence sort of single-object batches: 2^bits cells per axis (0 = no sort, <= 7)
    uint32_t pair_bits;       // grouping of pairs within an object: 2^bits cells per axis (1..6)
    int32_t R[kMaxLevels];
    float lsc[kMaxLevels];    // (float)R / (float)V
    uint32_t my[kMaxLevels], mz[kMaxLevels], dmask[kMaxLevels], hmask[kMaxLevels];
};

// A ray in voxel space with its slab interval.
struct VRay {
    float o[3], d[3], inv[3];
    uint32_t mov;             // bit a: axis a moves (d != 0 with a finite reciprocal)
    float ta, tb, tmax, tmin;
    bool valid, cand;
};

__device__ __forceinline__ float fmin2(float a, float b) { return a < b ? a : b; }
__device__ __forceinline__ float fmax2(float a, float b) { return a > b ? a : b; }

// Parameter where the line crosses the voxel-space plane x_a = k.
__device__ __forceinline__ float plane_t(float k, float o, float inv) { return (k - o) * inv; }

__device__ __forceinline__ bool bad(float x) { return !(x == x); }
__device__ __forceinline__ bool inf_or_nan(float x) { return !(__builtin_fabsf(x) <= 3.402823466e38f); }

// Validity, voxel-space transform and slab test against [0, V]^3.
__device__ __forceinline__ void setup_ray(const Geom &g, float4 r0, float4 r1, VRay &w)
{
    const float in[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
    w.valid = false;
    w.cand = false;
    w.mov = 0;
    w.ta = 0.0f;
    w.tb = 0.0f;
    w.tmax = in[7];
    w.tmin = in[6];
    bool ok = true;
#pragma unroll
    for (int i = 0; i < 6; ++i) ok = ok && !inf_or_nan(in[i]);
    ok = ok && !bad(in[6]) && !bad(in[7]);
    ok = ok && !(in[3] == 0.0f && in[4] == 0.0f && in[5] == 0.0f);
    ok = ok && !(in[6] > in[7]);
    if (!ok) return;
    w.valid = true;
    const float V = (float)g.V;
    float t0 = -__builtin_inff(), t1 = __builtin_inff();
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        w.o[a] = (in[a] - g.bmin[a]) * g.s[a];
        w.d[a] = in[3 + a] * g.s[a];
        w.inv[a] = 0.0f;
        if (w.d[a] != 0.0f) {
            float iv = 1.0f / w.d[a];
            if (__builtin_fabsf(iv) <= 3.402823466e38f) {
                w.mov |= 1u << a;
                w.inv[a] = iv;
            }
        }
        if (w.mov & (1u << a)) {
            float lo = plane_t(0.0f, w.o[a], w.inv[a]);
            float hi = plane_t(V, w.o[a], w.inv[a]);
            t0 = fmax2(t0, fmin2(lo, hi));
            t1 = fmin2(t1, fmax2(lo, hi));
        } else {
            inside = inside && (w.o[a] >= 0.0f && w.o[a] <= V);
        }
    }
    if (!inside || w.mov == 0) return;
    w.ta = fmax2(t0, in[6]);
    w.tb = t1;
    w.cand = w.ta < w.tb;
}

// Entry and exit parameter of cell k along one moving axis.
__device__ __forceinline__ void cell_span(const VRay &w, int a, int k, float &en, float &ex)
{
    float lo = plane_t((float)k, w.o[a], w.inv[a]);
    float hi = plane_t((float)(k + 1), w.o[a], w.inv[a]);
    if (w.d[a] > 0.0f) { en = lo; ex = hi; } else { en = hi; ex = lo; }
}

// Entry/exit of a cell: the latest axis entry and the earliest axis exit over
// moving axes, each tie going to the lowest axis.
__device__ __forceinline__ void cell_interval(const VRay &w, const int c[3], float &tin, float &tout,
                                              int &ia, int &oa)
{
    tin = -__builtin_inff();
    tout = __builtin_inff();
    ia = -1;
    oa = -1;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (w.mov & (1u << a)) {
            float en, ex;
            cell_span(w, a, c[a], en, ex);
            if (ia < 0 || en > tin) { tin = en; ia = a; }
            if (oa < 0 || ex < tout) { tout = ex; oa = a; }
        }
    }
}

__device__ __forceinline__ uint32_t pack_ijk(const int c[3])
{
    return (uint32_t)c[0] | ((uint32_t)c[1] << 10) | ((uint32_t)c[2] << 20);
}
__device__ __forceinline__ void unpack_ijk(uint32_t v, int c[3])
{
    c[0] = (int)(v & 1023u);
    c[1] = (int)((v >> 10) & 1023u);
    c[2] = (int)(v >> 20);
}

__device__ __forceinline__ uint32_t brick_of(const Geom &g, const int c[3])
{
    const uint32_t NB = (uint32_t)g.NB;
    return ((uint32_t)c[0] >> 2) + NB * (((uint32_t)c[1] >> 2) + NB * ((uint32_t)c[2] >> 2));
}

__device__ __forceinline__ uint32_t bit_in_brick(const int c[3])
{
    return ((uint32_t)c[0] & 3u) + 4u * ((uint32_t)c[1] & 3u) + 16u * ((uint32_t)c[2] & 3u);
}

// Start cell of the walk: on a moving axis the cell whose [entry, exit)
// holds ta (a floor guess corrected by at most a few steps), on a still axis
// the half-open cell of the origin with V mapped to V - 1.
__device__ __forceinline__ int start_cell(const Geom &g, const VRay &w, int a)
{
    const int V = g.V;
    if (!(w.mov & (1u << a))) {
        int k = (int)__builtin_floorf(w.o[a]);
        return k > V - 1 ? V - 1 : k;
    }
    float x = w.o[a] + w.ta * w.d[a];
    x = x < 0.0f ? 0.0f : (x > (float)(V - 1) ? (float)(V - 1) : x);
    int k = (int)__builtin_floorf(x);
    const int fwd = w.d[a] > 0.0f ? 1 : -1;
    for (int it = 0; it < V; ++it) {
        float en, ex;
        cell_span(w, a, k, en, ex);
        int nk;
        if (en > w.ta) nk = k - fwd;
        else if (ex <= w.ta) nk = k + fwd;
        else break;
        if (nk < 0 || nk >= V) break;
        k = nk;
    }
    return k;
}

// Optional float64 re-decision of a voxel the float32 walk finds grazing: its
// overlap with [ta, tb] is no longer than 2^-16 max(1, |entry|), or all of
// [ta, tb] is that short.  The slab intervals of the voxel and of the grid are
// recomputed in float64 (IEEE division) from the same float32 voxel-space
// origin and direction, over the axes the float32 walk moves along, and the
// voxel is kept iff the float64 overlap has positive length.  Only whether a
// visited voxel is listed changes; its t values stay float32.
__device__ __forceinline__ bool grazing(float tin, float tout, float ta, float tb)
{
    const float lo = fmax2(tin, ta), hi = fmin2(tout, tb);
    const float q = 0x1p-16f;
    return hi - lo <= q * fmax2(1.0f, __builtin_fabsf(tin)) || tb - ta <= q * fmax2(1.0f, __builtin_fabsf(ta));
}

__device__ __forceinline__ bool keep_f64(const VRay &w, const int c[3], int V)
{
    double t0 = -__builtin_inf(), t1 = __builtin_inf(), tin = -__builtin_inf(), tout = __builtin_inf();
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!(w.mov & (1u << a))) continue;
        const double o = w.o[a], d = w.d[a];
        const double g0 = (0.0 - o) / d, g1 = ((double)V - o) / d;
        const double e0 = ((double)c[a] - o) / d, e1 = ((double)(c[a] + 1) - o) / d;
        t0 = __builtin_fmax(t0, __builtin_fmin(g0, g1));
        t1 = __builtin_fmin(t1, __builtin_fmax(g0, g1));
        tin = __builtin_fmax(tin, __builtin_fmin(e0, e1));
        tout = __builtin_fmin(tout, __builtin_fmax(e0, e1));
    }
    const double ta = __builtin_fmax(t0, (double)w.tmin), tb = t1;
    return __builtin_fmin(tout, tb) > __builtin_fmax(tin, ta);
}

// The next float above a finite x.
__device__ __forceinline__ float next_up(float x)
{
    const int b = (int)__float_as_uint(x);
    return b == (int)0x80000000 ? __uint_as_float(1u) : __uint_as_float((uint32_t)(b >= 0 ? b + 1 : b - 1));
}

// The voxel walk.  Emits, in order along the ray, the packed coordinates of
// the first `cap` occupied voxels whose [entry, exit] overlaps [ta, tb] with
// positive length; list[j * stride] receives voxel j.  Steps the axis of the
// earliest exit, the lowest axis on ties.  Occupancy is read a brick at a
// time: the coarse bit (from `coarse`, LDS or global) and, for a non-empty
// brick, its 64-bit mask, loaded once on entering the brick.  An empty brick
// is crossed in one step; every decision still compares values of the same
// plane functions.
//
// The lanes of a wave are in bricks and cells of their own, so a wave pays for every path that
// some lane takes.  Both steps are therefore the same few instructions (the earliest of three
// planes, then that axis's next one, a cell or a brick further), and the cell at which a brick
// is entered is found only for bricks that hold voxels, without branches: the planes of each
// axis that come before the entry are counted.  One lane per ray (us; finding the entry cell
// of every brick with loops, then this): 1,048,576 rays at V = 32 237 and 150, 2,097,152 at
// V = 128 447 and 226, 262,144 152 and 68, 1,000,003 diffuse ones 231 and 102.  Waiting until
// 2, 4 or 16 lanes have a brick to enter: 241, 270 and 311 where this took 233.
template <bool RECHECK>
__device__ __forceinline__ int walk_voxels(const Geom &g, const VRay &w, const uint32_t *coarse,
                                           uint32_t *list, uint32_t stride, int cap)
{
    if (!w.cand) return 0;
    const int V = g.V;
    // Per axis: cell step (0 on a still axis, whose planes lie at infinity), next plane, where the
    // brick ends; ex: the next plane's t.
    float st[3], kp[3], bx[3], ex[3], o[3], iv[3];
    int sb[3], sl[3];   // steps of the brick's index and of the cell's bit in the brick
    int brick = 0;
    float tin = -__builtin_inff(), tb = w.tb;   // tb: no later than the grid's end, also beside an axis of NaN
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool mov = w.mov & (1u << a), up = w.d[a] > 0.0f;
        const int c = start_cell(g, w, a), pitch = a == 0 ? 1 : (a == 1 ? g.NB : g.NB * g.NB);
        st[a] = mov ? (up ? 1.0f : -1.0f) : 0.0f;
        o[a] = mov ? w.o[a] : -__builtin_inff();
        iv[a] = mov ? w.inv[a] : 1.0f;
        sb[a] = up ? pitch : -pitch;
        sl[a] = (up ? 1 : -1) * (1 << 2 * a);
        brick += (c >> 2) * pitch;
        bx[a] = mov ? (float)((c & ~3) + (up ? 4 : 0)) : (float)(c - 3);   // still: where it would enter at c
        kp[a] = bx[a];
        if (mov) {
            float en, e;
            cell_span(w, a, c, en, e);
            tin = fmax2(tin, en);
            tb = __builtin_fminf(tb, plane_t(up ? (float)V : 0.0f, w.o[a], w.inv[a]));
        }
        ex[a] = plane_t(kp[a], o[a], iv[a]);
    }
    const auto occupied = [&]() { return (coarse[(uint32_t)brick >> 5] >> ((uint32_t)brick & 31u)) & 1u; };
    bool enter = occupied(), cells = false;   // a brick to enter; in a brick, cell by cell
    int n = 0, as = 3, bit = 0;
    float T = w.ta;   // the crossing that led here, along axis `as`
    uint32_t lo32 = 0, hi32 = 0;
    for (;;) {   // a plane at a time, all before tb and so inside the grid
        if (enter) {
            // The cell-by-cell walk merges the axes' crossings in order of t, ties to the lowest
            // axis: it enters the brick after every in-brick plane that comes before (T, as) in
            // that order.
            const uint64_t mask = g.fine[brick];
            lo32 = (uint32_t)mask;
            hi32 = (uint32_t)(mask >> 32);
            bit = 0;
            const float after = next_up(T);   // t <= T is t < after
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const bool up = st[a] > 0.0f;
                const float first = up ? bx[a] - 4.0f : bx[a] + 3.0f, Ta = a < as ? after : T;
                const float p = up ? first + 1.0f : first;   // the entry cell's exit plane
                float k = 0.0f;
#pragma unroll
                for (int j = 0; j < 3; ++j) k += plane_t(p + (float)j * st[a], o[a], iv[a]) < Ta ? st[a] : 0.0f;
                kp[a] = p + k;
                bit |= ((int)(first + k) & 3) << 2 * a;
                ex[a] = plane_t(kp[a], o[a], iv[a]);
            }
            enter = false;
            cells = true;
        }
        // The exit axis is the lowest one whose exit equals the earliest (the axis order of ties).
        const float tout = __builtin_fminf(__builtin_fminf(ex[0], ex[1]), ex[2]);
        if (cells && (((bit & 32 ? hi32 : lo32) >> (bit & 31)) & 1u)) {
            bool keep = fmin2(tout, w.tb) > fmax2(tin, w.ta);
            const int c[3] = {(int)kp[0] - (st[0] > 0.0f), (int)kp[1] - (st[1] > 0.0f), (int)kp[2] - (st[2] > 0.0f)};
            if constexpr (RECHECK)
                if (g.recheck && grazing(tin, tout, w.ta, w.tb)) keep = keep_f64(w, c, V);
            if (keep) {
                list[(size_t)n * stride] = pack_ijk(c);
                if (++n == cap) break;
            }
        }
        if (tout >= tb) break;
        const bool s0 = ex[0] == tout, s1 = !s0 & (ex[1] == tout), s2 = !s0 & !s1;
        const bool left = (s0 & (kp[0] == bx[0])) | (s1 & (kp[1] == bx[1])) | (s2 & (kp[2] == bx[2]));
        tin = tout;
        bit += s0 ? sl[0] : (s1 ? sl[1] : sl[2]);
        kp[0] += s0 ? st[0] : 0.0f;
        kp[1] += s1 ? st[1] : 0.0f;
        kp[2] += s2 ? st[2] : 0.0f;
        if (left) {
            T = tout;
            as = s0 ? 0 : (s1 ? 1 : 2);
            brick += s0 ? sb[0] : (s1 ? sb[1] : sb[2]);
            bx[0] += s0 ? 4.0f * st[0] : 0.0f;
            bx[1] += s1 ? 4.0f * st[1] : 0.0f;
            bx[2] += s2 ? 4.0f * st[2] : 0.0f;
            kp[0] = bx[0];
            kp[1] = bx[1];
            kp[2] = bx[2];
            enter = occupied();
            cells = false;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) ex[a] = plane_t(kp[a], o[a], iv[a]);
    }
    return n;
}

// Planes of axis a that the line has crossed by parameter T, of the `most` inner
// planes it meets in order from cell c0: those with t < T, and with `ties` also
// those with t == T.  A guess from the position at T, corrected by comparing
// plane parameters (non-decreasing along the ray), so the count does not
// depend on the guess.
__device__ __forceinline__ int planes_crossed(const VRay &w, int a, int c0, int most, int V, float T, bool ties)
{
    const bool up = w.d[a] > 0.0f;
    const int st = up ? 1 : -1, first = c0 + (up ? 1 : 0);
    const float x = __builtin_fminf(__builtin_fmaxf(w.o[a] + T * w.d[a], 0.0f), (float)(V - 1));
    int i = ((int)x - c0) * st;
    i = i < 0 ? 0 : (i > most ? most : i);
    auto crossed = [&](int k) {
        const float t = plane_t((float)(first + k * st), w.o[a], w.inv[a]);
        return t < T || (ties && t == T);
    };
    while (i < most && crossed(i)) ++i;
    while (i > 0 && !crossed(i - 1)) --i;
    return i;
}

// The walk by G lanes of a wave together (`lane` = 0..G-1 of them): the voxels
// walk_voxels would list if it had no cap, in any order.  The cell-by-cell walk
// merges the axes' plane crossings in order of t, ties to the lowest axis, so the
// cell it enters at the crossing of plane i of axis a, and that cell's place in
// the walk, follow from counting the other axes' planes crossed before it.  Each
// lane takes one crossing at a time: of any plane, looking at the one cell entered
// (CELLS, the shortest chain), or of a brick boundary, stepping through the cells
// of the brick entered (at most 10) if it holds anything (about half the work).
// A listed voxel is appended to found[]: its place, then its planes crossed on
// axes 0 and 1 (12, 10 and 10 bits; c0 and the signs give the cell back).  *count
// may pass `room`: entries beyond it are dropped.
struct WalkStart {
    int c0[3];
    bool up[3];
};

template <bool RECHECK, int G, bool CELLS>
__device__ __forceinline__ void find_voxels(const Geom &g, const VRay &w, int lane, const uint32_t *coarse,
                                            uint32_t *count, uint32_t *found, uint32_t room, WalkStart &S)
{
    const int V = g.V;
    int n[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        S.c0[a] = start_cell(g, w, a);
        S.up[a] = w.d[a] > 0.0f;
        const int most = (w.mov & (1u << a)) ? (S.up[a] ? V - 1 - S.c0[a] : S.c0[a]) : 0;
        n[a] = most > 0 ? planes_crossed(w, a, S.c0[a], most, V, w.tb, false) : 0;
    }
    // the cell entered after k[] crossings, and without CELLS the rest of its brick
    auto enter = [&](int k0, int k1, int k2) {
        int k[3] = {k0, k1, k2}, c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) c[a] = S.c0[a] + (S.up[a] ? k[a] : -k[a]);
        const uint32_t b = brick_of(g, c);
        if (!CELLS && !((coarse[b >> 5] >> (b & 31u)) & 1u)) return;
        const uint64_t mask = g.fine[b];
        float en[3], ex[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (w.mov & (1u << a)) {
                cell_span(w, a, c[a], en[a], ex[a]);
            } else {
                en[a] = -__builtin_inff();
                ex[a] = __builtin_inff();
            }
        }
        for (int it = 0; it < (CELLS ? 1 : 10); ++it) {
            const float tin = __builtin_fmaxf(__builtin_fmaxf(en[0], en[1]), en[2]);
            const float tout = __builtin_fminf(__builtin_fminf(ex[0], ex[1]), ex[2]);
            bool keep = fmin2(tout, w.tb) > fmax2(tin, w.ta);
            if constexpr (RECHECK)
                if (g.recheck && grazing(tin, tout, w.ta, w.tb)) keep = keep_f64(w, c, V);
            if (keep && ((mask >> bit_in_brick(c)) & 1ull)) {
                const uint32_t at = atomicAdd(count, 1u);
                if (at < room)
                    found[at] = ((uint32_t)(k[0] + k[1] + k[2]) << 20) | ((uint32_t)k[0] << 10) | (uint32_t)k[1];
            }
            if (CELLS || tout >= w.tb) break;
            bool left = false;
            const int oa = ex[0] == tout ? 0 : (ex[1] == tout ? 1 : 2);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (a != oa) continue;
                const int nc = c[a] + (S.up[a] ? 1 : -1);
                left = ((nc ^ c[a]) & ~3) != 0;
                c[a] = nc;
                ++k[a];
                en[a] = ex[a];
                ex[a] = plane_t((float)(nc + (S.up[a] ? 1 : 0)), w.o[a], w.inv[a]);
            }
            if (left) break;
        }
    };
    if (lane == 0) enter(0, 0, 0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // i: planes of the axis before this one; brick boundaries are every fourth plane
        constexpr int every = CELLS ? 1 : 4;
        const int first = CELLS ? 0 : (S.up[a] ? 3 - (S.c0[a] & 3) : S.c0[a] & 3);
        for (int i = first + every * lane; i < n[a]; i += every * G) {
            const float T = plane_t((float)(S.c0[a] + (S.up[a] ? i + 1 : -i)), w.o[a], w.inv[a]);
            int k[3];
#pragma unroll
            for (int b = 0; b < 3; ++b)
                k[b] = b == a ? i + 1 : (n[b] ? planes_crossed(w, b, S.c0[b], n[b], V, T, b < a) : 0);
            enter(k[0], k[1], k[2]);
        }
    }
}

// walk_voxels by one lane, cell by cell: for rays that meet many voxels, whose list
// is full after a few cells, so that entering bricks gains nothing (us, walk_voxels here
// and this: 40,000 rays, 90 % of V = 32 occupied 56 and 53, 30 % of V = 128 147 and 130, 20 %
// of V = 256 248 and 218).
template <bool RECHECK>
__device__ __forceinline__ int walk_cells(const Geom &g, const VRay &w, const WalkStart &S, uint32_t *list,
                                          uint32_t stride, int cap)
{
    int c[3] = {S.c0[0], S.c0[1], S.c0[2]}, n = 0;
    float en[3], ex[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (w.mov & (1u << a)) {
            cell_span(w, a, c[a], en[a], ex[a]);
        } else {
            en[a] = -__builtin_inff();
            ex[a] = __builtin_inff();
        }
    }
    for (int it = 0; it < 3 * g.V; ++it) {
        const float tin = __builtin_fmaxf(__builtin_fmaxf(en[0], en[1]), en[2]);
        const float tout = __builtin_fminf(__builtin_fminf(ex[0], ex[1]), ex[2]);
        bool keep = fmin2(tout, w.tb) > fmax2(tin, w.ta);
        if constexpr (RECHECK)
            if (g.recheck && grazing(tin, tout, w.ta, w.tb)) keep = keep_f64(w, c, g.V);
        if (keep && ((g.fine[brick_of(g, c)] >> bit_in_brick(c)) & 1ull)) {
            list[(size_t)n * stride] = pack_ijk(c);
            if (++n == cap) break;
        }
        if (tout >= w.tb) break;
        const int oa = ex[0] == tout ? 0 : (ex[1] == tout ? 1 : 2);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (a != oa) continue;
            c[a] += S.up[a] ? 1 : -1;
            en[a] = ex[a];
            ex[a] = plane_t((float)(c[a] + (S.up[a] ? 1 : 0)), w.o[a], w.inv[a]);
        }
    }
    return n;
}

// Boundary point h of a listed voxel: even h = where the line enters the
// voxel, odd h = where it leaves.  The crossing axis takes the face plane
// itself; other axes are evaluated on the line and clamped into the voxel.
// Also returns the crossing axis.
__device__ __forceinline__ int boundary_point(const VRay &w, uint32_t packed, bool is_exit, float p[3])
{
    int c[3];
    unpack_ijk(packed, c);
    float tin, tout;
    int ia, oa;
    cell_interval(w, c, tin, tout, ia, oa);
    const float t = is_exit ? tout : tin;
    const int face = is_exit ? oa : ia;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const float lo = (float)c[b], hi = (float)(c[b] + 1);
        if (b == face) {
            const bool upper = (w.d[b] > 0.0f) == is_exit;
            p[b] = upper ? hi : lo;
        } else {
            float v = w.o[b] + t * w.d[b];
            p[b] = v < lo ? lo : (v > hi ? hi : v);
        }
    }
    return face;
}

// Cell of level l holding p: base vertex i and fractional weights wt.
__device__ __forceinline__ void level_cell(const Geom &g, int l, const float p[3], uint32_t i[3], float wt[3])
{
    const int R = g.R[l];
    const float Rf = (float)R;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        float x = p[b] * g.lsc[l];
        x = x < 0.0f ? 0.0f : (x > Rf ? Rf : x);
        int k = (int)__builtin_floorf(x);
        k = k > R - 1 ? R - 1 : k;
        i[b] = (uint32_t)k;
        wt[b] = x - (float)k;
    }
}

// Table slot of vertex v on level l.
__device__ __forceinline__ uint32_t vertex_slot(const Geom &g, int l, uint32_t vx, uint32_t vy, uint32_t vz)
{
    const uint32_t y = vy * g.my[l], z = vz * g.mz[l];
    return ((vx + y + z) & g.dmask[l]) | ((vx ^ y ^ z) & g.hmask[l]);
}

}  // namespace lsnif
