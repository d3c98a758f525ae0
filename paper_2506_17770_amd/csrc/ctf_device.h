// ctf_device.h -- device-side building blocks for gfx950 (wave64).
//
// Wave primitives, the per-lane bilinear footprint, the stochastic draw and
// the texel producers shared by every filter kernel.  Compiled with
// -ffp-contract=off: every fused multiply-add below is written explicitly so
// the float32 decisions are the ones the method fixes.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ctf.h"

namespace ctf {

constexpr int kWave = 64;
constexpr int kTile = 8;              // 8x8 pixels per wave
constexpr int kMaxItems = CTF_MAX_ITEMS;
constexpr float kRange = 16777216.0f; // |texel position| < 2^24

// ---------------------------------------------------------------------------
// wave primitives
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Index of this wave in its workgroup, as a wave-uniform (scalar) value so
// that everything derived from it (tile walks, layer loops) stays scalar.
__device__ __forceinline__ int wave_in_block() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// number of set bits of m below this lane (rank of the lane in m)
__device__ __forceinline__ int mbcnt(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int popc64(uint64_t m) { return __popcll(m); }

// Cross-lane LDS hand-off inside one wave: the wave's LDS instructions
// execute in order, so only compiler reordering has to be prevented.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-wide min / max (all 64 lanes must be active): DPP exchanges reduce
// each row of 16 lanes (quad_perm [1,0,3,2], quad_perm [2,3,0,1],
// row_half_mirror, row_mirror), then the four row results are read with
// v_readlane and combined as scalars.  The result is wave-uniform.
template <class Op>
__device__ __forceinline__ int wave_reduce(int v, Op op)
{
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false));
    const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return op(op(r0, r1), op(r2, r3));
}

struct MinOp {
    __device__ __forceinline__ int operator()(int a, int b) const { return a < b ? a : b; }
};
struct MaxOp {
    __device__ __forceinline__ int operator()(int a, int b) const { return a > b ? a : b; }
};

__device__ __forceinline__ int wave_min(int v) { return wave_reduce(v, MinOp()); }
__device__ __forceinline__ int wave_max(int v) { return wave_reduce(v, MaxOp()); }

// ---------------------------------------------------------------------------
// per-lane footprint (Section 3 and the supplement's code listings)
// ---------------------------------------------------------------------------

struct Footprint {
    bool active;   // finite, in-range texel position
    bool magnify;  // both screen-axis footprints span at most one texel
    int x0, y0;    // upper-left texel of the 2x2 footprint
    float s, t;    // position inside the footprint, in [0,1)
};

// No branches: a NaN or infinite u or v leaves fx or fy NaN or infinite, so
// the range test alone decides `active`.  A coordinate out of range is not
// converted: its x0 or y0 is 0 (the conversion would be undefined, and the
// wave-wide tests read every lane's x0 and y0 before they mask them).  The
// other members of an inactive lane are unused values.
__device__ __forceinline__ Footprint footprint(float u, float v, float4 d, float W, float H)
{
    Footprint f;
    const float fx = __builtin_fmaf(u, W, -0.5f);
    const float fy = __builtin_fmaf(v, H, -0.5f);
    const bool inx = __builtin_fabsf(fx) < kRange, iny = __builtin_fabsf(fy) < kRange;
    f.active = inx && iny;
    const float flx = __builtin_floorf(fx), fly = __builtin_floorf(fy);
    f.x0 = (int)(inx ? flx : 0.0f);
    f.y0 = (int)(iny ? fly : 0.0f);
    f.s = fx - flx;
    f.t = fy - fly;
    const float a = d.x * W, b = d.y * H, c = d.z * W, e = d.w * H;
    const float rx2 = __builtin_fmaf(a, a, b * b);
    const float ry2 = __builtin_fmaf(c, c, e * e);
    f.magnify = rx2 <= 1.0f && ry2 <= 1.0f;
    return f;
}

// The footprint with the wave's decisions as lane masks: act (active lanes)
// and A (active and magnifying).  Each mask is an AND of compare results in
// scalar registers.
struct WaveFootprint {
    uint64_t act, A;
    int x0, y0;
    float s, t;
};

__device__ __forceinline__ WaveFootprint wave_footprint(float u, float v, float4 d, float W, float H)
{
    WaveFootprint f;
    const float fx = __builtin_fmaf(u, W, -0.5f);
    const float fy = __builtin_fmaf(v, H, -0.5f);
    const bool inx = __builtin_fabsf(fx) < kRange, iny = __builtin_fabsf(fy) < kRange;
    f.act = ballot(inx) & ballot(iny);
    const float flx = __builtin_floorf(fx), fly = __builtin_floorf(fy);
    f.x0 = (int)(inx ? flx : 0.0f);
    f.y0 = (int)(iny ? fly : 0.0f);
    f.s = fx - flx;
    f.t = fy - fly;
    const float a = d.x * W, b = d.y * H, c = d.z * W, e = d.w * H;
    const float rx2 = __builtin_fmaf(a, a, b * b);
    const float ry2 = __builtin_fmaf(c, c, e * e);
    f.A = f.act & ballot(rx2 <= 1.0f) & ballot(ry2 <= 1.0f);
    return f;
}

// This lane's bit of a wave-uniform mask, as a predicate.
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Bilinear filtering of texels v0 = (x0,y0), v1 = (x0+1,y0), v2 = (x0,y0+1),
// v3 = (x0+1,y0+1) as two lerps in x and one in y, lerp(a, b, s) =
// fma(s, b - a, a): weights (1-s)(1-t), s(1-t), (1-s)t, st, with constants
// reproduced exactly.  One fixed op sequence used by every method, so exact
// filtering gives the same bits whichever lane produced the texels.
__device__ __forceinline__ float lerp1(float a, float b, float s)
{
    return __builtin_fmaf(s, b - a, a);
}

__device__ __forceinline__ float4 bilerp(float s, float t, float4 v0, float4 v1, float4 v2,
                                         float4 v3)
{
    float4 r;
    r.x = lerp1(lerp1(v0.x, v1.x, s), lerp1(v2.x, v3.x, s), t);
    r.y = lerp1(lerp1(v0.y, v1.y, s), lerp1(v2.y, v3.y, s), t);
    r.z = lerp1(lerp1(v0.z, v1.z, s), lerp1(v2.z, v3.z, s), t);
    r.w = lerp1(lerp1(v0.w, v1.w, s), lerp1(v2.w, v3.w, s), t);
    return r;
}

// ---------------------------------------------------------------------------
// one-tap STF draw [Pharr et al. 2024]: texel (x0 + [u1 < s], y0 + [u2 < t])
// ---------------------------------------------------------------------------

// The "pcg" hash of Jarzynski & Olano, "Hash Functions for GPU Rendering"
// (JCGT 2020): an LCG step followed by PCG's RXS-M-XS output permutation.
__device__ __forceinline__ uint32_t pcg_hash(uint32_t v)
{
    const uint32_t state = v * 747796405u + 2891336453u;
    const uint32_t word = ((state >> ((state >> 28u) + 4u)) ^ state) * 277803737u;
    return (word >> 22u) ^ word;
}

// The per-pixel hash chain of the one-tap draws: h1 and h2 choose the texel
// of the footprint (stf_pick); h3 = pcg(h2) is the spare-lane choice of
// fallback C+.
__device__ __forceinline__ void stf_hashes(uint64_t seed, uint32_t layer, int px, int py, uint32_t& h1,
                                           uint32_t& h2)
{
    uint32_t h = pcg_hash(layer ^ (uint32_t)(seed >> 32));
    h = pcg_hash((uint32_t)py ^ h);
    h = pcg_hash((uint32_t)px ^ h);
    h1 = pcg_hash((uint32_t)seed ^ h);
    h2 = pcg_hash(h1);
}

__device__ __forceinline__ int2 stf_pick_h(const Footprint& f, uint32_t h1, uint32_t h2)
{
    const float u1 = (float)(h1 >> 8) * 0x1p-24f;
    const float u2 = (float)(h2 >> 8) * 0x1p-24f;
    return make_int2(f.x0 + (u1 < f.s ? 1 : 0), f.y0 + (u2 < f.t ? 1 : 0));
}

__device__ __forceinline__ int2 stf_pick(const Footprint& f, uint64_t seed, uint32_t layer,
                                         int px, int py)
{
    uint32_t h1, h2;
    stf_hashes(seed, layer, px, py, h1, h2);
    return stf_pick_h(f, h1, h2);
}

// ---------------------------------------------------------------------------
// reconstruction filters (Section 5): 2x2 bilinear or 4x4 bicubic taps
// ---------------------------------------------------------------------------

template <int FILTER>
struct Taps {
    static constexpr int F = FILTER == CTF_FILTER_BILINEAR ? 2 : 4;  // footprint side
    static constexpr int O = F == 4 ? 1 : 0;                         // origin = x0 - O
};

// 1-D tap weights at position x in [0,1), float32, one fixed op order
// (products, then sums left to right, then the constant factor).
template <int FILTER>
__device__ __forceinline__ void taps32(float x, float w[4])
{
    const float x2 = x * x, x3 = x2 * x, om = 1.0f - x;
    if constexpr (FILTER == CTF_FILTER_BSPLINE) {
        const float sixth = (float)(1.0 / 6.0);
        w[0] = ((om * om) * om) * sixth;
        w[1] = ((3.0f * x3 - 6.0f * x2) + 4.0f) * sixth;
        w[2] = (((-3.0f * x3 + 3.0f * x2) + 3.0f * x) + 1.0f) * sixth;
        w[3] = x3 * sixth;
    } else if constexpr (FILTER == CTF_FILTER_CATMULL_ROM) {
        w[0] = ((2.0f * x2 - x3) - x) * 0.5f;
        w[1] = ((3.0f * x3 - 5.0f * x2) + 2.0f) * 0.5f;
        w[2] = ((-3.0f * x3 + 4.0f * x2) + x) * 0.5f;
        w[3] = (x3 - x2) * 0.5f;
    } else {
        w[0] = om;
        w[1] = x;
        w[2] = w[3] = 0.0f;
    }
}

// Cubic one-tap draw along one axis: tap i with probability |w_i| / sum |w|.
// The drawn tap is the number of float32 partial sums (left to right) at or
// below u * sum, so a zero-weight tap is never drawn.
__device__ __forceinline__ int cubic_tap(const float w[4], float u)
{
    const float a0 = __builtin_fabsf(w[0]), a1 = __builtin_fabsf(w[1]);
    const float a2 = __builtin_fabsf(w[2]), a3 = __builtin_fabsf(w[3]);
    const float p1 = a0, p2 = p1 + a1, p3 = p2 + a2, sum = p3 + a3;
    const float thr = u * sum;
    return (thr >= p1) + (thr >= p2) + (thr >= p3);
}

// One-tap draw for any filter (bilinear: stf_pick_h).
template <int FILTER>
__device__ __forceinline__ int2 stf_pick_filter(const Footprint& f, uint32_t h1, uint32_t h2)
{
    if constexpr (FILTER == CTF_FILTER_BILINEAR) {
        return stf_pick_h(f, h1, h2);
    } else {
        float wx[4], wy[4];
        taps32<FILTER>(f.s, wx);
        taps32<FILTER>(f.t, wy);
        return make_int2(f.x0 - 1 + cubic_tap(wx, (float)(h1 >> 8) * 0x1p-24f),
                         f.y0 - 1 + cubic_tap(wy, (float)(h2 >> 8) * 0x1p-24f));
    }
}

// Exact cubic filtering of 16 texels v[4j + i] (tap (i, j)): each row as a
// fused chain in x, then the rows in y.  One fixed op sequence for every
// method, like bilerp for the 2x2 case.
__device__ __forceinline__ float4 row4(const float wx[4], float4 a, float4 b, float4 c, float4 d)
{
    float4 r;
    r.x = __builtin_fmaf(wx[3], d.x, __builtin_fmaf(wx[2], c.x, __builtin_fmaf(wx[1], b.x, wx[0] * a.x)));
    r.y = __builtin_fmaf(wx[3], d.y, __builtin_fmaf(wx[2], c.y, __builtin_fmaf(wx[1], b.y, wx[0] * a.y)));
    r.z = __builtin_fmaf(wx[3], d.z, __builtin_fmaf(wx[2], c.z, __builtin_fmaf(wx[1], b.z, wx[0] * a.z)));
    r.w = __builtin_fmaf(wx[3], d.w, __builtin_fmaf(wx[2], c.w, __builtin_fmaf(wx[1], b.w, wx[0] * a.w)));
    return r;
}

// accumulate row j (weight wyj) into acc: j == 0 starts the chain
__device__ __forceinline__ float4 col_acc(float wyj, float4 r, float4 acc, bool first)
{
    if (first) return make_float4(wyj * r.x, wyj * r.y, wyj * r.z, wyj * r.w);
    return make_float4(__builtin_fmaf(wyj, r.x, acc.x), __builtin_fmaf(wyj, r.y, acc.y),
                       __builtin_fmaf(wyj, r.z, acc.z), __builtin_fmaf(wyj, r.w, acc.w));
}

// 256-bit footprint mask from the mask of footprint corners:
// B = C | C<<1 | C<<16 | C<<17 (words low first; wave-uniform, scalar ops).
__device__ __forceinline__ void footprint_mask(const uint64_t C[4], uint64_t B[4])
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint64_t lo = w > 0 ? C[w - 1] : 0ull;
        B[w] = C[w] | (C[w] << 1) | (lo >> 63) | (C[w] << 16) | (lo >> 48) | (C[w] << 17) | (lo >> 47);
    }
}

// The same for FxF footprints: B = OR over 0 <= dx, dy < F of C << (16 dy + dx)
// (corners of a box inside 16x16 have dx <= 16 - F, so no row wraps).
template <int F>
__device__ __forceinline__ void footprint_mask_f(const uint64_t C[4], uint64_t B[4])
{
    if constexpr (F == 2) {
        footprint_mask(C, B);
    } else {
        uint64_t Hm[4];   // the row spread: C | C<<1 | C<<2 | C<<3
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint64_t lo = w > 0 ? C[w - 1] : 0ull;
            Hm[w] = C[w] | (C[w] << 1) | (lo >> 63) | (C[w] << 2) | (lo >> 62) | (C[w] << 3) | (lo >> 61);
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint64_t lo = w > 0 ? Hm[w - 1] : 0ull;
            B[w] = Hm[w] | (Hm[w] << 16) | (lo >> 48) | (Hm[w] << 32) | (lo >> 32) | (Hm[w] << 48) | (lo >> 16);
        }
    }
}

// Wave-wide inclusive sum (all 64 lanes active): DPP shifts inside the rows
// of 16 lanes, then the row totals broadcast to the rows behind.
__device__ __forceinline__ int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 to rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 to rows 2, 3
    return v;
}

// The distinct texels of a 16x16 window, four positions per lane: lane l
// holds positions 4l..4l+3 (window row l/4, columns 4 (l%4)..+3).  Byte lanes
// and one DPP prefix sum, in place of four byte ballots, 256-bit scalar shifts
// and a rank table filled from them: the List of a 1920x1080 procedural frame
// (32 terms) 52.4 -> 48.5 us; what bounds it is a tile's chain of LDS steps.
struct WindowSet {
    uint32_t set;     // byte q: 1 if position 4l+q is needed by some lane
    uint32_t ranks;   // byte q: number of needed positions before 4l+q (row-major)
    int n;            // needed positions in all
};

// LDS of window_set: 64 words of position bytes behind 16 words that stay
// zero (kWindowPad; the caller clears them once).
constexpr int kWindowPad = 16;
constexpr int kWindowWords = kWindowPad + kWave;

// FxF spread of the corner bytes around word w (rows r, r-1, .. r-F+1): a
// corner sits at column <= 16 - F, so the bytes shifted in from the previous
// word of the same row never cross a row.
template <int F>
__device__ __forceinline__ uint32_t window_spread(const uint32_t* w)
{
    uint32_t cur = 0u, prev = 0u;
#pragma unroll
    for (int r = 0; r < F; ++r) {
        cur |= w[-4 * r];
        prev |= w[-4 * r - 1];
    }
    uint32_t set = cur;
#pragma unroll
    for (int c = 1; c < F; ++c) set |= __builtin_amdgcn_alignbyte(cur, prev, 4 - c);
    return set;
}

// Ranks of a word's four positions: exclusive byte sums inside the word plus
// the lane's base in each byte (a rank is below 256, so no byte carries).
__device__ __forceinline__ uint32_t window_ranks(uint32_t set, uint32_t base)
{
    uint32_t t = (set << 8) + set;
    t = (t << 16) + t;
    return (t << 8) + __builtin_amdgcn_perm(0u, base, 0u);
}

// Each lane of A marks its footprint's corner byte; the distinct texels are
// the FxF spread of the marks, and the ranks one wave-wide sum.  One LDS
// round trip and no mask in scalar registers: the earlier form (four byte
// reads, four ballots, 256-bit scalar shifts, a rank per ballot) took four
// serial LDS round trips and about 130 scalar instructions.
template <int F>
__device__ __forceinline__ WindowSet window_set(uint32_t* words, bool inA, int corner)
{
    uint32_t* const w = words + kWindowPad + lane_id();
    *w = 0u;
    wave_lds_sync();
    if (inA) reinterpret_cast<uint8_t*>(words + kWindowPad)[corner] = 1;
    wave_lds_sync();
    WindowSet S;
    S.set = window_spread<F>(w);
    const int cnt = (int)__builtin_amdgcn_sad_u8(S.set, 0u, 0u);
    const int incl = wave_scan(cnt);
    S.n = __builtin_amdgcn_readlane(incl, 63);
    S.ranks = window_ranks(S.set, (uint32_t)(incl - cnt));
    return S;
}

// The same for the two half-waves' windows (words: two windows of
// kWindowWords, half 0 first): every lane holds four positions of each, and
// both counts go through one sum.
template <int F>
__device__ __forceinline__ void window_set_halves(uint32_t* words, bool inA, int half, int corner, WindowSet S[2])
{
    uint32_t* const w0 = words + kWindowPad + lane_id();
    uint32_t* const w1 = w0 + kWindowWords;
    *w0 = 0u;
    *w1 = 0u;
    wave_lds_sync();
    if (inA) reinterpret_cast<uint8_t*>(words + kWindowPad)[4 * kWindowWords * half + corner] = 1;
    wave_lds_sync();
    S[0].set = window_spread<F>(w0);
    S[1].set = window_spread<F>(w1);
    const int cnt = (int)(__builtin_amdgcn_sad_u8(S[0].set, 0u, 0u) | (__builtin_amdgcn_sad_u8(S[1].set, 0u, 0u) << 16));
    const int incl = wave_scan(cnt);
    const int n = __builtin_amdgcn_readlane(incl, 63);
    S[0].n = n & 0xffff;
    S[1].n = n >> 16;
    S[0].ranks = window_ranks(S[0].set, (uint32_t)((incl - cnt) & 0xffff));
    S[1].ranks = window_ranks(S[1].set, (uint32_t)((incl - cnt) >> 16));
}

// The distinct texels of footprints that do not fit a window (any box size).
// A footprint is F row segments of F texels; the segments are sorted by
// (row, column), and since a row's segments are then met left to right, a
// segment adds min(F, distance to the one before it) texels to the row-major
// list and its own texels are the last F so far.  F |A| keys instead of the
// F^2 |A| texels: for the cubic filters 256 in place of 1024, and shifts in
// place of the divisions of a general stride (a wave of a B-spline List at
// 3840x2160 that took this path ran for over 100 us alone at the frame's end).
template <int F>
struct SegmentScratch {
    uint64_t keys[kWave * F];   // group << 60 | dy << 34 | dx << 8 | id, sorted
    uint16_t ends[kWave * F];   // items up to and including the segment's
};

// Sorts the wave's segments and counts; group: 0 or 1 (two sets, group 0
// first).  Returns the number of distinct texels of both groups, n0 that of
// group 0, and leaves in first[F lane + r] the item (in its group) of the
// first texel of this lane's row r, valid where the group has at most 256.
template <int F>
__device__ __forceinline__ int segment_sort(SegmentScratch<F>& S, uint8_t* first, bool inA, uint32_t group, int ox,
                                            int oy, int xmin, int ymin, int& n0)
{
    constexpr int N = kWave * F;
    const int lane = lane_id();
    const uint32_t dx = (uint32_t)ox - (uint32_t)xmin, dy = (uint32_t)oy - (uint32_t)ymin;   // below 2^26
#pragma unroll 1
    for (int r = 0; r < F; ++r)
        S.keys[F * lane + r] = inA ? ((uint64_t)group << 60) | ((uint64_t)(dy + r) << 34) | ((uint64_t)dx << 8) |
                                         (uint32_t)(F * lane + r)
                                   : ~0ull;
#pragma unroll 1
    for (int size = 2; size <= N; size <<= 1)
#pragma unroll 1
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            wave_lds_sync();
#pragma unroll 1
            for (int p = lane; p < N / 2; p += kWave) {
                const int i = ((p & -stride) << 1) | (p & (stride - 1));
                const uint64_t x = S.keys[i], y = S.keys[i + stride];
                if ((x > y) == ((i & size) == 0)) {
                    S.keys[i] = y;
                    S.keys[i + stride] = x;
                }
            }
        }
    wave_lds_sync();
    // this lane counts segments F lane .. F lane + F - 1
    uint64_t prev = lane ? S.keys[F * lane - 1] : ~0ull;
    int sum = 0, sum0 = 0;
    uint32_t sums = 0;   // byte r: texels of the lane's segments up to r
#pragma unroll
    for (int r = 0; r < F; ++r) {
        const uint64_t k = S.keys[F * lane + r];
        if (k != ~0ull) {
            const uint32_t gap = ((uint32_t)(k >> 8) & 0x3ffffffu) - ((uint32_t)(prev >> 8) & 0x3ffffffu);
            const int c = (k >> 34) == (prev >> 34) && gap < (uint32_t)F ? (int)gap : F;
            sum += c;
            if ((k >> 60) == 0) sum0 += c;
        }
        sums |= (uint32_t)sum << (8 * r);
        prev = k;
    }
    const int incl = wave_scan(sum), base = incl - sum;
    const int n = __builtin_amdgcn_readlane(incl, 63);
    n0 = __builtin_amdgcn_readlane(wave_scan(sum0), 63);
#pragma unroll
    for (int r = 0; r < F; ++r) {
        const uint64_t k = S.keys[F * lane + r];
        const int end = base + (int)((sums >> (8 * r)) & 0xffu);
        S.ends[F * lane + r] = (uint16_t)end;
        if (k != ~0ull) first[k & 0xffu] = (uint8_t)(end - F - ((k >> 60) ? n0 : 0));
    }
    wave_lds_sync();
    return n;
}

// Calls emit(item, group, dx, dy) for every distinct texel (items of both
// groups in one sequence).
template <int F, class Emit>
__device__ __forceinline__ void segment_emit(const SegmentScratch<F>& S, Emit&& emit)
{
    const int lane = lane_id();
#pragma unroll 1
    for (int p = F * lane; p < F * lane + F; ++p) {
        const uint64_t k = S.keys[p];
        if (k == ~0ull) continue;
        const int begin = p ? S.ends[p - 1] : 0, end = S.ends[p];
        const int dx = (int)((uint32_t)(k >> 8) & 0x3ffffffu) + F - end, dy = (int)((uint32_t)(k >> 34) & 0x3ffffffu);
#pragma unroll 1
        for (int i = begin; i < end; ++i) emit(i, (int)(k >> 60), dx + i, dy);
    }
}

// A wave's walk over tiles t0, t0 + step, ... of a row-major tile grid,
// keeping (tx, ty) up to date with scalar adds: one division per wave
// instead of a 64-bit division per tile.
struct TileWalk {
    int64_t tile;
    int tx, ty;
    int dtx, dty, tiles_x;
    __device__ __forceinline__ TileWalk(int64_t t0, int64_t step, int tiles_x_) : tile(t0), tiles_x(tiles_x_)
    {
        tx = (int)(t0 % tiles_x_);
        ty = (int)(t0 / tiles_x_);
        dtx = (int)(step % tiles_x_);
        dty = (int)(step / tiles_x_);
    }
    __device__ __forceinline__ void advance(int64_t step)
    {
        tile += step;
        tx += dtx;
        ty += dty;
        if (tx >= tiles_x) {
            tx -= tiles_x;
            ++ty;
        }
    }
};

// Frame totals of one wave over all its tiles, added to the frame record
// once at the end (one set of atomics per wave).
// Per-wave sums of the frame counters, added to the frame's 64-bit counters
// at the end of the kernel.  32-bit (half the scalar registers): a tile adds
// at most 2^13 to any of them, and every launch gives each wave at most
// kMaxWaveTileVisits tile visits (layers counted once each), so none can
// overflow.
constexpr int64_t kMaxWaveTileVisits = int64_t(1) << 18;

// Workgroups of `waves_per_block` waves a launch needs so that no wave visits
// more than kMaxWaveTileVisits tiles.
inline int64_t counter_min_blocks(int64_t tile_visits, int waves_per_block)
{
    const int64_t waves = (tile_visits + kMaxWaveTileVisits - 1) / kMaxWaveTileVisits;
    return (waves + waves_per_block - 1) / waves_per_block;
}

struct FrameCounters {
    uint32_t evals = 0, active = 0, stf = 0, minify = 0, tiles = 0, rows = 0, ok = 0, fail = 0;
    __device__ __forceinline__ void add(int e, int act, int nstf, int mini, int rws, bool okk, bool fl)
    {
        evals += e;
        active += act;
        stf += nstf;
        minify += mini;
        rows += rws;
        tiles += 1;
        ok += okk;
        fail += fl;
    }
    // Every lane of the wave calls this.  The eight totals of a frame are one
    // 64-byte line, and every wave's atomics wait for it in turn: lanes 0..7 add
    // a total each, one access per wave instead of eight.  With frame totals
    // the List of a 1920x1080 procedural frame takes 138 us instead of 1426
    // (B-spline 132, 1146), that of a 3840x2160 decoder frame 149 instead of 406.
    __device__ __forceinline__ void flush(ctf_frame_stats* F) const
    {
        if (!tiles) return;
        static_assert(offsetof(ctf_frame_stats, active) == 8 && offsetof(ctf_frame_stats, stf) == 16 &&
                          offsetof(ctf_frame_stats, minify) == 24 && offsetof(ctf_frame_stats, tiles) == 32 &&
                          offsetof(ctf_frame_stats, tiles_ok) == 40 && offsetof(ctf_frame_stats, tiles_fail) == 48 &&
                          offsetof(ctf_frame_stats, rows) == 56,
                      "the order of c");
        // (read as scalars, and the lane's index from an opaque mask: otherwise
        // the counters are kept in vector registers for this select, and the
        // index from the kernel's start, and the decoder kernels spill)
        uint32_t c[8] = {evals, active, stf, minify, tiles, ok, fail, rows};
#pragma unroll
        for (int i = 0; i < 8; ++i) c[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)c[i]);
        uint32_t all = ~0u;
        asm volatile("" : "+s"(all));
        const int lane = (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
        uint32_t v = c[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) v = lane == i ? c[i] : v;
        if (lane < 8) atomicAdd(reinterpret_cast<unsigned long long*>(F) + lane, (unsigned long long)v);
    }
};

// ---------------------------------------------------------------------------
// texel producers
// ---------------------------------------------------------------------------

struct DevTexture {
    int kind;
    int width, height;
    uint32_t wmask, hmask;
    float inv_w;
    int n_terms;
    const int4* __restrict__ terms;   // [4][K] = (p, q, j, bits of amp)
    // [4][K] = (p'/W, q'/W, j'/W, amp) with p', q' the residues of p, q mod W
    // in [-W/2, W/2) and j' = j mod W; null when W > 4096
    const float4* __restrict__ fterms;
    float affine[4][3];
    float constant[4];
    const float4* __restrict__ table; // [height][width]
};

// 1/2 + 1/2 sum_k a_k sin(2 pi r_k / W), r_k = (p x + q y + j) mod W.  The
// phase is an exact integer, r/W is exact in float32, and v_sin_f32 takes
// its argument in revolutions, so each term is one hardware sine.
// The term arrays in device memory are read through the constant address
// space: with a wave-uniform address each term is one scalar load
// (s_load_dwordx4 through the scalar cache) instead of a 64-lane broadcast
// vector load and its wait.  Only for global memory that the kernel never
// writes -- LDS-staged terms keep their generic pointer.
typedef int TermVec __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) TermVec* ConstTerms;

__device__ __forceinline__ ConstTerms const_terms(const int4* global_terms)
{
    return (ConstTerms)global_terms;
}

typedef float FTermVec __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) FTermVec* ConstFTerms;

__device__ __forceinline__ ConstFTerms const_fterms(const float4* global_terms)
{
    return (ConstFTerms)global_terms;
}

// The same channel from the float terms: v = p' x + q' y + j' is an integer
// with |v| < W^2 <= 2^24, so both fused products and sums below are exact
// and fract(v / W) is exactly (v mod W) / W, the argument the integer form
// passes to the sine: the results are bit-identical to sinusoid_channel, in
// five instructions per term instead of eight.
template <class TermPtr>
__device__ __forceinline__ float sinusoid_channel_f(TermPtr tc, int K, float xf, float yf)
{
    float acc = 0.0f;
    // eight terms per iteration: their loads are issued together (one wait)
    int k = 0;
    for (; k + 8 <= K; k += 8) {
        decltype(tc[0] + 0) t8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t8[u] = tc[k + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float ph = __builtin_fmaf(t8[u].x, xf, __builtin_fmaf(t8[u].y, yf, t8[u].z));
            const float sn = __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(ph));
            acc = __builtin_fmaf(t8[u].w, sn, acc);
        }
    }
    for (; k < K; ++k) {
        const auto tk = tc[k];
        const float ph = __builtin_fmaf(tk.x, xf, __builtin_fmaf(tk.y, yf, tk.z));
        const float sn = __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(ph));
        acc = __builtin_fmaf(tk.w, sn, acc);
    }
    return __builtin_fmaf(0.5f, acc, 0.5f);
}

// One channel of four texels: columns x and x + 1 of rows y and y + 1, or (ROW)
// columns x .. x + 3 of row y.  The phases of neighbours differ by p' / W and
// q' / W; with W <= 2048 every sum stays below 2^24 units of 1 / W even where a
// neighbour passes the texture's edge, so each phase is exact and its fract is
// that of the wrapped texel: the values are those of sinusoid_channel_f, in 17
// instructions per term instead of 20 and with one read of the term instead of
// four (4-tap at 1920x1080, 32 terms: 154 -> 140 us, bound by the VALU: four
// quarter-rate v_sin and 13 others per term).  Wider textures could round: they
// keep the four evaluations.
constexpr int kJointWidth = 2048;

template <bool ROW, class TermPtr>
__device__ __forceinline__ void sinusoid_channel_4(TermPtr tc, int K, float xf, float yf, float out[4])
{
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto term = [&](decltype(tc[0] + 0) t) __attribute__((always_inline)) {
        float ph[4];
        const float r = __builtin_fmaf(t.y, yf, t.z);
        ph[0] = __builtin_fmaf(t.x, xf, r);
        if constexpr (ROW) {
            ph[1] = ph[0] + t.x;
            ph[2] = ph[1] + t.x;
            ph[3] = ph[2] + t.x;
        } else {
            ph[1] = ph[0] + t.x;
            ph[2] = ph[0] + t.y;
            ph[3] = ph[1] + t.y;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            acc[i] = __builtin_fmaf(t.w, __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(ph[i])), acc[i]);
    };
    int k = 0;
    for (; k + 4 <= K; k += 4) {
        decltype(tc[0] + 0) t4[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t4[u] = tc[k + u];
#pragma unroll
        for (int u = 0; u < 4; ++u) term(t4[u]);
    }
    for (; k < K; ++k) term(tc[k]);
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = __builtin_fmaf(0.5f, acc[i], 0.5f);
}

template <class TermPtr>
__device__ __forceinline__ float sinusoid_channel(TermPtr tc, int K, uint32_t wmask, float inv_w, int xm, int ym)
{
    float acc = 0.0f;
    for (int k = 0; k < K; ++k) {
        const auto tk = tc[k];
        const uint32_t r = (uint32_t)(__mul24(tk.x, xm) + __mul24(tk.y, ym) + tk.z) & wmask;
        const float sn = __builtin_amdgcn_sinf((float)r * inv_w);
        acc = __builtin_fmaf(__int_as_float(tk.w), sn, acc);
    }
    return __builtin_fmaf(0.5f, acc, 0.5f);
}

template <int KIND>
__device__ __forceinline__ float4 texel_eval(const DevTexture& T, int x, int y)
{
    float4 r;
    if constexpr (KIND == CTF_TEX_SINUSOIDS) {
        const int xm = x & (int)T.wmask, ym = y & (int)T.wmask;
        const int K = T.n_terms;
        if (T.fterms) {
            const ConstFTerms tc = const_fterms(T.fterms);
            const float xf = (float)xm, yf = (float)ym;
            r.x = sinusoid_channel_f(tc + 0 * K, K, xf, yf);
            r.y = sinusoid_channel_f(tc + 1 * K, K, xf, yf);
            r.z = sinusoid_channel_f(tc + 2 * K, K, xf, yf);
            r.w = sinusoid_channel_f(tc + 3 * K, K, xf, yf);
        } else {
            const ConstTerms tc = const_terms(T.terms);
            r.x = sinusoid_channel(tc + 0 * K, K, T.wmask, T.inv_w, xm, ym);
            r.y = sinusoid_channel(tc + 1 * K, K, T.wmask, T.inv_w, xm, ym);
            r.z = sinusoid_channel(tc + 2 * K, K, T.wmask, T.inv_w, xm, ym);
            r.w = sinusoid_channel(tc + 3 * K, K, T.wmask, T.inv_w, xm, ym);
        }
    } else if constexpr (KIND == CTF_TEX_AFFINE) {
        const float fx = (float)x, fy = (float)y;
        r.x = __builtin_fmaf(T.affine[0][2], fy, __builtin_fmaf(T.affine[0][1], fx, T.affine[0][0]));
        r.y = __builtin_fmaf(T.affine[1][2], fy, __builtin_fmaf(T.affine[1][1], fx, T.affine[1][0]));
        r.z = __builtin_fmaf(T.affine[2][2], fy, __builtin_fmaf(T.affine[2][1], fx, T.affine[2][0]));
        r.w = __builtin_fmaf(T.affine[3][2], fy, __builtin_fmaf(T.affine[3][1], fx, T.affine[3][0]));
    } else if constexpr (KIND == CTF_TEX_CONSTANT) {
        r = make_float4(T.constant[0], T.constant[1], T.constant[2], T.constant[3]);
    } else {  // CTF_TEX_TABLE
        r = T.table[(size_t)(y & (int)T.hmask) * T.width + (x & (int)T.wmask)];
    }
    return r;
}

// Terms of a sinusoid texture staged in a workgroup's LDS: [4][K + 1] entries
// (each channel's row padded by one entry, so that lanes reading the same
// term of different channels hit different banks), the float terms when the
// texture has them.  Textures with more terms are not staged.  62 terms:
// 4032 bytes, so that a per-lane workgroup (four 7 KiB wave slices and the
// terms) stays within 32 KiB and five of them fit in a CU's 160 KiB.
constexpr int kLdsTerms = 62;
constexpr int kLdsTermEntries = 4 * (kLdsTerms + 1);

// Every thread of the workgroup calls this (it synchronises the workgroup).
__device__ inline bool stage_terms(const DevTexture& T, int4* terms_lds)
{
    if (T.kind != CTF_TEX_SINUSOIDS || T.n_terms > kLdsTerms) return false;
    const int4* src = T.fterms ? reinterpret_cast<const int4*>(T.fterms) : T.terms;
    for (int i = threadIdx.x; i < 4 * T.n_terms; i += blockDim.x) terms_lds[i + i / T.n_terms] = src[i];
    __syncthreads();
    return true;
}

// A texel from staged float terms (every lane reads the same entry, a
// broadcast; the operands are then all vector registers, one instruction
// fewer per term than with terms in scalar registers).  Textures whose
// terms are not staged read them with vector loads: the scalar form would
// hold 32 scalar registers for its eight terms in flight across the whole
// kernel, and the per-lane kernels are short of scalar registers.  The same
// values either way.
template <int KIND>
__device__ __forceinline__ float4 texel_eval_staged(const DevTexture& T, const int4* terms_lds, bool lds_float, int x,
                                                    int y)
{
    if constexpr (KIND == CTF_TEX_SINUSOIDS) {
        const int K = T.n_terms;
        const int xm = x & (int)T.wmask, ym = y & (int)T.wmask;
        const float xf = (float)xm, yf = (float)ym;
        if (lds_float) {
            const float4* tl = reinterpret_cast<const float4*>(terms_lds);
            return make_float4(sinusoid_channel_f(tl + 0 * (K + 1), K, xf, yf),
                               sinusoid_channel_f(tl + 1 * (K + 1), K, xf, yf),
                               sinusoid_channel_f(tl + 2 * (K + 1), K, xf, yf),
                               sinusoid_channel_f(tl + 3 * (K + 1), K, xf, yf));
        }
        // (an offset the compiler cannot prove uniform keeps these loads in
        // vector registers)
        int zero = 0;
        asm volatile("" : "+v"(zero));
        if (T.fterms) {
            const float4* tf = T.fterms + zero;
            return make_float4(sinusoid_channel_f(tf + 0 * K, K, xf, yf), sinusoid_channel_f(tf + 1 * K, K, xf, yf),
                               sinusoid_channel_f(tf + 2 * K, K, xf, yf), sinusoid_channel_f(tf + 3 * K, K, xf, yf));
        }
        const int4* ti = T.terms + zero;
        return make_float4(sinusoid_channel(ti + 0 * K, K, T.wmask, T.inv_w, xm, ym),
                           sinusoid_channel(ti + 1 * K, K, T.wmask, T.inv_w, xm, ym),
                           sinusoid_channel(ti + 2 * K, K, T.wmask, T.inv_w, xm, ym),
                           sinusoid_channel(ti + 3 * K, K, T.wmask, T.inv_w, xm, ym));
    }
    return texel_eval<KIND>(T, x, y);
}

// Whether a workgroup's LDS holds a texture's terms as floats.
__host__ __device__ __forceinline__ bool lds_terms(const DevTexture& T)
{
    return T.kind == CTF_TEX_SINUSOIDS && T.fterms != nullptr && T.n_terms <= kLdsTerms;
}

// Whether sinusoid_channel_4 serves a texture.
__host__ __device__ __forceinline__ bool joint_texels(const DevTexture& T)
{
    return lds_terms(T) && T.width <= kJointWidth;
}

// Texels (x, y), (x+1, y), (x, y+1), (x+1, y+1), or (ROW) (x .. x+3, y), from
// staged float terms.
template <bool ROW>
__device__ __forceinline__ void texel_eval_4(const DevTexture& T, const int4* terms_lds, int x, int y, float4 v[4])
{
    const int K = T.n_terms;
    const float4* tl = reinterpret_cast<const float4*>(terms_lds);
    const float xf = (float)(x & (int)T.wmask), yf = (float)(y & (int)T.wmask);
    float c[4][4];
#pragma unroll
    for (int ch = 0; ch < 4; ++ch) sinusoid_channel_4<ROW>(tl + ch * (K + 1), K, xf, yf, c[ch]);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = make_float4(c[0][i], c[1][i], c[2][i], c[3][i]);
}

// The full filter of a lane: every tap of its footprint (upper-left tap
// ox, oy) through texel(x, y), the four bilinear or each row of cubic taps in
// one evaluation where the texture allows.
template <int FILTER, int TEX, class Texel>
__device__ __forceinline__ float4 full_filter(const DevTexture& T, const int4* terms_lds, bool joint, float s, float t,
                                              int ox, int oy, Texel&& texel)
{
    float4 res;
    float4 v[4];
    if constexpr (FILTER == CTF_FILTER_BILINEAR) {
        if (TEX == CTF_TEX_SINUSOIDS && joint) {
            texel_eval_4<false>(T, terms_lds, ox, oy, v);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = texel(ox + (q & 1), oy + (q >> 1));
        }
        res = bilerp(s, t, v[0], v[1], v[2], v[3]);
    } else {
        float wx[4], wy[4];
        taps32<FILTER>(s, wx);
        taps32<FILTER>(t, wy);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (TEX == CTF_TEX_SINUSOIDS && joint) {
                texel_eval_4<true>(T, terms_lds, ox, oy + j, v);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = texel(ox + i, oy + j);
            }
            res = col_acc(wy[j], row4(wx, v[0], v[1], v[2], v[3]), res, j == 0);
        }
    }
    return res;
}

}  // namespace ctf
