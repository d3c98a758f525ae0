// filter_decoder.h -- collaborative filtering with the learned texel producer.
//
// Same decisions as the per-lane path (Sections 3.1-3.3, remapping, the
// fallbacks of Section 3.4 and the bicubic filters of Section 5), but texel
// production is batched: the wave writes the (x, y) of every texel it must
// produce into an LDS row list (the unique texels first, then one row per
// one-tap draw; in a wave that takes fallback C or C+, the planned texels of
// A, then the minifying lanes' draws) and decodes the rows 16 at a time on
// MFMA (decoder_mlp.h).  Dedup therefore turns the per-tap decode into one
// dense MLP pass over the wave's distinct texels.
//
// Waves are persistent: each loads the MLP weights into registers once and
// takes tiles from its workgroup's share until it is used up (TileQueue).
// Workgroups are dispatched round-robin over the 8 XCDs; XCD x takes every
// eighth strip of two tile rows, so that the latent-grid reads of neighbouring
// tiles share an L2 while every XCD gets a like share of the frame's work.
//
// Instantiated per reconstruction filter (FxF footprints, F = 2 or 4): the
// bilinear kernels in filter_decoder.hip, the bicubic ones in
// filter_decoder_cubic.hip.
#pragma once

#include <stddef.h>

#include <type_traits>

#include "ctf_device.h"
#include "ctf_internal.h"
#include "decoder_mlp.h"
#include "fallback.h"

namespace ctf {

namespace dec {

// Waves of a workgroup: a whole CU's worth (three per SIMD, the occupancy the
// kernels' registers allow) on a large frame, four on a small one
// (dec_waves).  Each wave has a slice of the dynamic LDS behind the queues.
constexpr int kDecWavesMax = 12, kDecWavesMin = 4;

constexpr bool collaborative(int m) { return m == CTF_LIST || m == CTF_BOX || m == CTF_MASK; }

// The launches whose tiles are decoded in batches: every method but the full
// filter, without fallback C / C+ (FB).
template <int METHOD, bool FB>
constexpr bool batched()
{
    return !FB && METHOD != CTF_BILINEAR4;
}

struct DecLds {
    float4 vals[kMaxItems];     // decoded texels, by row; the List's sort before any row is decoded
    int2 rows[kMaxItems];       // texel coordinates to decode
    uint64_t keys[kMaxItems];   // fallback planning
    uint8_t rank[256];          // Mask/List: position t -> row (h^-1); List past 16x16: first item of a lane's rows
    uint8_t bytes[256];         // footprint-corner scatter before the ballots
    __device__ uint8_t* byte_area() { return bytes; }
};

// Rows past R read whatever the row list holds there (the index is kept
// inside the list): the inference fetch maps any texel to cells inside the
// grid, and those rows' results are never stored.
template <int P>
__device__ __forceinline__ void fetch_row(const int2* rows, int row, const InferGrid& G, const InferLane<P>& K,
                                          InferFetch& F)
{
    const int2 p = rows[row & (kMaxItems - 1)];
    infer_fetch<P>(G, K, p.x, p.y, F);
}

template <int P>
__device__ __forceinline__ void finish_row(float4* vals, int R, int row, const FwdWeights<P>& W,
                                           const Biases& Bz, u16x4 x, int g)
{
    const f4 y = mlp_forward_b<P>(W, Bz, x, nullptr, nullptr);
    if (g == 0 && row < R) vals[row] = make_float4(y[0], y[1], y[2], y[3]);
}

// rows[0..R) -> vals[0..R): latents 32 rows at a time, the MLP on 16-row
// tiles (the last 32 rows may hold one).  The next 32 rows' gathers are
// issued, unconditionally, once the current features are interpolated, so
// they are in flight during two MLP passes.
template <int P>
__device__ __forceinline__ void decode_rows(const int2* rows, float4* vals, int R, const InferGrid& G,
                                            const FwdWeights<P>& W, const Biases& Bz)
{
    if (R == 0) return;
    const int j = lane_id() & 15, g = lane_id() >> 4;
    const InferLane<P> K(G, g >= 2);
    const int jf = j + 16 * (g & 1);
    InferFetch F;
    u16x4 xa, xb;
    fetch_row<P>(rows, jf, G, K, F);
    int r0 = 0;
    for (; r0 + 16 < R; r0 += 32) {
        infer_combine<P>(F, K, xa, xb);
        fetch_row<P>(rows, r0 + 32 + jf, G, K, F);
        const f4 ya = mlp_forward_b<P>(W, Bz, xa, nullptr, nullptr);
        const f4 yb = mlp_forward_b<P>(W, Bz, xb, nullptr, nullptr);
        if (g == 0) {
            vals[r0 + j] = make_float4(ya[0], ya[1], ya[2], ya[3]);
            if (r0 + 16 + j < R) vals[r0 + 16 + j] = make_float4(yb[0], yb[1], yb[2], yb[3]);
        }
    }
    // With 16 rows or fewer left the last fetch is theirs.  Otherwise it is
    // never used: wait for it here, while it is nearly done, rather than
    // where its registers are next written, which may be after the next
    // tile's inputs were requested (memory counters drain in order, so that
    // wait would cover them too).
    if (r0 < R) {
        infer_combine<P>(F, K, xa, xb);
        finish_row<P>(vals, R, r0 + j, W, Bz, xa, g);
    } else {
        asm volatile("" ::"v"(F.v[0]), "v"(F.v[1]), "v"(F.v[2]), "v"(F.v[3]));
    }
}

__device__ __forceinline__ void write_tile_stats(const FilterArgs& a, int64_t tile, uint64_t act, uint64_t A,
                                                 uint64_t stfmask, bool fits16, const uint64_t B[4], int xmin,
                                                 int ymin, int bbw, int bbh, int n, int unique, int evals,
                                                 bool success, bool cap_ok, bool count_ok, int nA)
{
    ctf_tile_stats S;
    S.active = act;
    S.part = A;
    S.stf = stfmask;
    for (int w = 0; w < 4; ++w) S.mask[w] = fits16 ? B[w] : 0ull;
    S.xmin = xmin;
    S.ymin = ymin;
    S.bbw = bbw;
    S.bbh = bbh;
    S.n = n;
    S.unique = unique;
    S.evals = evals;
    S.flags = (success ? CTF_TILE_OK : 0) | (nA && !cap_ok ? CTF_TILE_CAP : 0) |
              (nA && cap_ok && !count_ok ? CTF_TILE_OVERFLOW : 0) | (nA == 0 ? CTF_TILE_EMPTY : 0);
    for (int r = 0; r < 10; ++r) S.reserved[r] = 0;
    a.tile_stats[tile] = S;
}

// One tile of the decoder-path filter: decisions, row list, MFMA decode,
// gather and outputs.  `f` is the lanes' footprint (already in this
// layer's coordinates); a.out / a.tile_stats / a.stf_xy point at this
// layer's planes.  `after_decode` runs once, right after the tile's (first)
// decode pass: the caller requests the next tile's inputs there, so that no
// wait for the decode's latent loads covers them.
template <int METHOD, int P, bool STATS, bool FB, int FILTER, class AfterDecode>
__device__ __forceinline__ void dec_tile(const FilterArgs& a, const InferGrid& G, const FwdWeights<P>& W,
                                         const Biases& Bz, DecLds& L, int64_t tile, int tx, int ty,
                                         const Footprint& f, FrameCounters& fc, AfterDecode&& after_decode)
{
    static_assert(!batched<METHOD, FB>(), "the other calls run k_filter_dec_batch");
    constexpr int F = Taps<FILTER>::F, O = Taps<FILTER>::O;
    const int lane = lane_id();
    const int px = tx * kTile + (lane & 7), py = ty * kTile + (lane >> 3);
    const bool in_screen = px < a.sw && py < a.sh;
    const int64_t pix = (int64_t)py * a.sw + px;
    const int ox = f.x0 - O, oy = f.y0 - O;   // upper-left tap of the FxF footprint
    const bool inA = f.active && f.magnify;
    const uint64_t act = ballot(f.active);
    const uint64_t A = ballot(inA);
    const int nA = popc64(A);

    int xmin = 0, ymin = 0, bbw = 0, bbh = 0;
    constexpr bool kCollab = METHOD == CTF_LIST || METHOD == CTF_BOX || METHOD == CTF_MASK;
    if ((kCollab || STATS) && nA > 0) {
        xmin = wave_min(inA ? ox : INT32_MAX);
        ymin = wave_min(inA ? oy : INT32_MAX);
        bbw = wave_max(inA ? ox + F - 1 : INT32_MIN) - xmin + 1;
        bbh = wave_max(inA ? oy + F - 1 : INT32_MIN) - ymin + 1;
    }
    const bool fits16 = nA > 0 && bbw <= 16 && bbh <= 16;

    // ---- 16x16 wave mask B (Mask Sampling; also the exact set when it
    // fits).  Each lane of A marks only its footprint's upper-left texel
    // (mask C, one LDS byte and four ballots); B is C spread over the FxF
    // footprint with 256-bit shifts (rows of 16 do not wrap when the box
    // fits).
    uint64_t B[4] = {0, 0, 0, 0};
    int nmask = 0;
    constexpr bool kNeedMask = METHOD == CTF_MASK || METHOD == CTF_LIST || STATS;
    if (kNeedMask && fits16) {
        reinterpret_cast<uint32_t*>(L.bytes)[lane] = 0u;
        wave_lds_sync();
        if (inA) L.bytes[16 * (oy - ymin) + (ox - xmin)] = 1;
        wave_lds_sync();
        uint64_t C[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) C[w] = ballot(L.bytes[64 * w + lane] != 0);
        footprint_mask_f<F>(C, B);
        nmask = popc64(B[0]) + popc64(B[1]) + popc64(B[2]) + popc64(B[3]);
    }

    const int k = a.max_evals;
    auto& seg = reinterpret_cast<SegmentScratch<F>&>(L.vals);
    int n = 0, n0 = 0;
    bool cap_ok = true, count_ok = true, success = false, sorted = false;
    int unique = nmask;
    if constexpr (METHOD == CTF_BOX) {
        const int64_t area = (int64_t)bbw * bbh;
        n = area > INT32_MAX ? INT32_MAX : (int)area;
        cap_ok = (a.box_w == 0 || bbw <= a.box_w) && (a.box_h == 0 || bbh <= a.box_h);
        count_ok = area <= (int64_t)k * nA;
        success = nA > 0 && cap_ok && count_ok;
    } else if constexpr (METHOD == CTF_MASK) {
        cap_ok = fits16;
        n = fits16 ? nmask : 0;
        count_ok = n <= k * nA;
        success = fits16 && count_ok;
    } else if constexpr (METHOD == CTF_LIST) {
        if (nA > 0 && !fits16) {
            n = segment_sort(seg, L.rank, inA, 0, ox, oy, xmin, ymin, n0);
            sorted = true;
        } else {
            n = nmask;
        }
        unique = n;
        count_ok = n <= k * nA;
        success = nA > 0 && count_ok;
    }
    if constexpr (STATS && METHOD != CTF_LIST) {
        if (nA > 0 && !fits16) unique = segment_sort(seg, L.rank, inA, 0, ox, oy, xmin, ymin, n0);
    }
    if (nA == 0) unique = 0;

    bool exact, draws;
    if constexpr (METHOD == CTF_BILINEAR4) {
        exact = f.active;
        draws = false;
    } else {
        exact = inA && success;
        draws = f.active && !exact;
    }
    const uint64_t stfmask = ballot(draws);
    const int nstf = popc64(stfmask);
    int2 pick = make_int2(INT32_MIN, INT32_MIN);
    uint32_t h1 = 0, h2 = 0;
    if (draws) {
        stf_hashes(a.seed, a.layer, px, py, h1, h2);
        pick = stf_pick_filter<FILTER>(f, h1, h2);
    }
    const int rank_act = mbcnt(act);

    if constexpr (METHOD == CTF_BILINEAR4 && F == 4) {
        // ---- the full 4x4 filter: 16 taps per active lane do not fit one
        // row list, so the footprint rows are decoded one at a time (4 taps
        // per lane, up to 256 rows) and accumulated as in the gather below
        float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
        const int R = 4 * popc64(act);
        for (int jr = 0; jr < 4; ++jr) {
            if (f.active) {
#pragma unroll
                for (int i = 0; i < 4; ++i) L.rows[4 * rank_act + i] = make_int2(ox + i, oy + jr);
            }
            wave_lds_sync();
            decode_rows<P>(L.rows, L.vals, R, G, W, Bz);
            if (jr == 0) after_decode();
            wave_lds_sync();
            if (exact) {
                float wx[4], wy[4];
                taps32<FILTER>(f.s, wx);
                taps32<FILTER>(f.t, wy);
                const int b = 4 * rank_act;
                const float4 r = row4(wx, L.vals[b], L.vals[b + 1], L.vals[b + 2], L.vals[b + 3]);
                res = col_acc(wy[jr], r, res, jr == 0);
            }
            wave_lds_sync();
        }
        if (in_screen) {
            reinterpret_cast<float4*>(a.out)[pix] = res;
            if (a.stf_xy) reinterpret_cast<int2*>(a.stf_xy)[pix] = make_int2(INT32_MIN, INT32_MIN);
        }
        if (STATS && lane == 0 && a.tile_stats)
            write_tile_stats(a, tile, act, A, stfmask, fits16, B, xmin, ymin, bbw, bbh, n, unique, 4 * R, success,
                             cap_ok, count_ok, nA);
        if (act) fc.add(4 * R, popc64(act), nstf, popc64(act & ~A), 4 * ((R + 15) & ~15), false, false);
        return;
    }

    // fallback C / C+ for the lanes of A of a failed wave (fallback.h)
    const bool fallback = FB && !success && nA > 0;
    const uint64_t mdraw = stfmask & ~A;   // minifying draws in a fallback wave
    FallbackPlan fp{};

    // ---- row list: the texels to produce (unique texels first, in the
    // method's order, then one row per fallback draw) and the inverse table
    // of Mask/List
    const int ns = success ? n : 0;
    int R;
    if constexpr (METHOD == CTF_BILINEAR4) {
        R = 4 * popc64(act);
        if (f.active) {
#pragma unroll
            for (int q = 0; q < 4; ++q) L.rows[4 * rank_act + q] = make_int2(f.x0 + (q & 1), f.y0 + (q >> 1));
        }
    } else if (fallback) {
        fp = plan_fallback<FILTER>(L, a.fallback, inA, nA, mbcnt(A), f, pick, pcg_hash(h2), fits16, xmin, ymin);
        R = fp.nprod + popc64(mdraw);
        if (fp.produces) L.rows[fp.slot] = fp.texel;
        if (draws && !inA) L.rows[fp.nprod + mbcnt(mdraw)] = pick;
    } else {
        R = ns + nstf;
        if (success) {
            if (sorted) {
                segment_emit(seg, [&](int i, int, int dx, int dy) {
                    L.rows[i] = make_int2(xmin + dx, ymin + dy);
                    if (STATS && a.lists)
                        reinterpret_cast<int2*>(a.lists)[(size_t)tile * kMaxItems + i] = make_int2(xmin + dx, ymin + dy);
                });
            } else if (METHOD == CTF_BOX) {
                for (int i = lane; i < ns; i += kWave) {
                    const int2 c = make_int2(xmin + i % bbw, ymin + i / bbw);
                    L.rows[i] = c;
                    if (STATS && a.lists) reinterpret_cast<int2*>(a.lists)[(size_t)tile * kMaxItems + i] = c;
                }
            } else {
                // set bit t of B with rank r: row r, and rank[t] = r (h^-1)
                int base = 0;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    if ((B[w] >> lane) & 1u) {
                        const int r = base + mbcnt(B[w]);
                        const int t = 64 * w + lane;
                        const int2 c = make_int2(xmin + (t & 15), ymin + (t >> 4));
                        L.rank[t] = (uint8_t)r;
                        L.rows[r] = c;
                        if (STATS && a.lists) reinterpret_cast<int2*>(a.lists)[(size_t)tile * kMaxItems + r] = c;
                    }
                    base += popc64(B[w]);
                }
            }
        }
        if (draws) L.rows[ns + mbcnt(stfmask)] = pick;
    }
    // the debug draws are known now; write them before the decode so the
    // draw is not kept live across it
    if (in_screen && a.stf_xy)
        reinterpret_cast<int2*>(a.stf_xy)[pix] = draws ? pick : make_int2(INT32_MIN, INT32_MIN);
    // where the first tap of this lane's footprint row j sits: gi + gd j (Box:
    // the item; Mask and List: its place in the table); the row's other taps
    // are the next items
    int gi = 0, gd = 0;
    if constexpr (METHOD == CTF_BOX) {
        gi = (ox - xmin) + (oy - ymin) * bbw;
        gd = bbw;
    } else if constexpr (METHOD == CTF_LIST || METHOD == CTF_MASK) {
        gi = sorted ? F * lane : 16 * (oy - ymin) + (ox - xmin);
        gd = sorted ? 1 : 16;
    }
    const int draw_row = ns + mbcnt(stfmask);
    wave_lds_sync();

    // ---- decode the rows, 16 per MFMA tile; the latent gathers of the
    // next tile are in flight during the MLP of the current one
    decode_rows<P>(L.rows, L.vals, R, G, W, Bz);
    after_decode();
    wave_lds_sync();

    // ---- gather and weight
    float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (METHOD == CTF_BILINEAR4) {
        if (exact) {
            const int b = 4 * rank_act;
            res = bilerp(f.s, f.t, L.vals[b], L.vals[b + 1], L.vals[b + 2], L.vals[b + 3]);
        }
    } else if (fallback) {
        if (draws && !inA) res = L.vals[fp.nprod + mbcnt(mdraw)];
        if (inA) res = fallback_color<FILTER>(L, fp, f, pick, xmin, ymin);
    } else {
        if (draws) res = L.vals[draw_row];
        if (kCollab && exact) {
            auto row_item = [&](int jj) -> int {
                if constexpr (METHOD == CTF_BOX) return gi + gd * jj;
                else return L.rank[gi + gd * jj];
            };
            if constexpr (F == 2) {
                const int i0 = row_item(0), i1 = row_item(1);
                res = bilerp(f.s, f.t, L.vals[i0], L.vals[i0 + 1], L.vals[i1], L.vals[i1 + 1]);
            } else {
                float wx[4], wy[4];
                taps32<FILTER>(f.s, wx);
                taps32<FILTER>(f.t, wy);
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const float4* const v = L.vals + row_item(jj);
                    res = col_acc(wy[jj], row4(wx, v[0], v[1], v[2], v[3]), res, jj == 0);
                }
            }
        }
    }
    if (in_screen) reinterpret_cast<float4*>(a.out)[pix] = res;
    if (STATS && lane == 0 && a.tile_stats)
        write_tile_stats(a, tile, act, A, stfmask, fits16, B, xmin, ymin, bbw, bbh, n, unique, R, success, cap_ok,
                         count_ok, nA);
    if (act) fc.add(R, popc64(act), nstf, popc64(act & ~A), (R + 15) & ~15, kCollab && success,
                    kCollab && nA && !success);
    wave_lds_sync();  // the next tile reuses this wave's LDS slice
}

// Pixel offset of this lane inside its tile, (lane / 8) sw + lane % 8: a
// tile's pixel addresses are a scalar base plus this per-lane constant.
__device__ __forceinline__ uint32_t lane_pixel(const FilterArgs& a)
{
    const int lane = lane_id();
    uint32_t lp = (uint32_t)(lane >> 3) * (uint32_t)a.sw + (uint32_t)(lane & 7);
    // opaque to the optimizer, so that an access stays "scalar base + this
    // 32-bit offset" (an SGPR-based global access) rather than a hoisted
    // 64-bit per-lane pointer
    asm volatile("" : "+v"(lp));
    return lp;
}

// First pixel of tile (tx, ty) and whether all of its pixels are on screen
// (both wave-uniform).
__device__ __forceinline__ int64_t tile_pixel0(const FilterArgs& a, int tx, int ty)
{
    return (int64_t)ty * kTile * a.sw + (int64_t)tx * kTile;
}

__device__ __forceinline__ bool tile_interior(const FilterArgs& a, int tx, int ty)
{
    return tx * kTile + kTile <= a.sw && ty * kTile + kTile <= a.sh;
}

__device__ __forceinline__ bool lane_on_screen(const FilterArgs& a, int tx, int ty)
{
    if (tile_interior(a, tx, ty)) return true;
    const int lane = lane_id();
    return tx * kTile + (lane & 7) < a.sw && ty * kTile + (lane >> 3) < a.sh;
}

// Tiles of a workgroup, taken one at a time by its waves.
//
// The share: workgroups go round-robin over the 8 XCDs, and XCD x owns the
// strips of kStripRows tile rows whose index is x mod 8 (neighbouring tile
// rows, which share latent cells, stay in one XCD's L2).  Contiguous eighths
// of the screen balance badly: the texels a tile decodes vary down a frame (a
// minifying region decodes one per pixel), so on a 3840x2160 frame of four
// planes the costliest eighth decoded twice the rows of the cheapest and its
// XCD finished last.  The XCD's workgroups take runs of 2^run tiles of its
// rows in turn, left to right.
//
// Inside the workgroup the waves draw tiles from an LDS counter.  With a
// fixed share per wave the SIMD's issue order (oldest wave first) let one
// wave of a SIMD run ahead of its two neighbours and end early: on a
// 3840x2160 List frame the waves ended between 88 and 153 us (mean 112) though
// their rows differ by 4 %, and the frame's last quarter ran with one or two
// waves per SIMD.  With 12 waves a workgroup fills a CU, so all waves that
// compete for a SIMD draw from one counter and end together.
constexpr int kStripLog = 1;   // strips of 2 tile rows
constexpr int kStripRows = 1 << kStripLog;

struct TilePos {
    int tx, ty;   // ty >= the frame's tile rows: no tile
};

struct TileQueue {
    int* counter;   // LDS: next index of the share
    int tiles_x, tiles_y;
    uint32_t inv;   // floor((2^32 - 1) / tiles_x)
    int wg, nwg, xcd, run;

    __device__ __forceinline__ TileQueue(int* c, const FilterArgs& a) : counter(c)
    {
        tiles_x = a.tiles_x;
        tiles_y = (int)(a.ntiles / a.tiles_x);
        inv = 0xffffffffu / (uint32_t)tiles_x;
        xcd = blockIdx.x & 7;
        wg = blockIdx.x >> 3;
        nwg = gridDim.x >> 3;
        // runs of neighbouring tiles share L1 lines; shorter ones where a
        // share holds few, so that the shares stay even.  4-tap frames, runs
        // of 1, 4, 8 and 16 (us): 640x480 (share 18) 19.8, 19.9, 24.0, 27.7;
        // 1279x717 (56) 49.5, 48.9, 54.3, 53.8; 1920x1080 (126) 100.5, 103.7,
        // 103.0, 106.7; 2560x1440 (225) and 3840x2160 (506) within 2 %, List
        // frames alike: only the short side of the rule is sharp
        const int64_t share = a.ntiles / gridDim.x;
        run = share >= 256 ? 3 : share >= 64 ? 2 : 0;
    }
    __device__ __forceinline__ bool has(TilePos p) const { return p.ty < tiles_y; }
    // Draws the next index (valid in lane 0 only; place() reads it there).
    __device__ __forceinline__ int draw() const
    {
        int i = 0;
        if (lane_id() == 0) i = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return i;
    }
    // Tile of share index i: index n of the XCD, whose row r is tile row
    // ((r / kStripRows) * 8 + xcd) * kStripRows + r mod kStripRows.  Rows grow
    // with i, so every index behind one past the frame is past it too.
    __device__ __forceinline__ TilePos place(int drawn) const
    {
        const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane(drawn);
        const uint32_t n = ((((i >> run) * (uint32_t)nwg + (uint32_t)wg) << run) | (i & ((1u << run) - 1u)));
        // the quotient estimate is exact or one low for n < 2^31
        uint32_t r = __umulhi(n, inv), tx = n - r * (uint32_t)tiles_x;
        if (tx >= (uint32_t)tiles_x) {
            tx -= (uint32_t)tiles_x;
            ++r;
        }
        TilePos p;
        p.tx = (int)tx;
        p.ty = (int)((((r >> kStripLog) << (3 + kStripLog)) + (uint32_t)(xcd << kStripLog)) | (r & (kStripRows - 1)));
        return p;
    }
};

// Zeroes a workgroup's queues (one per layer) behind the first tiles, which
// its waves take by their index; every thread calls this.
__device__ __forceinline__ void queue_init(int* queues, int layers)
{
    if ((int)threadIdx.x < layers) queues[threadIdx.x] = (int)(blockDim.x >> 6);
    __syncthreads();
}

// Inputs of a tile for this lane, NaN (inactive) off the screen or without a
// tile (per-lane 64-bit addresses: the per-tile kernels run faster with these
// than with load_tile_px_s, measured).
__device__ __forceinline__ void load_tile_px(const FilterArgs& a, const TileQueue& q, TilePos t, float2& uv, float4& d)
{
    const int lane = lane_id();
    uv = make_float2(__builtin_nanf(""), 0.f);
    d = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!q.has(t)) return;
    const int px = t.tx * kTile + (lane & 7), py = t.ty * kTile + (lane >> 3);
    if (px < a.sw && py < a.sh) {
        const int64_t i = (int64_t)py * a.sw + px;
        uv = reinterpret_cast<const float2*>(a.uv)[i];
        d = reinterpret_cast<const float4*>(a.duv)[i];
    }
}

// The same with a scalar tile base plus the lane's offset (the batched
// kernel).
__device__ __forceinline__ void load_tile_px_s(const FilterArgs& a, const TileQueue& q, TilePos t, float2& uv,
                                               float4& d)
{
    uv = make_float2(__builtin_nanf(""), 0.f);
    d = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!q.has(t)) return;
    if (lane_on_screen(a, t.tx, t.ty)) {
        const int64_t p0 = tile_pixel0(a, t.tx, t.ty);
        const uint32_t lp = lane_pixel(a);
        const char* const ub = reinterpret_cast<const char*>(reinterpret_cast<const float2*>(a.uv) + p0);
        const char* const db = reinterpret_cast<const char*>(reinterpret_cast<const float4*>(a.duv) + p0);
        uv = *reinterpret_cast<const float2*>(ub + lp * 8u);
        d = *reinterpret_cast<const float4*>(db + lp * 16u);
    }
}

// Wait for the first tile's inputs before entering a tile loop.  The loop
// loads each next tile's inputs one tile ahead and copies them at the top of
// the next iteration; without this, the loads issued before the loop are
// still pending into the registers the first iteration reads, and the
// memory-counter wait placed at the loop head (counters drain in order)
// would also wait for the prefetch issued in every later iteration.
__device__ __forceinline__ void settle(const float2& uv, const float4& d)
{
    asm volatile("" ::"v"(uv.x), "v"(uv.y), "v"(d.x), "v"(d.y), "v"(d.z), "v"(d.w));
}

// Dynamic LDS of a workgroup: the queues, then one slice per wave.
constexpr int kQueueBytes = 64;
extern __shared__ __align__(16) char dec_lds[];

template <class Slice>
__device__ __forceinline__ Slice& wave_slice()
{
    return reinterpret_cast<Slice*>(dec_lds + kQueueBytes)[wave_in_block()];
}

// Walk of the per-tile kernels: foot(uv, d) is the lanes' footprint in the
// layer's coordinates.
template <int METHOD, int P, bool STATS, bool FB, int FILTER, class Foot>
__device__ __forceinline__ void tile_walk(const FilterArgs& a, DecLds& L, const InferGrid& G, const FwdWeights<P>& W,
                                          const Biases& Bz, const TileQueue& q, FrameCounters& fc, Foot&& foot)
{
    // the inputs of the wave's next tile are loaded one tile ahead, its index
    // is drawn two ahead
    float2 uv;
    float4 d;
    TilePos next = q.place(wave_in_block());
    int ahead = q.draw();
    load_tile_px(a, q, next, uv, d);
    settle(uv, d);
    while (q.has(next)) {
        const TilePos cur = next;
        const Footprint f = foot(uv, d);
        dec_tile<METHOD, P, STATS, FB, FILTER>(a, G, W, Bz, L, (int64_t)cur.ty * a.tiles_x + cur.tx, cur.tx, cur.ty, f,
                                               fc, [&] {
            next = q.place(ahead);
            ahead = q.draw();
            load_tile_px(a, q, next, uv, d);
        });
    }
}

template <int METHOD, int P, bool STATS, bool FB, int FILTER>
__global__ __launch_bounds__(64 * kDecWavesMax) void k_filter_dec(FilterArgs a, DevDecoderWeights D)
{
    const int lane = lane_id();
    int* const queues = reinterpret_cast<int*>(dec_lds);
    queue_init(queues, 1);
    FwdWeights<P> W;
    W.load(D.w, lane);
    Biases Bz;
    Bz.load(D.bias, lane);
    const float tex_w = (float)D.grid.tex_w;
    FrameCounters fc;
    tile_walk<METHOD, P, STATS, FB, FILTER>(a, wave_slice<DecLds>(), D.grid, W, Bz, TileQueue(queues, a), fc,
                                            [&](float2 uv, float4 d) {
        return footprint(uv.x, uv.y, d, tex_w, tex_w);
    });
    if (a.frame_stats) fc.flush(a.frame_stats);
}

// ---------------------------------------------------------------------------
// Batched decode (every method but the full filter, no C / C+ fallback).  A
// wave plans up to batch_slots() tiles, each tile's rows behind the last one's
// (at most 256 rows), decodes them in one pass and gathers the tiles, so the
// pass's start-up and its partial last MFMA tile are shared.  A planned
// tile's per-lane state waits in LDS until its gather, so no two tiles' state
// is live in registers.  Bound by issue: at 3840x2160 a List tile takes about
// 150 VALU and 220 scalar instructions to plan and gather, and its rows, in
// three 16-row tiles, 62 VALU and 14 MFMA each.
// Against one tile per pass: B-spline List 299 -> 184 us, six layers 1120 ->
// 880 us; against two tiles and bitonic sets, bilinear List 162 -> 135 us.
// ---------------------------------------------------------------------------

// Tiles per batch, measured at 3840x2160 with 2, 3, 4: bilinear List 139.7,
// 139.1, 137.5 us; B-spline List, whose tiles decode 70 rows on average,
// 184.9, 195.1, 197.9 us.
template <int F>
constexpr int batch_slots()
{
    return F == 2 ? 4 : 2;
}

// Per wave.  vals also holds the sort of a List past 16x16: no value is live
// while a tile is planned.
template <int F>
struct BatchLds {
    float4 vals[kMaxItems];               // decoded texels, by row
    int2 rows[kMaxItems];                 // texel coordinates to decode
    uint32_t window[kWindowWords];        // window_set
    uint8_t rank[256];                    // position of the window -> item
    static constexpr int kSlots = batch_slots<F>();
    float2 st[kSlots][kWave];             // footprint position of the lane
    uint32_t item[kSlots][kWave];         // F = 2: items of the two footprint rows, draw row and flags; F = 4: items
    uint32_t draw[F == 4 ? kSlots : 1][F == 4 ? kWave : 1];   // F = 4: draw row and flags
    int4 info[kSlots];                   // tile x, y, first row, whether wholly on screen
};
static_assert(sizeof(SegmentScratch<4>) <= kMaxItems * sizeof(float4), "sort in vals");

// Per-lane flags over the draw row.
constexpr uint32_t kExact = 1u << 15, kDraws = 1u << 14;

// Plan one tile on the batch's rows from `base`: decisions, rows, per-lane
// state of `slot`, debug outputs, tile record and counters.  Returns the
// tile's row count, or -1, with nothing written, if its rows do not fit behind
// the others.
template <int METHOD, bool STATS, int FILTER>
__device__ __forceinline__ int plan_tile(const FilterArgs& a, BatchLds<Taps<FILTER>::F>& BL, int slot, int base,
                                         int64_t tile, int tx, int ty, const WaveFootprint& f, FrameCounters& fc)
{
    constexpr int F = Taps<FILTER>::F, O = Taps<FILTER>::O;
    constexpr bool kCollab = collaborative(METHOD);
    constexpr bool kWindowed = METHOD == CTF_LIST || METHOD == CTF_MASK;
    auto& seg = reinterpret_cast<SegmentScratch<F>&>(BL.vals);
    const int lane = lane_id();
    const bool inside = tile_interior(a, tx, ty);
    const uint64_t act = f.act, A = f.A;
    const int nA = popc64(A);
    const int ox = f.x0 - O, oy = f.y0 - O;   // upper-left tap of the FxF footprint

    int xmin = 0, ymin = 0, bbw = 0, bbh = 0;
    // Mask and List only need a 16x16 window that holds every footprint of
    // A: try the one centred on a lane of A (lane 36 when it is in A) before
    // reducing the exact box.  Positions are relative to the window's corner;
    // the texels, their order and every decision are the same.
    bool window = false;
    if constexpr (kWindowed && !STATS) {
        if (A) {
            const int rl = ((A >> 36) & 1ull) ? 36 : (int)__builtin_ctzll(A);
            xmin = __builtin_amdgcn_readlane(ox, rl) - (16 - F) / 2;
            ymin = __builtin_amdgcn_readlane(oy, rl) - (16 - F) / 2;
            const uint32_t dx = (uint32_t)ox - (uint32_t)xmin, dy = (uint32_t)oy - (uint32_t)ymin;
            window = (ballot((dx > dy ? dx : dy) > (uint32_t)(16 - F)) & A) == 0;
        }
    }
    if ((kCollab || STATS) && A && !window) {
        const bool inA = lane_in(A);
        xmin = wave_min(inA ? ox : INT32_MAX);
        ymin = wave_min(inA ? oy : INT32_MAX);
        bbw = wave_max(inA ? ox + F - 1 : INT32_MIN) - xmin + 1;
        bbh = wave_max(inA ? oy + F - 1 : INT32_MIN) - ymin + 1;
    }
    const bool fits16 = window || (A && bbw <= 16 && bbh <= 16);

    const int corner = lane_in(A) ? 16 * (oy - ymin) + (ox - xmin) : 0;
    WindowSet S{0u, 0u, 0};
    uint64_t B[4] = {0, 0, 0, 0};   // tile records only
    if ((kWindowed || STATS) && fits16) {
        S = window_set<F>(BL.window, lane_in(A), corner);
        if constexpr (STATS) {
            const uint8_t* bytes = reinterpret_cast<const uint8_t*>(BL.window + kWindowPad);
            uint64_t C[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) C[w] = ballot(bytes[64 * w + lane] != 0);
            footprint_mask_f<F>(C, B);
        }
    }

    const int k = a.max_evals;
    int n = 0, n0 = 0;
    bool cap_ok = true, count_ok = true, success = false, sorted = false;
    int unique = S.n;
    if constexpr (METHOD == CTF_BOX) {
        const int64_t area = (int64_t)bbw * bbh;
        n = area > INT32_MAX ? INT32_MAX : (int)area;
        cap_ok = (a.box_w == 0 || bbw <= a.box_w) && (a.box_h == 0 || bbh <= a.box_h);
        count_ok = area <= (int64_t)k * nA;
        success = nA > 0 && cap_ok && count_ok;
    } else if constexpr (METHOD == CTF_MASK) {
        cap_ok = fits16;
        n = S.n;
        count_ok = n <= k * nA;
        success = fits16 && count_ok;
    } else if constexpr (METHOD == CTF_LIST) {
        n = S.n;
        if (A && !fits16) {
            n = segment_sort(seg, BL.rank, lane_in(A), 0, ox, oy, xmin, ymin, n0);
            sorted = true;
        }
        unique = n;
        count_ok = n <= k * nA;
        success = nA > 0 && count_ok;
    }
    if constexpr (STATS && METHOD != CTF_LIST) {
        if (A && !fits16) unique = segment_sort(seg, BL.rank, lane_in(A), 0, ox, oy, xmin, ymin, n0);
    }
    if (nA == 0) unique = 0;

    // lanes filtered exactly; the other active lanes draw one texel
    const uint64_t exact = kCollab && success ? A : 0ull;
    const uint64_t stfmask = act & ~exact;
    const int nstf = popc64(stfmask);
    const int ns = success ? n : 0;
    const int R = ns + nstf;
    if (base + R > kMaxItems) return -1;
    int2 pick = make_int2(INT32_MIN, INT32_MIN);
    int2* const dst = BL.rows + base;
    const int draw_row = ns + mbcnt(stfmask);
    if (lane_in(stfmask)) {
        uint32_t h1, h2;
        stf_hashes(a.seed, a.layer, tx * kTile + (lane & 7), ty * kTile + (lane >> 3), h1, h2);
        Footprint g;
        g.x0 = f.x0;
        g.y0 = f.y0;
        g.s = f.s;
        g.t = f.t;
        pick = stf_pick_filter<FILTER>(g, h1, h2);
        dst[draw_row] = pick;
    }

    // rows and the items of this lane's footprint rows (their first taps: in
    // a row-major list the texel right of a footprint texel is the next item)
    int item[F];
#pragma unroll
    for (int r = 0; r < F; ++r) item[r] = 0;
    auto list_out = [&](int i, int2 c) {
        if (STATS && a.lists) reinterpret_cast<int2*>(a.lists)[(size_t)tile * kMaxItems + i] = c;
    };
    if (success) {
        if (METHOD == CTF_BOX) {
            for (int i = lane; i < ns; i += kWave) {
                const int2 c = make_int2(xmin + i % bbw, ymin + i / bbw);
                dst[i] = c;
                list_out(i, c);
            }
#pragma unroll
            for (int r = 0; r < F; ++r) item[r] = (ox - xmin) + (oy + r - ymin) * bbw;
        } else if (sorted) {
            segment_emit(seg, [&](int i, int, int dx, int dy) {
                dst[i] = make_int2(xmin + dx, ymin + dy);
                list_out(i, make_int2(xmin + dx, ymin + dy));
            });
#pragma unroll
            for (int r = 0; r < F; ++r) item[r] = BL.rank[F * lane + r];
        } else {
            reinterpret_cast<uint32_t*>(BL.rank)[lane] = S.ranks;
            const int cx = xmin + 4 * (lane & 3), cy = ymin + (lane >> 2);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (S.set & (1u << (8 * q))) {
                    const int r = (int)((S.ranks >> (8 * q)) & 0xffu);
                    dst[r] = make_int2(cx + q, cy);
                    list_out(r, make_int2(cx + q, cy));
                }
            }
            wave_lds_sync();
#pragma unroll
            for (int r = 0; r < F; ++r) item[r] = BL.rank[(corner + 16 * r) & 0xff];
        }
    }
    if (a.stf_xy && (inside || lane_on_screen(a, tx, ty)))
        reinterpret_cast<int2*>(a.stf_xy)[tile_pixel0(a, tx, ty) + lane_pixel(a)] = pick;
    BL.st[slot][lane] = make_float2(f.s, f.t);
    const uint32_t misc = (uint32_t)(draw_row & 0xff) | (lane_in(exact) ? kExact : 0u) | (lane_in(stfmask) ? kDraws : 0u);
    if constexpr (F == 2) {
        BL.item[slot][lane] = (uint32_t)(item[0] & 0xff) | (uint32_t)(item[1] & 0xff) << 8 | misc << 16;
    } else {
        BL.item[slot][lane] = (uint32_t)(item[0] & 0xff) | (uint32_t)(item[1] & 0xff) << 8 |
                              (uint32_t)(item[2] & 0xff) << 16 | (uint32_t)(item[3] & 0xff) << 24;
        BL.draw[slot][lane] = misc;
    }
    if (lane == 0) BL.info[slot] = make_int4(tx, ty, base, inside ? 1 : 0);
    if (STATS && lane == 0 && a.tile_stats)
        write_tile_stats(a, tile, act, A, stfmask, fits16, B, xmin, ymin, bbw, bbh, n, unique, R, success, cap_ok,
                         count_ok, nA);
    if (act) fc.add(R, popc64(act), nstf, popc64(act & ~A), 0, kCollab && success, kCollab && nA && !success);
    return R;
}

// Gather and weight a decoded tile from its per-lane state.
template <int METHOD, int FILTER>
__device__ __forceinline__ void gather_tile(const FilterArgs& a, const BatchLds<Taps<FILTER>::F>& BL, int slot)
{
    constexpr int F = Taps<FILTER>::F;
    const int lane = lane_id();
    const int4 info = BL.info[slot];
    const float2 st = BL.st[slot][lane];
    const uint32_t item = BL.item[slot][lane];
    const uint32_t misc = F == 2 ? item >> 16 : BL.draw[F == 4 ? slot : 0][F == 4 ? lane : 0];
    const int tx = __builtin_amdgcn_readfirstlane(info.x), ty = __builtin_amdgcn_readfirstlane(info.y);
    const float4* const vals = BL.vals + __builtin_amdgcn_readfirstlane(info.z);
    float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
    if (misc & kDraws) res = vals[misc & 0xff];
    if (collaborative(METHOD) && (misc & kExact)) {
        if constexpr (F == 2) {
            const int i0 = item & 0xff, i1 = (item >> 8) & 0xff;
            res = bilerp(st.x, st.y, vals[i0], vals[i0 + 1], vals[i1], vals[i1 + 1]);
        } else {
            float wx[4], wy[4];
            taps32<FILTER>(st.x, wx);
            taps32<FILTER>(st.y, wy);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4* const v = vals + ((item >> (8 * r)) & 0xff);
                res = col_acc(wy[r], row4(wx, v[0], v[1], v[2], v[3]), res, r == 0);
            }
        }
    }
    if (__builtin_amdgcn_readfirstlane(info.w) || lane_on_screen(a, tx, ty)) {
        char* const ob = reinterpret_cast<char*>(reinterpret_cast<float4*>(a.out) + tile_pixel0(a, tx, ty));
        *reinterpret_cast<float4*>(ob + lane_pixel(a) * 16u) = res;
    }
}

// The wave's share of one layer: plan, decode and gather its tiles in
// batches.  foot(uv, d) is the lanes' footprint in the layer's coordinates.
template <int METHOD, int P, bool STATS, int FILTER, class Foot>
__device__ __forceinline__ void batch_walk(const FilterArgs& a, BatchLds<Taps<FILTER>::F>& BL, const InferGrid& G,
                                           const FwdWeights<P>& W, const Biases& Bz, const TileQueue& q,
                                           FrameCounters& fc, Foot&& foot)
{
    int npend = 0, rows = 0, last = 0;
    bool redo = false;
    TilePos next = q.place(wave_in_block()), held{0, 0};
    int ahead = q.draw();
    float2 uv_next;
    float4 d_next;
    load_tile_px_s(a, q, next, uv_next, d_next);
    for (;;) {
        // The next tile's inputs were requested before the last tile was
        // planned: wait for them here, before the gather's stores, which
        // complete in order with them.
        settle(uv_next, d_next);
        const bool more = q.has(next);
        // a batch is full when no slot is left or a tile like the last one
        // would not fit (plan_tile has the final word)
        if (npend && (!more || redo || npend == BatchLds<Taps<FILTER>::F>::kSlots || rows + last > kMaxItems)) {
            wave_lds_sync();
            decode_rows<P>(BL.rows, BL.vals, rows, G, W, Bz);
            wave_lds_sync();
            for (int i = 0; i < npend; ++i) gather_tile<METHOD, FILTER>(a, BL, i);
            fc.rows += (uint32_t)((rows + 15) & ~15);
            npend = 0;
            rows = 0;
            wave_lds_sync();
        }
        if (!more) break;
        float2 uv = uv_next;
        float4 d = d_next;
        // (copies made here: otherwise the next request goes to other
        // registers and is waited for at once, to be moved into these)
        asm volatile("" : "+v"(uv.x), "+v"(uv.y), "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w));
        const TilePos cur = next;
        if (redo) {
            next = held;
        } else {
            next = q.place(ahead);
            ahead = q.draw();
        }
        load_tile_px_s(a, q, next, uv_next, d_next);
        const WaveFootprint f = foot(uv, d);
        const int R = plan_tile<METHOD, STATS, FILTER>(a, BL, npend, rows, (int64_t)cur.ty * a.tiles_x + cur.tx, cur.tx,
                                                       cur.ty, f, fc);
        redo = R < 0;
        if (redo) {
            held = next;
            next = cur;
            load_tile_px_s(a, q, next, uv_next, d_next);
        } else {
            ++npend;
            rows += R;
            last = R;
        }
    }
}

template <int F>
__device__ __forceinline__ void batch_init(BatchLds<F>& BL)
{
    if (lane_id() < kWindowPad) BL.window[lane_id()] = 0u;
    wave_lds_sync();
}

template <int METHOD, int P, bool STATS, int FILTER>
__global__ __launch_bounds__(64 * kDecWavesMax) void k_filter_dec_batch(FilterArgs a, DevDecoderWeights D)
{
    const int lane = lane_id();
    auto& BL = wave_slice<BatchLds<Taps<FILTER>::F>>();
    int* const queues = reinterpret_cast<int*>(dec_lds);
    batch_init(BL);
    queue_init(queues, 1);
    FwdWeights<P> W;
    W.load(D.w, lane);
    Biases Bz;
    Bz.load(D.bias, lane);
    const float tex_w = (float)D.grid.tex_w;
    FrameCounters fc;
    batch_walk<METHOD, P, STATS, FILTER>(a, BL, D.grid, W, Bz, TileQueue(queues, a), fc, [&](float2 uv, float4 d) {
        return wave_footprint(uv.x, uv.y, d, tex_w, tex_w);
    });
    if (a.frame_stats) fc.flush(a.frame_stats);
}

// Waves of a workgroup for n units of work (tiles, or 32-texel passes): twelve
// from seven units per CU, four below.  A large workgroup's waves share the
// work of their CU through one counter (see TileQueue); four-wave workgroups
// spread a small frame over all CUs, but a CU may get one or three of them.
// Fp16 frames, four and twelve waves (us): 384x256 (6 tiles per CU) List 11.7,
// 12.0, 4-tap 10.6, 13.1; 384x320 (7.5) 13.1, 12.6 and 16.8, 15.9; 640x480
// (18.8) 16.0, 15.4 and 24.0, 20.8; 1280x720 25.5, 23.4 and 54.5, 50.6; texel
// evaluation is within 4 % either way.
inline int dec_waves(int64_t n, int64_t cus) { return n >= 7 * cus ? kDecWavesMax : kDecWavesMin; }

// Persistent grid: the workgroups that fill the chip with three waves per
// SIMD, a multiple of the 8 XCDs.
struct DecLaunch {
    int threads;
    int64_t blocks;
    unsigned lds;
};

template <class Slice>
DecLaunch dec_launch(const FilterArgs& a, int layers)
{
    static_assert(kQueueBytes + kDecWavesMax * sizeof(Slice) <= 160 * 1024, "a workgroup's LDS");
    const int64_t cus = a.cus;
    const int waves = dec_waves(a.ntiles, cus);
    DecLaunch g;
    g.threads = 64 * waves;
    g.blocks = (a.ntiles + waves - 1) / waves;
    if (g.blocks > cus * (kDecWavesMax / waves)) g.blocks = cus * (kDecWavesMax / waves);
    // one wave may take its workgroup's whole share (32-bit frame counters):
    // at most the frame's tiles and a strip per XCD, shared by the workgroups
    const int64_t least = counter_min_blocks((a.ntiles + (int64_t)8 * kStripRows * a.tiles_x) * layers, 1);
    if (g.blocks < least) g.blocks = least;
    g.blocks = (g.blocks + 7) / 8 * 8;
    g.lds = (unsigned)(kQueueBytes + waves * sizeof(Slice));
    return g;
}

// Tile indices of an XCD are 32-bit (2^30 tiles are 1 TB of output).
inline bool dec_indexable(const FilterArgs& a) { return a.ntiles <= (int64_t)1 << 30; }

// Instantiation for the call's statistics and fallback flags; waves of a
// collaborative method carry the C / C+ code only when it is asked for, so
// the common path keeps its register budget.
template <int METHOD, int P, template <int, int, bool, bool> class Go, class... Args>
hipError_t dispatch_flags(const FilterArgs& a, Args&&... args)
{
    // the instantiation with statistics also writes the texel lists; the
    // plain one writes the per-pixel draws only
    const bool st = a.tile_stats != nullptr || a.lists != nullptr;
    if constexpr (collaborative(METHOD)) {
        if (a.fallback != CTF_FB_STF1)
            return st ? Go<METHOD, P, true, true>::run(a, args...) : Go<METHOD, P, false, true>::run(a, args...);
    }
    return st ? Go<METHOD, P, true, false>::run(a, args...) : Go<METHOD, P, false, false>::run(a, args...);
}

template <int FILTER>
struct GoFilter {
    template <int METHOD, int P, bool STATS, bool FB>
    struct Go {
        static hipError_t run(const FilterArgs& a, const DevDecoderWeights& d, hipStream_t s)
        {
            if (!dec_indexable(a)) return hipErrorInvalidValue;
            if constexpr (batched<METHOD, FB>()) {
                const DecLaunch g = dec_launch<BatchLds<Taps<FILTER>::F>>(a, 1);
                hipLaunchKernelGGL((k_filter_dec_batch<METHOD, P, STATS, FILTER>), dim3((unsigned)g.blocks),
                                   dim3((unsigned)g.threads), g.lds, s, a, d);
            } else {
                const DecLaunch g = dec_launch<DecLds>(a, 1);
                hipLaunchKernelGGL((k_filter_dec<METHOD, P, STATS, FB, FILTER>), dim3((unsigned)g.blocks),
                                   dim3((unsigned)g.threads), g.lds, s, a, d);
            }
            return hipGetLastError();
        }
    };
};

template <int P, int FILTER>
hipError_t launch_dec_p(const FilterArgs& a, const DevDecoderWeights& d, hipStream_t s)
{
    switch (a.method) {
    case CTF_BILINEAR4: return dispatch_flags<CTF_BILINEAR4, P, GoFilter<FILTER>::template Go>(a, d, s);
    case CTF_STF1: return dispatch_flags<CTF_STF1, P, GoFilter<FILTER>::template Go>(a, d, s);
    case CTF_LIST: return dispatch_flags<CTF_LIST, P, GoFilter<FILTER>::template Go>(a, d, s);
    case CTF_BOX: return dispatch_flags<CTF_BOX, P, GoFilter<FILTER>::template Go>(a, d, s);
    case CTF_MASK: return dispatch_flags<CTF_MASK, P, GoFilter<FILTER>::template Go>(a, d, s);
    default: return hipErrorInvalidValue;
    }
}

// Several material layers in one launch: layer l samples its own decoder at
// uv_l = M_l uv (derivatives alike).  Layers are the outer loop so that one
// layer's latent grids stay resident in the L2 while its tiles are walked;
// each wave reloads the MLP weights once per layer.
constexpr int kMaxLayers = 8;
static_assert(kMaxLayers * sizeof(int) <= kQueueBytes, "a queue per layer");

struct LayerSet {
    DevDecoderWeights dec[kMaxLayers];
    float xf[kMaxLayers][4];   // row-major 2x2
    int n;
};

// LDS of one wave of the layered launch.
template <int METHOD, bool FB, int FILTER>
struct LayerLds {
    using Type = DecLds;
};
template <int METHOD, int FILTER>
struct LayerLds<METHOD, false, FILTER> {
    using Type = std::conditional_t<batched<METHOD, false>(), BatchLds<Taps<FILTER>::F>, DecLds>;
};

template <int METHOD, int P, bool STATS, bool FB, int FILTER>
__global__ __launch_bounds__(64 * kDecWavesMax) void k_filter_layers(FilterArgs a, LayerSet LS)
{
    const int lane = lane_id();
    auto& L = wave_slice<typename LayerLds<METHOD, FB, FILTER>::Type>();
    int* const queues = reinterpret_cast<int*>(dec_lds);
    if constexpr (batched<METHOD, FB>()) batch_init(L);
    queue_init(queues, LS.n);
    const int64_t npix = (int64_t)a.sw * a.sh;
    FrameCounters fc;
    for (int l = 0; l < LS.n; ++l) {
        const DevDecoderWeights& D = LS.dec[l];
        // (opaque, so that the lane's weight offsets are not kept in registers
        // across the tile walk for the next layer)
        int wl = lane;
        asm volatile("" : "+v"(wl));
        FwdWeights<P> W;
        W.load(D.w, wl);
        Biases Bz;
        Bz.load(D.bias, wl);
        const float tex_w = (float)D.grid.tex_w;
        const float m00 = LS.xf[l][0], m01 = LS.xf[l][1], m10 = LS.xf[l][2], m11 = LS.xf[l][3];
        FilterArgs al = a;
        al.out = a.out + (size_t)l * npix * 4;
        al.tile_stats = a.tile_stats ? a.tile_stats + (size_t)l * a.ntiles : nullptr;
        al.stf_xy = a.stf_xy ? a.stf_xy + (size_t)l * npix * 2 : nullptr;
        al.lists = nullptr;
        al.layer = (uint32_t)l;
        // layer coordinates, float32: u' = fma(m01, v, m00 u), v' = fma(m11, v, m10 u)
        auto layer_uv = [&](float2 uv) {
            return make_float2(__builtin_fmaf(m01, uv.y, m00 * uv.x), __builtin_fmaf(m11, uv.y, m10 * uv.x));
        };
        auto layer_d = [&](float4 d) {
            return make_float4(__builtin_fmaf(m01, d.y, m00 * d.x), __builtin_fmaf(m11, d.y, m10 * d.x),
                               __builtin_fmaf(m01, d.w, m00 * d.z), __builtin_fmaf(m11, d.w, m10 * d.z));
        };
        const TileQueue q(queues + l, a);
        if constexpr (batched<METHOD, FB>()) {
            batch_walk<METHOD, P, STATS, FILTER>(al, L, D.grid, W, Bz, q, fc, [&](float2 uv, float4 d) {
                const float2 lu = layer_uv(uv);
                return wave_footprint(lu.x, lu.y, layer_d(d), tex_w, tex_w);
            });
        } else {
            tile_walk<METHOD, P, STATS, FB, FILTER>(al, L, D.grid, W, Bz, q, fc, [&](float2 uv, float4 d) {
                const float2 lu = layer_uv(uv);
                return footprint(lu.x, lu.y, layer_d(d), tex_w, tex_w);
            });
        }
    }
    if (a.frame_stats) fc.flush(a.frame_stats);
}


template <int FILTER>
struct GoLayers {
    template <int METHOD, int P, bool STATS, bool FB>
    struct Go {
        static hipError_t run(const FilterArgs& a, const LayerSet& LS, hipStream_t s)
        {
            if (!dec_indexable(a)) return hipErrorInvalidValue;
            const DecLaunch g = dec_launch<typename LayerLds<METHOD, FB, FILTER>::Type>(a, LS.n);
            hipLaunchKernelGGL((k_filter_layers<METHOD, P, STATS, FB, FILTER>), dim3((unsigned)g.blocks),
                               dim3((unsigned)g.threads), g.lds, s, a, LS);
            return hipGetLastError();
        }
    };
};

template <int P, int FILTER>
hipError_t launch_layers_p(const FilterArgs& a, const LayerSet& LS, hipStream_t s)
{
    switch (a.method) {
    case CTF_BILINEAR4: return dispatch_flags<CTF_BILINEAR4, P, GoLayers<FILTER>::template Go>(a, LS, s);
    case CTF_STF1: return dispatch_flags<CTF_STF1, P, GoLayers<FILTER>::template Go>(a, LS, s);
    case CTF_LIST: return dispatch_flags<CTF_LIST, P, GoLayers<FILTER>::template Go>(a, LS, s);
    case CTF_BOX: return dispatch_flags<CTF_BOX, P, GoLayers<FILTER>::template Go>(a, LS, s);
    case CTF_MASK: return dispatch_flags<CTF_MASK, P, GoLayers<FILTER>::template Go>(a, LS, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dec

}  // namespace ctf
