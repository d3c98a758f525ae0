// filter_wave32.hip -- the paper's wave shape on gfx950: 8x4-pixel tiles of
// 32 lanes (Section 3: 8x4 pixels per wave32), two per wave64, one per
// half-wave.  Each half-wave takes its own collaborative step (Box, Mask,
// List, remapping and the one-tap fallback) exactly as a wave32 would, so
// the success regions of Figure 4 (bilinear) and of the bicubic maps of the
// supplement's additional bicubic results, and the evaluation counts, can
// be checked on hardware.  Per-lane texel production, bilinear or bicubic
// (FxF footprints, F = 2 or 4) filters, one-tap STF fallback.
//
// Half-wave quantities are computed for both halves as scalars (ballots
// split into their 32-bit halves, DPP reductions combined per pair of
// 16-lane rows) and each lane selects its own half's value.  Texels are
// evaluated once for the wave, whatever the halves decided: a half that
// succeeded and one that fell back fill the lanes of the same rounds, the
// terms come from the workgroup's LDS and the next pair's inputs are
// requested a pair ahead (Mask with C+ at 1920x1080, 32 terms: 95 -> 71 us,
// bound by the texel evaluations and the chain of LDS steps of a tile).
#include <type_traits>

#include "ctf_device.h"
#include "ctf_internal.h"
#include "fallback.h"

namespace ctf {

namespace {

constexpr int kW32Waves = 4;
constexpr int kHalfItems = kMaxItems / 2;  // n <= k |A| <= 4 * 32 per half

struct W32Lds {
    float4 vals[2][kHalfItems];   // produced texel values, by half and item; the List's sort before any
    // per half: the texels of a List past 16x16 by item, or (a failed half)
    // fallback C+'s footprints, or the texels produced by C past 16x16
    union Half {
        int2 list[kHalfItems];
        StashEntry stash[32];
        int2 produced[32];
    } half[2];
    uint32_t window[2 * kWindowWords];   // window_set_halves; fallback C+: byte scatter
    uint8_t items[2][256];        // Mask: item i -> position t = h(i, B)
    uint8_t rank[2][256];         // Mask: position t -> item index h^-1(t, B); fallback: slot + 1
    uint8_t first[256];           // List past 16x16: first items of each lane's footprint rows
    __device__ uint8_t* bytes(int h) { return reinterpret_cast<uint8_t*>(window + kWindowPad + kWindowWords * h); }
};
static_assert(sizeof(SegmentScratch<4>) <= 2 * kHalfItems * sizeof(float4), "sort in vals");
static_assert(kW32Waves * sizeof(W32Lds) + kLdsTermEntries * sizeof(int4) <= 40960, "four workgroups per CU");

// min/max over each half-wave (all 64 lanes active): DPP over the 16-lane
// rows, then rows 0,1 make half 0 and rows 2,3 half 1.
template <class Op>
__device__ __forceinline__ void halves_reduce(int v, Op op, int& r0, int& r1)
{
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false));
    v = op(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false));
    r0 = op(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
    r1 = op(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48));
}

__device__ __forceinline__ uint32_t lo32(uint64_t m) { return (uint32_t)m; }
__device__ __forceinline__ uint32_t hi32(uint64_t m) { return (uint32_t)(m >> 32); }

// Fallbacks C and C+ (Section 3.4, Eq. 1 and Eq. 2) per half-wave: the
// wave64 planning of fallback.h with every ballot, rank and table taken over
// the lanes of one 8x4 tile, so Eq. 2 spreads the spare lanes of a 32-lane
// wave as the paper writes it.  `fbl`: this lane's half takes the fallback.
struct W32Fallback {
    bool produces;
    int2 texel;
    int slot;
    bool table;
};

template <int FILTER, int F>
__device__ W32Fallback plan_fallback_w32(W32Lds& L, int fb, bool fbl, bool inA, int h, int nA, int rankA,
                                         const Footprint& f, int2 pick, uint32_t h3, bool fits16, int xmin, int ymin,
                                         uint64_t Hm, int& nprod0, int& nprod1)
{
    const int lane = lane_id(), ll = lane & 31;
    const bool mine = fbl && inA;
    W32Fallback P;
    P.produces = mine;
    P.texel = pick;
    P.table = fits16;
    if (fb == CTF_FB_CPLUS && ballot(fbl && fits16) != 0) {
        const bool cplus = fbl && fits16;
        reinterpret_cast<uint32_t*>(L.bytes(0))[lane] = 0u;
        reinterpret_cast<uint32_t*>(L.bytes(1))[lane] = 0u;
        if (cplus) L.half[h].stash[ll] = StashEntry{f.x0, f.y0, f.s, f.t};
        wave_lds_sync();
        if (mine && cplus) L.bytes(h)[16 * (pick.y - ymin) + (pick.x - xmin)] = 1;
        wave_lds_sync();
        // S per half: the distinct drawn texels of its lanes of A
        uint64_t S0[4], S1[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            S0[w] = ballot(L.bytes(0)[64 * w + lane] != 0);
            S1[w] = ballot(L.bytes(1)[64 * w + lane] != 0);
        }
        // items of the failed halves only: the other half keeps its own
        int ns0 = 0, ns1 = 0;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            const uint64_t* Sh = hh ? S1 : S0;
            int base = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if ((Sh[w] >> lane) & 1u) L.items[hh][base + mbcnt(Sh[w])] = (uint8_t)(64 * w + lane);
                base += popc64(Sh[w]);
            }
            if (hh) ns1 = base;
            else ns0 = base;
        }
        wave_lds_sync();
        // lane of each rank of A in its half (the bytes are free after the ballots)
        if (inA) L.bytes(h)[rankA] = (uint8_t)ll;
        wave_lds_sync();
        if (mine && cplus) {
            const int ns = h ? ns1 : ns0;
            P.produces = false;
            if (rankA < ns) {
                const int t = L.items[h][rankA];
                P.produces = true;
                P.texel = make_int2(xmin + (t & 15), ymin + (t >> 4));
            } else {
                constexpr int O = Taps<FILTER>::O;
                const StashEntry T = L.half[h].stash[L.bytes(h)[cplus_target(nA, ns, rankA)]];
                float wx[4], wy[4];
                taps32<FILTER>(T.s, wx);
                taps32<FILTER>(T.t, wy);
                const int ox = T.x0 - O, oy = T.y0 - O;
                // candidates: taps (row-major) with a nonzero weight, not in S
                uint32_t cand = 0u;
                float wsum = 0.f;
#pragma unroll
                for (int q = 0; q < F * F; ++q) {
                    const float wq = wx[q % F] * wy[q / F];
                    const int tq = 16 * (oy + q / F - ymin) + (ox + q % F - xmin);
                    const uint64_t Sw = h ? S1[tq >> 6] : S0[tq >> 6];
                    if (wq != 0.0f && !((Sw >> (tq & 63)) & 1u)) {
                        cand |= 1u << q;
                        wsum += __builtin_fabsf(wq);
                    }
                }
                if (cand) {
                    const float thr = (float)(h3 >> 8) * 0x1p-24f * wsum;
                    float run = 0.f;
                    int pq = -1;
                    bool done = false;
#pragma unroll
                    for (int q = 0; q < F * F; ++q) {
                        if (!((cand >> q) & 1u) || done) continue;
                        pq = q;
                        run += __builtin_fabsf(wx[q % F] * wy[q / F]);
                        done = run > thr;
                    }
                    P.produces = true;
                    P.texel = make_int2(ox + pq % F, oy + pq / F);
                }
            }
        }
    }
    const uint64_t prod = ballot(P.produces);
    nprod0 = __popc(lo32(prod));
    nprod1 = __popc(hi32(prod));
    P.slot = mbcnt(prod & Hm);
    // slot table of the fallback halves (the other half keeps its rank table)
    if (fbl && fits16) {
        reinterpret_cast<uint32_t*>(L.rank[h])[ll] = 0u;
        reinterpret_cast<uint32_t*>(L.rank[h])[32 + ll] = 0u;
    }
    wave_lds_sync();
    if (P.produces) {
        if (P.table) L.rank[h][16 * (P.texel.y - ymin) + (P.texel.x - xmin)] = (uint8_t)(P.slot + 1);
        else L.half[h].produced[P.slot] = P.texel;
    }
    wave_lds_sync();
    return P;
}

// Eq. 1 for a lane of A of a fallback half (fallback_color of fallback.h over
// this half's slots).
template <int FILTER, int F>
__device__ float4 fallback_color_w32(const W32Lds& L, const W32Fallback& P, int h, int nprod, const Footprint& f,
                                     int2 pick, int xmin, int ymin)
{
    constexpr int O = Taps<FILTER>::O;
    float wx[4], wy[4];
    taps32<FILTER>(f.s, wx);
    taps32<FILTER>(f.t, wy);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), sum = acc;
    float wsum = 0.f;
    int N = 0, own = 0;
#pragma unroll
    for (int q = 0; q < F * F; ++q) {
        const int x = f.x0 - O + q % F, y = f.y0 - O + q / F;
        const float wq = wx[q % F] * wy[q / F];
        int slot = -1;
        if (P.table) {
            slot = (int)L.rank[h][16 * (y - ymin) + (x - xmin)] - 1;
        } else {
            for (int r = 0; r < nprod; ++r) {
                const int2 e = L.half[h].produced[r];
                if (e.x == x && e.y == y) {
                    slot = r;
                    break;
                }
            }
        }
        if (x == pick.x && y == pick.y) own = slot;
        if (slot < 0 || wq == 0.0f) continue;
        const float4 v = L.vals[h][slot];
        acc.x = __builtin_fmaf(wq, v.x, acc.x);
        acc.y = __builtin_fmaf(wq, v.y, acc.y);
        acc.z = __builtin_fmaf(wq, v.z, acc.z);
        acc.w = __builtin_fmaf(wq, v.w, acc.w);
        sum.x += v.x;
        sum.y += v.y;
        sum.z += v.z;
        sum.w += v.w;
        wsum += wq;
        ++N;
    }
    if (N == 0) return L.vals[h][own];
    const float inv = 1.0f / (float)N, rest = 1.0f - wsum;
    return make_float4(__builtin_fmaf(rest, sum.x * inv, acc.x), __builtin_fmaf(rest, sum.y * inv, acc.y),
                       __builtin_fmaf(rest, sum.z * inv, acc.z), __builtin_fmaf(rest, sum.w * inv, acc.w));
}

struct HalfDecision {
    int n, unique;
    bool cap_ok, count_ok, success;
};

// LDS_TERMS (collaborative methods): lds_terms; the other methods choose at run
// time.  Five instructions per term need the terms in vector registers, from
// LDS by broadcast (a vector instruction reads one scalar register).  Terms
// that are not staged as floats (more than kLdsTerms, or the integer form of
// textures wider than 4096) are scalar loads instead: as broadcast vector
// loads, as in the 8x8 kernels, which have no scalar registers left for them,
// Mask at 1920x1080 takes 258 us in place of 130 with 70 terms and 81 in place
// of 60 with 16 integer ones.  With the LDS slices and the staged terms four
// workgroups fit a CU.
template <int METHOD, int TEX, bool STATS, int FILTER, bool FB, bool LDS_TERMS>
__global__ __launch_bounds__(kWave * kW32Waves, 4) void k_filter_w32(FilterArgs a, DevTexture T)
{
    constexpr int F = Taps<FILTER>::F, O = Taps<FILTER>::O;
    constexpr bool kCollab = METHOD == CTF_LIST || METHOD == CTF_BOX || METHOD == CTF_MASK;
    constexpr bool kStage = TEX == CTF_TEX_SINUSOIDS && (!kCollab || LDS_TERMS);
    constexpr bool kWindowed = METHOD == CTF_LIST || METHOD == CTF_MASK;
    __shared__ W32Lds lds_all[kW32Waves];
    __shared__ int4 terms_lds[kStage ? kLdsTermEntries : 1];
    const int wid = wave_in_block();
    const int lane = lane_id();
    const int h = lane >> 5, ll = lane & 31;
    W32Lds& L = lds_all[wid];
    if constexpr (kWindowed || STATS)
        if (lane < kWindowPad) L.window[lane] = L.window[kWindowWords + lane] = 0u;
    bool lds_float = false;
    if constexpr (kStage) lds_float = (stage_terms(T, terms_lds) && T.fterms != nullptr) || kCollab;
    const bool joint = lds_float && joint_texels(T);
    auto texel = [&](int x, int y) __attribute__((always_inline)) -> float4 {
        if constexpr (kStage) return texel_eval_staged<TEX>(T, terms_lds, lds_float, x, y);
        else return texel_eval<TEX>(T, x, y);
    };
    auto half_mask = [](uint64_t m, int hh) -> uint64_t {
        return hh ? m & 0xffffffff00000000ull : m & 0x00000000ffffffffull;
    };
    FrameCounters fc;
    // Pairs of tiles, the inputs of the wave's next pair loaded one pair
    // ahead; loads and the output store are unconditional (see
    // k_filter_simt).  A walk's tile is the pair's first, its second the next
    // one in row-major order.
    const int64_t nw = (int64_t)gridDim.x * kW32Waves;
    auto place = [&](const TileWalk& w, int& tx, int& ty) __attribute__((always_inline)) -> bool {
        const bool wrap = w.tx + 1 >= a.tiles_x;
        tx = h ? (wrap ? 0 : w.tx + 1) : w.tx;
        ty = h && wrap ? w.ty + 1 : w.ty;
        return w.tile + h < a.ntiles;
    };
    auto load_px = [&](const TileWalk& w, float2& uv, float4& d) __attribute__((always_inline)) -> bool {
        int tx, ty;
        const bool tile_ok = place(w, tx, ty);
        const int qx = tx * 8 + (ll & 7), qy = ty * 4 + (ll >> 3);
        const bool ok = tile_ok && qx < a.sw && qy < a.sh;
        const int64_t q = ok ? (int64_t)qy * a.sw + qx : 0;
        uv = reinterpret_cast<const float2*>(a.uv)[q];
        d = reinterpret_cast<const float4*>(a.duv)[q];
        return ok;
    };
    TileWalk next(2 * ((int64_t)blockIdx.x * kW32Waves + wid), 2 * nw, a.tiles_x);
    float2 uv_next;
    float4 d_next;
    bool ok_next = load_px(next, uv_next, d_next);
    asm volatile("" ::"v"(uv_next.x), "v"(uv_next.y), "v"(d_next.x), "v"(d_next.y), "v"(d_next.z), "v"(d_next.w));
    while (next.tile < a.ntiles) {
        const TileWalk cur = next;
        const float2 uv_cur = ok_next ? uv_next : make_float2(__builtin_nanf(""), 0.f);
        const float4 d_cur = ok_next ? d_next : make_float4(0.f, 0.f, 0.f, 0.f);
        next.advance(2 * nw);
        ok_next = load_px(next, uv_next, d_next);
        int tx, ty;
        const bool tile_ok = place(cur, tx, ty);
        const int64_t tile = cur.tile + h;
        const int px = tx * 8 + (ll & 7), py = ty * 4 + (ll >> 3);
        const bool in_screen = tile_ok && px < a.sw && py < a.sh;
        const int64_t pix = (int64_t)py * a.sw + px;

        const WaveFootprint f = wave_footprint(uv_cur.x, uv_cur.y, d_cur, (float)T.width, (float)T.height);
        const bool inA = lane_in(f.A);
        const int ox = f.x0 - O, oy = f.y0 - O;   // upper-left tap of the FxF footprint
        // (an opaque second half: as "A < 2^32" the test for an empty one became
        // a vector compare, and this compiler then lost the scalar condition
        // between two selects on it)
        uint32_t A0 = lo32(f.A), A1 = hi32(f.A);
        asm("" : "+s"(A0), "+s"(A1));
        const int nAs[2] = {(int)__popc(A0), (int)__popc(A1)};
        const int nA = h ? nAs[1] : nAs[0];
        const int rankA = h ? mbcnt(half_mask(f.A, 1)) : mbcnt(half_mask(f.A, 0));

        // ---- box per half.  Mask and List only need a 16x16 window that
        // holds every footprint of the half: try the one centred on a lane of
        // it (the tile's middle when it is in A) before reducing the boxes.
        int xmins[2] = {0, 0}, ymins[2] = {0, 0}, bbw[2] = {0, 0}, bbh[2] = {0, 0};
        bool window = false;
        if constexpr (kWindowed && !STATS) {
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const uint64_t m = half_mask(f.A, hh);
                if (m) {
                    const int mid = 32 * hh + 20;
                    const int rl = ((m >> mid) & 1ull) ? mid : (int)__builtin_ctzll(m);
                    xmins[hh] = __builtin_amdgcn_readlane(ox, rl) - (16 - F) / 2;
                    ymins[hh] = __builtin_amdgcn_readlane(oy, rl) - (16 - F) / 2;
                }
            }
            const uint32_t dx = (uint32_t)ox - (uint32_t)(h ? xmins[1] : xmins[0]);
            const uint32_t dy = (uint32_t)oy - (uint32_t)(h ? ymins[1] : ymins[0]);
            window = (ballot((dx > dy ? dx : dy) > (uint32_t)(16 - F)) & f.A) == 0;
        }
        bool fits[2] = {nAs[0] > 0, nAs[1] > 0};
        if ((kCollab || STATS) && f.A && !window) {
            int xmax[2], ymax[2];
            halves_reduce(inA ? ox : INT32_MAX, MinOp(), xmins[0], xmins[1]);
            halves_reduce(inA ? oy : INT32_MAX, MinOp(), ymins[0], ymins[1]);
            halves_reduce(inA ? ox + F - 1 : INT32_MIN, MaxOp(), xmax[0], xmax[1]);
            halves_reduce(inA ? oy + F - 1 : INT32_MIN, MaxOp(), ymax[0], ymax[1]);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                bbw[hh] = nAs[hh] ? xmax[hh] - xmins[hh] + 1 : 0;
                bbh[hh] = nAs[hh] ? ymax[hh] - ymins[hh] + 1 : 0;
                if (!nAs[hh]) xmins[hh] = ymins[hh] = 0;
                fits[hh] = nAs[hh] > 0 && bbw[hh] <= 16 && bbh[hh] <= 16;
            }
        }
        const int xmin = h ? xmins[1] : xmins[0], ymin = h ? ymins[1] : ymins[0];
        const int bw = h ? bbw[1] : bbw[0];
        const bool fits16 = h ? fits[1] : fits[0];

        // ---- distinct texels of the halves whose box fits 16x16
        WindowSet S[2] = {{0u, 0u, 0}, {0u, 0u, 0}};
        uint64_t B[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};   // tile records only
        const int corner = inA && fits16 ? 16 * (oy - ymin) + (ox - xmin) : 0;
        if ((kWindowed || STATS) && (fits[0] || fits[1])) {
            window_set_halves<F>(L.window, inA && fits16, h, corner, S);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                if constexpr (STATS) {
                    uint64_t C[4];
#pragma unroll
                    for (int w = 0; w < 4; ++w) C[w] = ballot(L.bytes(hh)[64 * w + lane] != 0);
                    footprint_mask_f<F>(C, B[hh]);
                }
                // h and h^-1 as tables
                reinterpret_cast<uint32_t*>(L.rank[hh])[lane] = S[hh].ranks;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (S[hh].set & (1u << (8 * q))) L.items[hh][(S[hh].ranks >> (8 * q)) & 0xffu] = (uint8_t)(4 * lane + q);
            }
            wave_lds_sync();
        }

        // ---- the method's decision, per half
        const int k = a.max_evals;
        HalfDecision D[2];
        bool sorted = false;
        int n0s = 0, ntot = 0;
        auto& seg = reinterpret_cast<SegmentScratch<F>&>(L.vals);
        const bool any_sort = (nAs[0] && !fits[0]) || (nAs[1] && !fits[1]);
        if constexpr (METHOD == CTF_LIST || STATS) {
            if (any_sort) {
                ntot = segment_sort(seg, L.first, inA && !fits16, (uint32_t)h, ox, oy, xmin, ymin, n0s);
                sorted = METHOD == CTF_LIST;
            }
        }
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            HalfDecision& d = D[hh];
            const int nseg = hh ? ntot - n0s : n0s;
            d.cap_ok = true;
            d.count_ok = true;
            d.success = false;
            d.n = 0;
            d.unique = fits[hh] ? S[hh].n : nAs[hh] ? nseg : 0;
            if constexpr (METHOD == CTF_BOX) {
                const int64_t area = (int64_t)bbw[hh] * bbh[hh];
                d.n = area > INT32_MAX ? INT32_MAX : (int)area;
                d.cap_ok = (a.box_w == 0 || bbw[hh] <= a.box_w) && (a.box_h == 0 || bbh[hh] <= a.box_h);
                d.count_ok = area <= (int64_t)k * nAs[hh];
                d.success = nAs[hh] > 0 && d.cap_ok && d.count_ok;
            } else if constexpr (METHOD == CTF_MASK) {
                d.cap_ok = fits[hh];
                d.n = fits[hh] ? S[hh].n : 0;
                d.count_ok = d.n <= k * nAs[hh];
                d.success = fits[hh] && d.count_ok;
            } else if constexpr (METHOD == CTF_LIST) {
                d.n = d.unique;
                d.count_ok = d.n <= k * nAs[hh];
                d.success = nAs[hh] > 0 && d.count_ok;
            }
        }
        const int n = h ? D[1].n : D[0].n;
        const bool success = h ? D[1].success : D[0].success;
        const bool half_sorted = sorted && nA > 0 && !fits16;
        if constexpr (METHOD == CTF_LIST) {
            if (sorted) {
                segment_emit(seg, [&](int i, int g, int dx, int dy) {
                    if (!(g ? D[1].success : D[0].success)) return;
                    const int2 c = make_int2((g ? xmins[1] : xmins[0]) + dx, (g ? ymins[1] : ymins[0]) + dy);
                    L.half[g].list[i - (g ? n0s : 0)] = c;
                });
                wave_lds_sync();
            }
        }

        const bool active = lane_in(f.act);
        bool exact, draws;
        if constexpr (METHOD == CTF_BILINEAR4) {
            exact = active;
            draws = false;
        } else if constexpr (METHOD == CTF_STF1) {
            exact = false;
            draws = active;
        } else {
            exact = inA && success;
            draws = active && !exact;
        }
        const uint64_t stfw = ballot(draws);

        // ---- production: each lane evaluates at most one texel per round
        float4 res = make_float4(0.f, 0.f, 0.f, 0.f);
        int2 pick = make_int2(INT32_MIN, INT32_MIN);
        uint32_t h1 = 0, h2 = 0;
        Footprint fl;
        fl.x0 = f.x0;
        fl.y0 = f.y0;
        fl.s = f.s;
        fl.t = f.t;
        if (draws) {
            stf_hashes(a.seed, a.layer, px, py, h1, h2);
            pick = stf_pick_filter<FILTER>(fl, h1, h2);
        }
        // fallback C / C+ for the lanes of A of a failed half
        bool fbl = false;
        W32Fallback P{};
        int nprod0 = 0, nprod1 = 0;
        if constexpr (FB && kCollab) {
            fbl = !success && nA > 0;
            if (ballot(fbl) != 0)
                P = plan_fallback_w32<FILTER, F>(L, a.fallback, fbl, inA, h, nA, rankA, fl, pick, pcg_hash(h2), fits16,
                                                  xmin, ymin, half_mask(~0ull, h), nprod0, nprod1);
        }
        if constexpr (METHOD == CTF_BILINEAR4) {
            if (exact) res = full_filter<FILTER, TEX>(T, terms_lds, joint, f.s, f.t, ox, oy, texel);
        } else {
            for (int round = 0; round < (kCollab ? k : 1); ++round) {
                // round 0 also evaluates the one-tap draws and the texels a
                // failed half planned, in the same pass as the other half's
                const int item = rankA + round * nA;
                const bool produce = kCollab && success && inA && item < n;
                const bool planned = FB && kCollab && round == 0 && fbl && inA && P.produces;
                const bool draw_now = draws && round == 0 && !(fbl && inA);
                if (ballot(produce || draw_now || planned) == 0) break;
                int2 e = planned ? P.texel : pick;
                if (produce) {
                    if constexpr (METHOD == CTF_BOX) {
                        e = make_int2(xmin + item % bw, ymin + item / bw);
                    } else if (half_sorted) {
                        e = L.half[h].list[item];
                    } else {
                        const int t = L.items[h][item];
                        e = make_int2(xmin + (t & 15), ymin + (t >> 4));
                    }
                    if (STATS && a.lists) reinterpret_cast<int2*>(a.lists)[(size_t)tile * kMaxItems + item] = e;
                }
                if (produce || draw_now || planned) {
                    const float4 v = texel(e.x, e.y);
                    if (produce || planned) L.vals[h][produce ? item : P.slot] = v;
                    if (draw_now) res = v;
                }
            }
            if constexpr (kCollab) {
                wave_lds_sync();
                if (FB && fbl && inA)
                    res = fallback_color_w32<FILTER, F>(L, P, h, h ? nprod1 : nprod0, fl, pick, xmin, ymin);
                if (exact) {
                    // first item of footprint row j; the row's other taps follow
                    auto row_item = [&](int j) -> int {
                        if constexpr (METHOD == CTF_BOX) return (ox - xmin) + (oy + j - ymin) * bw;
                        else return half_sorted ? L.first[F * lane + j] : L.rank[h][corner + 16 * j];
                    };
                    if constexpr (F == 2) {
                        const float4 *v0 = L.vals[h] + row_item(0), *v1 = L.vals[h] + row_item(1);
                        res = bilerp(f.s, f.t, v0[0], v0[1], v1[0], v1[1]);
                    } else {
                        float wx[4], wy[4];
                        taps32<FILTER>(f.s, wx);
                        taps32<FILTER>(f.t, wy);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float4* const v = L.vals[h] + row_item(j);
                            res = col_acc(wy[j], row4(wx, v[0], v[1], v[2], v[3]), res, j == 0);
                        }
                    }
                }
            }
        }

        // ---- outputs, per-tile records (lanes 0 and 32), frame counters
        {
            // unconditional: a lane off the screen repeats its tile's first
            // pixel, the pair's first tile if its own is past the last
            const int src = h && !tile_ok ? 0 : lane & 32;
            auto from = [&](float v) { return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * src, __float_as_int(v))); };
            float4 o = res;
            if (ballot(!in_screen) != 0) {
                const float4 e = make_float4(from(res.x), from(res.y), from(res.z), from(res.w));
                o = make_float4(in_screen ? res.x : e.x, in_screen ? res.y : e.y, in_screen ? res.z : e.z,
                                in_screen ? res.w : e.w);
            }
            const int ftx = h && !tile_ok ? cur.tx : tx, fty = h && !tile_ok ? cur.ty : ty;
            reinterpret_cast<float4*>(a.out)[in_screen ? pix : (int64_t)(fty * 4) * a.sw + ftx * 8] = o;
        }
        if (in_screen && a.stf_xy)
            reinterpret_cast<int2*>(a.stf_xy)[pix] = draws ? pick : make_int2(INT32_MIN, INT32_MIN);
        int evals[2];
        const uint32_t actm[2] = {lo32(f.act), hi32(f.act)}, stfm[2] = {lo32(stfw), hi32(stfw)};
        const uint32_t Am[2] = {lo32(f.A), hi32(f.A)};
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            if constexpr (METHOD == CTF_BILINEAR4) evals[hh] = F * F * __popc(actm[hh]);
            else if (FB && kCollab && !D[hh].success && __popc(Am[hh]) > 0)
                evals[hh] = (hh ? nprod1 : nprod0) + __popc(stfm[hh] & ~Am[hh]);
            else evals[hh] = (D[hh].success ? D[hh].n : 0) + __popc(stfm[hh]);
        }
        if (STATS && ll == 0 && tile_ok && a.tile_stats) {
            const HalfDecision& d = D[h];
            ctf_tile_stats S;
            S.active = actm[h];
            S.part = Am[h];
            S.stf = stfm[h];
            for (int w = 0; w < 4; ++w) S.mask[w] = fits16 ? B[h][w] : 0ull;
            S.xmin = xmin;
            S.ymin = ymin;
            S.bbw = bbw[h];
            S.bbh = bbh[h];
            S.n = d.n;
            S.unique = d.unique;
            S.evals = evals[h];
            S.flags = (d.success ? CTF_TILE_OK : 0) | (nA && !d.cap_ok ? CTF_TILE_CAP : 0) |
                      (nA && d.cap_ok && !d.count_ok ? CTF_TILE_OVERFLOW : 0) | (nA == 0 ? CTF_TILE_EMPTY : 0);
            for (int r = 0; r < 10; ++r) S.reserved[r] = 0;
            a.tile_stats[tile] = S;
        }
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
            if (actm[hh])
                fc.add(evals[hh], __popc(actm[hh]), __popc(stfm[hh]), __popc(actm[hh] & ~Am[hh]), 0,
                       kCollab && D[hh].success, kCollab && Am[hh] && !D[hh].success);
        wave_lds_sync();  // the next pair reuses this wave's LDS slice
    }
    if (a.frame_stats) fc.flush(a.frame_stats);
}

template <int METHOD, int TEX, int FILTER>
hipError_t launch_w32_m_t(const FilterArgs& a, const DevTexture& T, hipStream_t s)
{
    const int64_t npairs = (a.ntiles + 1) / 2;
    int64_t blocks = (npairs + kW32Waves - 1) / kW32Waves;
    if (blocks > (int64_t)a.cus * 8) blocks = (int64_t)a.cus * 8;
    const int64_t least = counter_min_blocks(a.ntiles, kW32Waves);   // 32-bit frame counters
    if (blocks < least) blocks = least;
    const dim3 grid((unsigned)blocks), block(kWave * kW32Waves);
    constexpr bool kCollab = METHOD == CTF_LIST || METHOD == CTF_BOX || METHOD == CTF_MASK;
    // the instantiation with statistics also writes the texel lists
    const bool st = a.tile_stats != nullptr || a.lists != nullptr;
    auto go = [&](auto lds) {
        constexpr bool LDS = decltype(lds)::value;
        if (kCollab && a.fallback != CTF_FB_STF1) {
            if (st) hipLaunchKernelGGL((k_filter_w32<METHOD, TEX, true, FILTER, kCollab, LDS>), grid, block, 0, s, a, T);
            else hipLaunchKernelGGL((k_filter_w32<METHOD, TEX, false, FILTER, kCollab, LDS>), grid, block, 0, s, a, T);
        } else {
            if (st) hipLaunchKernelGGL((k_filter_w32<METHOD, TEX, true, FILTER, false, LDS>), grid, block, 0, s, a, T);
            else hipLaunchKernelGGL((k_filter_w32<METHOD, TEX, false, FILTER, false, LDS>), grid, block, 0, s, a, T);
        }
    };
    if constexpr (kCollab && TEX == CTF_TEX_SINUSOIDS) {
        if (lds_terms(T)) go(std::true_type{});
        else go(std::false_type{});
    } else {
        go(std::false_type{});
    }
    return hipGetLastError();
}

template <int TEX, int FILTER>
hipError_t launch_w32_tf(const FilterArgs& a, const DevTexture& T, hipStream_t s)
{
    switch (a.method) {
    case CTF_BILINEAR4: return launch_w32_m_t<CTF_BILINEAR4, TEX, FILTER>(a, T, s);
    case CTF_STF1: return launch_w32_m_t<CTF_STF1, TEX, FILTER>(a, T, s);
    case CTF_LIST: return launch_w32_m_t<CTF_LIST, TEX, FILTER>(a, T, s);
    case CTF_BOX: return launch_w32_m_t<CTF_BOX, TEX, FILTER>(a, T, s);
    case CTF_MASK: return launch_w32_m_t<CTF_MASK, TEX, FILTER>(a, T, s);
    default: return hipErrorInvalidValue;
    }
}

template <int TEX>
hipError_t launch_w32_t(const FilterArgs& a, const DevTexture& T, hipStream_t s)
{
    switch (a.filter) {
    case CTF_FILTER_BILINEAR: return launch_w32_tf<TEX, CTF_FILTER_BILINEAR>(a, T, s);
    case CTF_FILTER_BSPLINE: return launch_w32_tf<TEX, CTF_FILTER_BSPLINE>(a, T, s);
    case CTF_FILTER_CATMULL_ROM: return launch_w32_tf<TEX, CTF_FILTER_CATMULL_ROM>(a, T, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_filter_w32(const FilterArgs& a, const DevTexture& T, hipStream_t s)
{
    switch (T.kind) {
    case CTF_TEX_SINUSOIDS: return launch_w32_t<CTF_TEX_SINUSOIDS>(a, T, s);
    case CTF_TEX_AFFINE: return launch_w32_t<CTF_TEX_AFFINE>(a, T, s);
    case CTF_TEX_CONSTANT: return launch_w32_t<CTF_TEX_CONSTANT>(a, T, s);
    case CTF_TEX_TABLE: return launch_w32_t<CTF_TEX_TABLE>(a, T, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ctf
