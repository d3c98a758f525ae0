// The texel sets of csrc/ctf_device.h (segment_sort and segment_emit,
// window_set, window_set_halves) against std::set, lane by lane.
#include "ctf_device.h"

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <random>
#include <set>
#include <utility>
#include <vector>

Dim threadIdx, blockIdx, blockDim, gridDim;

namespace wave {
int lane;
uint64_t slot[kLanes];
static ucontext_t ctx[kLanes], home;
static char stack[kLanes][1 << 16];
static bool done[kLanes];
static std::function<void()> body;

void step()
{
    const int self = lane;
    lane = (self + 1) % kLanes;
    swapcontext(&ctx[self], &ctx[lane]);
    lane = self;
}

static void entry()
{
    const int self = lane;
    body();
    done[self] = true;
    lane = self + 1;   // the lanes end in order: every lane takes the same steps
    if (lane == kLanes) setcontext(&home);
    setcontext(&ctx[lane]);
}

static void run(std::function<void()> f)
{
    body = std::move(f);
    for (int l = 0; l < kLanes; ++l) {
        done[l] = false;
        getcontext(&ctx[l]);
        ctx[l].uc_stack.ss_sp = stack[l];
        ctx[l].uc_stack.ss_size = sizeof stack[l];
        ctx[l].uc_link = nullptr;
        makecontext(&ctx[l], entry, 0);
    }
    lane = 0;
    swapcontext(&home, &ctx[0]);
    for (int l = 0; l < kLanes; ++l)
        if (!done[l]) { std::printf("lane %d did not end\n", l); std::exit(1); }
}
}  // namespace wave

using Texel = std::pair<int, int>;   // (y, x): the list's order
using Set = std::vector<Texel>;

static void check(bool ok, const char* what, int F, int id)
{
    if (ok) return;
    std::printf("%s: F = %d, case %d\n", what, F, id);
    std::exit(1);
}

struct Lane {
    bool in;
    int group, x, y;   // upper-left tap
};

template <int F>
static Set set_of(const Lane* L, int group)
{
    std::set<Texel> s;
    for (int l = 0; l < 64; ++l)
        if (L[l].in && (group < 0 || L[l].group == group))
            for (int r = 0; r < F; ++r)
                for (int c = 0; c < F; ++c) s.insert({L[l].y + r, L[l].x + c});
    return Set(s.begin(), s.end());
}

// Sorted segments: counts, every lane's first items, the emitted list.
template <int F>
static void segments(const Lane* L, int id)
{
    static ctf::SegmentScratch<F> S;
    static uint8_t first[256];
    int xmin[2], ymin[2];
    for (int g = 0; g < 2; ++g) {
        xmin[g] = ymin[g] = INT32_MAX;
        for (int l = 0; l < 64; ++l)
            if (L[l].in && L[l].group == g) {
                xmin[g] = L[l].x < xmin[g] ? L[l].x : xmin[g];
                ymin[g] = L[l].y < ymin[g] ? L[l].y : ymin[g];
            }
    }
    const Set set[2] = {set_of<F>(L, 0), set_of<F>(L, 1)};
    const int n = (int)(set[0].size() + set[1].size()), n0 = (int)set[0].size();
    int got_n[64], got_n0[64];
    std::vector<int> written(n, 0);
    std::vector<Texel> out(n);
    wave::run([&] {
        const int l = wave::lane, g = L[l].group;
        got_n[l] = ctf::segment_sort(S, first, L[l].in, (uint32_t)g, L[l].x, L[l].y, xmin[g], ymin[g], got_n0[l]);
        ctf::segment_emit(S, [&](int i, int group, int dx, int dy) {
            check(i >= 0 && i < n && (i >= n0) == (group == 1), "item outside its group's list", F, id);
            ++written[i];
            out[i] = {ymin[group] + dy, xmin[group] + dx};
        });
    });
    for (int l = 0; l < 64; ++l) check(got_n[l] == n && got_n0[l] == n0, "counts", F, id);
    for (int i = 0; i < n; ++i) {
        check(written[i] == 1, "an item written once", F, id);
        check(out[i] == (i < n0 ? set[0][i] : set[1][i - n0]), "the list", F, id);
    }
    for (int l = 0; l < 64; ++l) {
        const Set& s = set[L[l].group];
        if (!L[l].in || s.size() > 256) continue;   // bytes hold the items of a list that succeeds
        for (int r = 0; r < F; ++r) {
            const size_t i = first[F * l + r];
            check(i + F <= s.size() && s[i] == Texel(L[l].y + r, L[l].x), "a row's first item", F, id);
        }
    }
}

// A window's set: positions 16 y + x, and their ranks.
static void window_result(const ctf::WindowSet* S, const Set& set, int F, int id)
{
    size_t seen = 0;
    for (int p = 0; p < 256; ++p) {
        const ctf::WindowSet& w = S[p / 4];
        const int shift = 8 * (p % 4);
        const bool need = w.set >> shift & 1;
        check(w.n == (int)set.size(), "window count", F, id);
        if (!need) continue;
        check(seen < set.size() && set[seen] == Texel(p / 16, p % 16), "window set", F, id);
        check((w.ranks >> shift & 255) == seen, "window rank", F, id);
        ++seen;
    }
    check(seen == set.size(), "window set", F, id);
}

template <int F>
static void windows(const Lane* L, int id)
{
    static uint32_t words[2 * ctf::kWindowWords];
    for (int i = 0; i < ctf::kWindowPad; ++i) words[i] = words[ctf::kWindowWords + i] = 0;
    ctf::WindowSet one[64], two[2][64];
    wave::run([&] {
        const int l = wave::lane, corner = L[l].in ? 16 * L[l].y + L[l].x : 0;
        one[l] = ctf::window_set<F>(words, L[l].in, corner);
        ctf::wave_lds_sync();
        ctf::WindowSet h[2];
        ctf::window_set_halves<F>(words, L[l].in, l >> 5, corner, h);
        two[0][l] = h[0];
        two[1][l] = h[1];
    });
    Lane half[64];
    for (int l = 0; l < 64; ++l) half[l] = Lane{L[l].in, l >> 5, L[l].x, L[l].y};
    window_result(one, set_of<F>(L, -1), F, id);
    for (int h = 0; h < 2; ++h) window_result(two[h], set_of<F>(half, h), F, id);
}

template <int F>
static void all(int cases, std::mt19937& rng)
{
    auto pick = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
    for (int id = 0; id < cases; ++id) {
        Lane L[64];
        // spread of the corners: one point, neighbours within a footprint, a
        // window, past it, the whole range of positions
        static const int spread[] = {0, 1, F, 16 - F, 24, 60, 400, (1 << 24) - 1};
        const int s = spread[id % 8], ox = pick(-50, 50), oy = pick(-50, 50), few = pick(0, 3);
        const int rows = pick(0, 1) ? s : pick(0, 3);   // long rows of overlapping segments
        for (int l = 0; l < 64; ++l) {
            L[l].in = few == 0 ? l == id % 64 : few == 1 ? true : pick(0, few) > 0;
            L[l].group = id % 3 == 0 ? l >> 5 : id % 3 == 1 ? 0 : pick(0, 1);
            L[l].x = s > 400 ? pick(-s, s) : ox + pick(0, s);
            L[l].y = s > 400 && rows == s ? pick(-s, s) : oy + pick(0, rows);
        }
        segments<F>(L, id);
        for (int l = 0; l < 64; ++l) {
            L[l].x = pick(0, s < 16 - F ? s : 16 - F);
            L[l].y = pick(0, rows < 16 - F ? rows : 16 - F);
        }
        if (id % 5 == 0)   // every texel of the window: 256 items
            for (int l = 0; l < 64; ++l) L[l] = Lane{true, 0, l % 8 * (16 - F) / 7, l / 8 * (16 - F) / 7};
        windows<F>(L, id);
    }
}

int main()
{
    std::mt19937 rng(1);
    all<2>(400, rng);
    all<4>(400, rng);
    std::puts("ok");
}
