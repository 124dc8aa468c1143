// The division of the learned scorers' half strips among waves, without a GPU:
// every wave of a launch is replayed by the functions that the kernels use.
// Test infrastructure only.
#include "ca_deal.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

using namespace ca;

namespace {

struct Size {
    int32_t W, H, first, count;
};

#define CHECK(c)                                                                            \
    do {                                                                                    \
        if (!(c)) {                                                                         \
            std::printf("FAIL %s:%d %s\n", __FILE__, __LINE__, #c);                          \
            std::exit(1);                                                                   \
        }                                                                                   \
    } while (0)

int steps_for(int positions, int halo) { return (positions + 2 * halo + kStep - 1) / kStep; }

// Steps of the last wave; every position of every half strip is taken once, in
// turn, and no piece needs more steps than it was dealt (but one, where shares are
// longer than the half strip).
int replay(const std::vector<Size> &sizes, int frames, int n_all, int n_h, int n_v, int resident,
           int halo, double *mean)
{
    StripDeal d = strip_deal(sizes.data(), (int)sizes.size(), frames, n_all, n_h, n_v,
                                   resident, halo);
    CHECK(d.groups >= 1 && d.groups <= std::min(resident, kStripGroups / kXcds));
    const int groups = kXcds * d.groups, waves = kStripWaves * groups;
    std::vector<std::pair<int, int>> halves;   // length, entries, in the list's order
    for (const Size &s : sizes) {
        if (sizes.size() > 1) {   // as the kernel counts them
            d.row = extent_entries(s.W, halo, d);
            d.col = extent_entries(s.H, halo, d);
        }
        const int each = 2 * (n_h * d.row + n_v * d.col);
        for (int f = 0; f < s.count; ++f) {
            std::vector<char> seen((size_t)2 * (n_h + n_v), 0);
            StripPlace next = strip_place(d, n_h, n_v, 0);
            for (int at = 0; at < each;) {
                const StripPlace p = strip_place(d, n_h, n_v, at);
                CHECK(p.at == 0 && p.half >= 0 && p.half < 2
                      && p.strip < (p.horizontal ? n_h : n_v)
                      && p.entries == (p.horizontal ? d.row : d.col));
                CHECK(next.strip == p.strip && next.half == p.half && next.at == 0
                      && next.horizontal == p.horizontal && next.entries == p.entries);
                char &once = seen[(size_t)2 * (p.horizontal ? p.strip : n_h + p.strip) + p.half];
                CHECK(!once);
                once = 1;
                const int L = p.horizontal ? s.W : s.H;
                halves.push_back({p.half ? L - (L >> 1) : L >> 1, p.entries});
                const StripPlace last = strip_place(d, n_h, n_v, at + p.entries - 1);
                CHECK(last.strip == p.strip && last.half == p.half
                      && last.horizontal == p.horizontal && last.at == p.entries - 1);
                at += p.entries;
                CHECK(strip_next(d, n_h, n_v, next) == (at < each));
            }
            const StripPlace first = strip_place(d, n_h, n_v, 0);
            CHECK(next.strip == 0 && next.half == 0 && next.horizontal == first.horizontal);
            for (const char once : seen)
                CHECK(once);
        }
    }
    int64_t total = 0;
    for (const auto &h : halves)
        total += h.second;
    if (sizes.size() == 1) {
        CHECK(d.each == 2 * (n_h * d.row + n_v * d.col) && (int64_t)d.each * frames == total);
    } else {
        CHECK(d.each == 0);
        d.share = (int)(total / groups);
        d.extra = (int)(total % groups);
    }
    CHECK((int64_t)d.share * groups + (int64_t)d.extra * d.more == total);
    int unit = 0, at = 0, done = 0, worst = 0;
    int64_t start = 0;   // of the unit
    for (int w = 0; w < waves; ++w) {
        int64_t t = wave_start(d, w);
        const int64_t end = wave_start(d, w + 1);
        CHECK(end - t <= (total + waves - 1) / waves);
        int used = 0;
        while (t < end) {
            CHECK(t == start + at && wave_of(d, (int)t) == w);
            const int len = halves[unit].first, s = halves[unit].second;
            const int take = (int)std::min<int64_t>(s - at, end - t);
            const int from = at ? wave_of(d, (int)start) : w;
            auto start_of = [&](int entry, int waves_on) {
                return piece_start(len, halo, entry, cuts_before(d.share, entry, waves_on), d.grain);
            };
            const int p0 = at ? start_of(at, w - from) : 0;
            const int p1 = at + take == s ? len : start_of(at + take, w - from + 1);
            CHECK(p0 == done && p1 >= p0);
            const int steps = p1 > p0 ? steps_for(p1 - p0, halo) : 0;
            if (d.cut == 0)
                CHECK(steps <= take * d.grain && (take == 1 || frames < n_all));
            else if (d.share / kStripWaves >= d.cut)
                CHECK(steps <= take + (s <= d.cut ? 1 : 0));
            used += steps;
            done = p1;
            t += take;
            at += take;
            if (at == s) {
                CHECK(done == len);
                start += s;
                ++unit;
                at = done = 0;
            }
        }
        worst = std::max(worst, used);
    }
    CHECK(unit == (int)halves.size());
    // steps without any cut, over the device's waves
    int64_t whole = 0;
    for (const auto &h : halves)
        whole += steps_for(h.first, halo);
    *mean = (double)whole / (kXcds * kStripWaves * std::min(resident, kStripGroups / kXcds));
    return worst;
}

// The last wave's steps where a workgroup's waves share every half strip evenly,
// `parts` to each, and the half strips are taken in turns of resident workgroups.
int by_turns(const Size &s, int n, int n_h, int n_v, int resident, int halo, int parts)
{
    const int S = n_h + n_v, items = n * S, per_xcd = (items + 7) / 8;
    const int sets = kStripWaves / parts;
    const int groups = std::min(resident, (2 * per_xcd + sets - 1) / sets), slots = groups * sets;
    int worst = 0;
    for (int x = 0; x < 8; ++x) {
        const int units = 2 * (std::min((x + 1) * per_xcd, items) - x * per_xcd);
        std::vector<int> load((size_t)slots, 0);
        for (int turn = 0; turn * slots < units; ++turn)
            for (int k = 0; k < slots; ++k) {
                const int unit = turn * slots + (k + turn * S) % slots;
                if (unit >= units)
                    continue;
                const int L = (x * per_xcd + (unit >> 1)) % S < n_h ? s.W : s.H;
                const int len = L - (L >> 1);
                load[(size_t)k] += steps_for((len + parts - 1) / parts, halo);
            }
        worst = std::max(worst, *std::max_element(load.begin(), load.end()));
    }
    return worst;
}

}  // namespace

int main()
{
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return (int)(lo + rng() % (uint32_t)(hi - lo + 1)); };
    double mean;
    int slower = 0, batches = 0;
    auto one = [&](int W, int H, int n, int n_h, int n_v, int resident, int halo) {
        const Size s = {W, H, 0, n};
        const int got = replay({s}, n, n, n_h, n_v, resident, halo, &mean);
        int best = 1 << 30;
        for (int parts = 1; parts <= 8; parts *= 2)
            best = std::min(best, by_turns(s, n, n_h, n_v, std::min(resident, 32), halo, parts));
        if (got > best)
            ++slower;
        // whole steps, of which a cut's halo may take one more
        if (got > 1.2 * mean + 2) {
            std::printf("FAIL %d x %dx%d, %d + %d strips, halo %d: %d steps, mean %.2f, turns %d\n",
                        n, W, H, n_h, n_v, halo, got, mean, best);
            std::exit(1);
        }
        ++batches;
    };
    for (int halo : {3, 8}) {
        for (int n : {1, 2, 7, 16, 64})
            for (int strips : {16, 32})
                for (auto wh : {std::make_pair(1920, 1080), std::make_pair(2142, 1416),
                                std::make_pair(640, 480), std::make_pair(3162, 1867)})
                    one(wh.first, wh.second, n, strips, strips, 32, halo);
        for (int k = 0; k < 4000; ++k)
            one(pick(16, k % 10 ? 4096 : 16384), pick(16, k % 10 ? 2400 : 16384), pick(1, 20),
                pick(0, 64), pick(1, 64), k % 7 ? 32 : pick(1, 40), halo);
        // several shapes, of a batch or (the launch counts for itself) a part of one
        for (int k = 0; k < 500; ++k) {
            std::vector<Size> sizes;
            int n = 0;
            for (int j = pick(2, 6); j > 0; --j) {
                sizes.push_back({pick(16, 4096), pick(16, 2400), 0, pick(1, 12)});
                n += sizes.back().count;
            }
            const int n_h = pick(0, 40), n_v = pick(1, 40);
            const int got = replay(sizes, n, n, n_h, n_v, 32, halo, &mean);
            CHECK(got <= 1.2 * mean + 2);
            replay(sizes, std::max(1, n / 2), n, n_h, n_v, 32, halo, &mean);
        }
    }
    std::printf("%d of %d batches take more steps than the best of turns\n", slower, batches);
    CHECK(100 * slower <= batches);
    std::printf("ok deal\n");
    return 0;
}
