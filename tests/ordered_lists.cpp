// The point lists of the frame setup and the update as their workgroups write
// them (csrc/ordered.h), on the host: a workgroup per part, counts published
// in words that may hold another launch's, waits that may expire.  Every
// position has to lie inside its list; complete lists have to be in order.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <vector>

#include "ordered.h"

using namespace rose;

static int failures = 0;
#define EXPECT(c)                                                   \
    do {                                                            \
        if (!(c) && ++failures < 20) printf("line %d: %s\n", __LINE__, #c); \
    } while (0)

// one list of su x sv samples in 8x8 tiles; keep[q]: whether sample q is valid
struct Grid {
    int su, sv, cap, padded, parts;
    Grid(int W, int H, int stride) {
        su = (W + stride - 1) / stride;
        sv = (H + stride - 1) / stride;
        cap = su * sv;
        padded = ((su + 7) / 8) * ((sv + 7) / 8) * 64;
        parts = (padded + kPartPoints - 1) / kPartPoints;
    }
    bool inside(int q) const {
        const int ntx = (su + 7) / 8, t = q / 64, e = q % 64;
        return q < padded && (t % ntx) * 8 + e % 8 < su && (t / ntx) * 8 + e / 8 < sv;
    }
};

struct Lists {
    std::vector<int> first, second;  // elements written, -1 where none
    int n_first = 0, n_second = 0;
    bool lost = false;
};

// counts_before of parts [p0, p1): a part whose word is another launch's makes the wait expire
static uint64_t before(const std::vector<uint64_t>& words, uint64_t tag, int p0, int p1) {
    uint64_t sum = 0;
    for (int p = p0; p < p1; ++p) {
        if (!part_published(words[p], tag)) return kCountsLost;
        sum += part_counts(words[p]);
    }
    return sum;
}

// the parts of `g` for which held[p], of a launch with `tag`; fraction: share of valid samples
static Lists write_lists(const Grid& g, std::vector<uint64_t>& words, uint64_t tag, const std::vector<bool>& held,
                         double fraction, std::mt19937& rng) {
    Lists out;
    out.first.assign(g.cap, -1);
    out.second.assign(g.cap, -1);
    std::vector<int> keep(g.padded, 0);
    std::uniform_real_distribution<double> u(0, 1);
    for (int q = 0; q < g.padded; ++q) keep[q] = g.inside(q) && u(rng) < fraction ? (u(rng) < 0.5 ? 2 : 1) : 0;
    auto count = [&](int p, int least) {
        int n = 0;
        for (int q = p * kPartPoints; q < std::min(g.padded, (p + 1) * kPartPoints); ++q) n += keep[q] >= least;
        return (uint32_t)n;
    };
    for (int p = 0; p < g.parts; ++p)
        if (held[p]) words[p] = part_word(tag, count(p, 1), count(p, 2));
    for (int p = 0; p < g.parts; ++p) {
        if (!held[p]) continue;
        const uint64_t b = before(words, tag, 0, p);
        out.lost = out.lost || b == kCountsLost;
        int pos[2] = {0, 0};
        for (int q = p * kPartPoints; q < std::min(g.padded, (p + 1) * kPartPoints); ++q)
            for (int w = 0; w < keep[q]; ++w) {
                const int at = list_slot(b, w, pos[w]++, g.cap);
                EXPECT(at >= -1 && at < g.cap);
                if (at >= 0 && at < g.cap) (w ? out.second : out.first)[at] = q;
            }
        if (p == g.parts - 1) {
            const uint64_t all = before(words, tag, 0, g.parts);
            out.lost = out.lost || all == kCountsLost;
            out.n_first = list_size(all, 0, g.cap);
            out.n_second = list_size(all, 1, g.cap);
            EXPECT(out.n_first >= 0 && out.n_first <= g.cap && out.n_second >= 0 && out.n_second <= g.cap);
        }
    }
    if (!out.lost && std::count(held.begin(), held.end(), true) == g.parts) {  // whole lists, in order
        std::vector<int> a, c;
        for (int q = 0; q < g.padded; ++q) {
            if (keep[q] >= 1) a.push_back(q);
            if (keep[q] >= 2) c.push_back(q);
        }
        EXPECT(out.n_first == std::min((int)a.size(), g.cap) && std::equal(a.begin(), a.end(), out.first.begin()));
        EXPECT(out.n_second == (int)c.size() && std::equal(c.begin(), c.end(), out.second.begin()));
    }
    return out;
}

int main() {
    std::mt19937 rng(5);
    const int sizes[][3] = {{804, 600, 4}, {640, 480, 4}, {160, 120, 3}, {641, 7, 1}, {1, 4000, 1}, {320, 240, 2}};
    for (auto& z : sizes) {
        const Grid g(z[0], z[1], z[2]);
        const std::vector<bool> all(g.parts, true);
        std::vector<uint64_t> words(4096, 0);
        // two frames in turn: every count, from nothing to everything
        for (uint64_t launch = 0; launch < 4; ++launch)
            EXPECT(!write_lists(g, words, launch_tag(launch), all, launch / 3.0, rng).lost);
        // full words of the step of an earlier frame (1024 points each) in which some parts never publish
        for (int miss = 0; miss < g.parts; ++miss) {
            std::fill(words.begin(), words.end(), part_word(launch_tag(8), 1024, 1024));
            std::vector<bool> held = all;
            held[miss] = false;
            const Lists l = write_lists(g, words, launch_tag(9), held, 1.0, rng);
            EXPECT(l.lost || miss == g.parts - 1);
        }
        // words that another camera's launch published under the same tag: any counts
        for (int rep = 0; rep < 8; ++rep) {
            std::vector<bool> held(g.parts);
            for (int p = 0; p < g.parts; ++p) {
                held[p] = rng() % 2;
                words[p] = part_word(launch_tag(20), rng() % 1025, rng() % 1025);
            }
            write_lists(g, words, launch_tag(20), held, 1.0, rng);
        }
    }
    // the largest sums: 4096 parts of 1024 in both counts stay apart
    uint64_t sum = 0;
    for (int p = 0; p < 4096; ++p) sum += part_counts(part_word(launch_tag(1ull << 40), 1024, 1024));
    EXPECT(list_slot(sum, 0, 0, 1 << 30) == 4096 * 1024 && list_slot(sum, 1, 5, 1 << 30) == 4096 * 1024 + 5);
    EXPECT(list_size(sum, 0, 100) == 100 && list_size(kCountsLost, 0, 100) == 0 && list_size(kCountsLost, 1, 100) == 0);
    printf(failures ? "%d failures\n" : "ok\n", failures);
    return failures != 0;
}
