// Cuts on the host, by the functions that both planners use: from recorded shares of any contents every line is covered once, and no stretch is
// far from an equal one; the sizes of stretches that end with their request cover every request and stay within a third of an equal one.
#include <stdio.h>

#include <random>
#include <vector>

#include "../paper_2511_14617_amd/csrc/seer_plan.h"

using namespace seer;

static std::mt19937 rng(7);
static double uniform(double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(rng); }

// The sums of rates, as the combine kernel records them.
static std::vector<uint32_t> recorded(int W, double lo, double hi) {
    std::vector<float> rate(W);
    float all = 0.f, before = 0.f;
    for (float& r : rate) r = static_cast<float>(uniform(lo, hi)), all += r;
    std::vector<uint32_t> s(kHistoryStride, 0xdeadbeefu);
    for (int w = 0; w < W; ++w) {
        s[w] = static_cast<uint32_t>(std::min(before / all, 0.99999994f) * 4294967296.f);
        before += rate[w];
    }
    return s;
}

int main() {
    int used = 0, refused = 0;
    for (int W : {2, 3, 7, 31, 32, 64, 100, 128, 255, 256, 511, 512, 513, 1000, 1024}) {
        AttnArgs a{};
        a.wgs_per_head = W, a.inv_wgs = reciprocal(W), a.max_splits = 256, a.inv_splits = reciprocal(255), a.min_tiles = 1, a.fine_pieces = 1 << 28;
        for (int kind = 0; kind < 9; ++kind)
            for (int rep = 0; rep < 40; ++rep) {
                std::vector<uint32_t> s = recorded(W, 0.75, 4. / 3.);
                const int at = static_cast<int>(rng() % W);
                if (kind == 1) s = recorded(W, 1., 1.);
                if (kind == 2)                                                   // the widest spread: one kind of rate, then the other
                    for (int w = 0; w < W; ++w) s[w] = static_cast<uint32_t>(4294967296. * (w <= at ? w * .75 : at * .75 + (w - at) * 4. / 3.) / (at * .75 + (W - at) * 4. / 3.));
                if (kind == 3) for (uint32_t& x : s) x = rng();                  // anything
                if (kind == 4) s[at] = rng();                                    // one word of anything
                if (kind == 5) for (int w = 0; w < W; ++w) s[w] = 0x3c000000u + (rng() & 0xffffffu);      // floating-point numbers near another
                if (kind == 6) for (int w = 0; w < W; ++w) s[w] = w * (a.inv_wgs + a.inv_wgs / 4 + a.inv_wgs / 8 + a.inv_wgs / 2);   // beyond the line
                if (kind == 7) for (int w = 0; w < W; ++w) s[w] = 0u - w * a.inv_wgs;                      // falling
                if (kind == 8) for (uint32_t& x : s) x += 1u << (rng() % 32);                              // not from 0 on
                bool usable = true;
                for (int w = 0; w < W; ++w) usable &= share_ok(a, w, s[w], s[w + 1]);
                if (kind < 3 && !usable) return printf("W %d kind %d: refused\n", W, kind), 1;
                usable ? ++used : ++refused;
                const int total = static_cast<int>(8 * W * std::exp2(uniform(0., 10.)));
                const Cut cut = cut_of(a, total, total);
                if (!cut.weighted) continue;
                int prev = 0;
                for (int w = 0; w < W; ++w) {
                    const int begin = cut_begin(cut, w, usable ? s[w] : equal_before(a, w));
                    const int end = cut_begin(cut, w + 1, usable ? s[w + 1] : equal_before(a, w + 1));
                    const double equal = static_cast<double>(total) / W;
                    if (begin != prev || end < begin || end - begin < equal / 2 - 2 || end - begin > equal * 15 / 8 + 2)
                        return printf("W %d kind %d total %d stretch %d: %d .. %d behind %d\n", W, kind, total, w, begin, end, prev), 1;
                    prev = end;
                }
                if (prev != total) return printf("W %d kind %d: ends at %d of %d\n", W, kind, prev, total), 1;
            }
    }
    // short lines: stretches of one size that end with their request
    int whole = 0, one_more = 0;
    for (int W : {1, 2, 31, 128, 256, 512, 1024})
        for (int rep = 0; rep < 2000; ++rep) {
            AttnArgs a{};
            a.wgs_per_head = W, a.inv_wgs = reciprocal(W), a.max_splits = rep % 3 ? 256 : 2 + static_cast<int>(rng() % 255), a.inv_splits = reciprocal(a.max_splits - 1);
            a.min_tiles = rep % 2 ? 1 : 4, a.fine_pieces = 1 << 28, a.B = 1 + static_cast<int>(rng() % kWholeRequests);
            std::vector<int> tiles(a.B);
            int total = 0, longest = 0;
            for (int& t : tiles) t = static_cast<int>(rng() % 5 ? std::exp2(uniform(0., 7.)) : 0), total += t, longest = std::max(longest, t);
            const Cut cut = cut_of(a, total, longest);
            if (cut.weighted || cut.equal < 2) continue;
            for (Cut tried = cut; tried.equal <= longest_whole(cut); ++tried.equal) {
                int used = 0, pieces = 0;
                for (int t : tiles) {
                    const int own = stretches_of(tried, t);
                    if (own * tried.equal < t || (own - 1) * tried.equal >= std::max(t, 1)) return printf("%d tiles in %d of %d\n", t, own, tried.equal), 1;
                    used += own, pieces = std::max(pieces, own);
                }
                if (pieces > a.max_splits || 3 * tried.equal > 4 * cut.equal + 2 * (cut.equal < 3)) return printf("%d pieces, %d for %d tiles\n", pieces, tried.equal, cut.equal), 1;
                if (used <= W) {
                    tried.equal == cut.equal ? ++whole : ++one_more;
                    break;
                }
            }
        }
    if (whole < 300 || one_more < 30) return printf("whole %d, one more %d\n", whole, one_more), 1;
    printf("used %d refused %d\n", used, refused);
    return used > 1000 && refused > 1000 ? 0 : 1;
}
