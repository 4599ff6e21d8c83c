// The cut of a question's key tiles into ranges (tile_ranges.hpp), on the CPU: random batches over the chip's slot counts,
// part limits and weights, among them one long dialogue between two short ones.  Checked for every batch:
//   * the ranges tile [0, total), none is empty, there are at most `slots` of them;
//   * at most max_parts ranges meet one sequence: the partial results of a row have room for that many and no more;
//   * sequences cut by themselves have at most max_parts pieces, at most `slots` together, which tile every sequence.
// And the number of ranges that launches of many query rows are given.
//
// usage: tile_ranges [seed] [cases]     exit status 0 = every check passed
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "tile_ranges.hpp"

using namespace ra;

static int bad = 0, weighted = 0, apart = 0;
static long long n_checked = 0;

template <int C>
static void check(const std::vector<int>& U, int slots, int min_tiles, int max_parts, bool full, const RangeWeights<C>& weights) {
    int total = 0, most = 0;
    for (int u : U) {
        total += u;
        most = u > most ? u : most;
    }
    if (slots > kMaxRanges) slots = kMaxRanges;
    const TileCut<C> cut(total, most, slots, min_tiles, max_parts, full, weights);
    ++n_checked;
    auto report = [&](const char* what, int b, int n) {
        if (++bad <= 10)
            std::fprintf(stderr, "  %s: sequence %d (%d tiles) %d, of %d tiles, %d slots, max_parts %d, %d classes, full %d\n", what, b,
                         b < 0 ? 0 : U[b], n, total, slots, max_parts, C, (int)full);
    };
    for (int len = cut.len; len <= cut.longest_apart((int)U.size()); ++len) {
        int n_apart = 0;
        for (int u : U) n_apart += cut.cuts(u, len);
        if (!cut.apart(n_apart, slots)) continue;
        ++apart;
        for (size_t b = 0; b < U.size(); ++b) {
            const int n = cut.cuts(U[b], len);
            if (n > max_parts) report("pieces of a sequence cut by itself", (int)b, n);
            for (int j = 0; j < n; ++j) {
                const int lo = piece_begin(U[b], j, n), hi = j + 1 < n ? piece_begin(U[b], j + 1, n) : U[b];
                if ((j == 0 && lo != 0) || lo >= hi || hi > U[b] || hi - lo > len) report("a piece of a sequence cut by itself", (int)b, j);
            }
        }
        return;
    }
    const double per_weight = cut.tiles_per_weight();
    if (cut.n_ranges > slots || cut.begin(0, per_weight) != 0 || cut.begin(cut.n_ranges, per_weight) != total)
        report("ranges do not tile the batch", -1, cut.n_ranges);
    bool unequal = false;
    for (int k = 0; k < C; ++k) unequal |= cut.w[k] != cut.w[0];
    if (unequal && (!full || cut.n_ranges != slots || cut.n_ranges % C)) report("unequal ranges where the classes are not even", -1, cut.n_ranges);
    weighted += unequal;
    if (total == 0) return;
    std::vector<int> begin;
    for (int r = 0; r <= cut.n_ranges; ++r) begin.push_back(cut.begin(r, per_weight));
    for (int r = 0; r < cut.n_ranges; ++r)
        if (begin[r] >= begin[r + 1]) report("empty range", -1, r);
    int lo = 0;
    for (size_t b = 0; b < U.size(); lo += U[b++]) {
        if (U[b] == 0) continue;
        int parts = 0;
        for (int r = 0; r < cut.n_ranges; ++r) parts += begin[r] < lo + U[b] && begin[r + 1] > lo;
        if (parts > max_parts) report("parts of a sequence", (int)b, parts);
    }
}

// Both kernels, and the shortest ranges of their launches.  The score kernel's limit is lifted where there are no more ranges.
static void check_both(const std::vector<int>& U, int slots, int max_parts, bool full) {
    for (int min_tiles : {2, 8}) {
        check(U, slots, min_tiles, max_parts, full, attn_range_weights());
        check(U, slots, min_tiles, max_parts >= slots ? kMaxRanges + 2 : max_parts, full, score_range_weights());
    }
}

// The limit that a launch asks for: what it costs is at most that ranges shorter than eight tiles have eight, and nothing where two
// dialogues or one share the ranges.
static void check_parts(const std::vector<int>& U, int slots, int slack) {
    int total = 0, most = 0;
    for (int u : U) {
        total += u;
        most = u > most ? u : most;
    }
    if (slots > kMaxRanges) slots = kMaxRanges;
    const int bound = most + slack, B = (int)U.size();
    if (bound < 2) return;  // (room for two parts is left to launches that are planned apart)
    const int S = question_parts(bound / 2 + 2, (bound + 7) / 8 + 2, slots, B);
    const int max_parts = S >= slots ? kMaxRanges + 2 : S;
    if (S < 1 || S > slots || (B <= 2 && S != std::min(bound / 2 + 2, slots)) || max_parts < 3) ++bad;
    if (max_parts < 3) return;
    check(U, slots, 2, max_parts, true, score_range_weights());
    const TileCut<3> cut(total, most, slots, 2, max_parts, false, score_range_weights()), free(total, most, slots, 2, kMaxRanges + 2, false, score_range_weights());
    if (cut.len > std::max(8, free.len) && ++bad <= 10) std::fprintf(stderr, "  ranges of %d tiles instead of %d by the limit %d\n", cut.len, free.len, S);
}

int main(int argc, char** argv) {
    const unsigned seed = argc > 1 ? (unsigned)std::atoi(argv[1]) : 1u;
    const int cases = argc > 2 ? std::atoi(argv[2]) : 20000;
    std::mt19937 rng(seed);
    auto uni = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    check_both({100, 1500, 100}, 19, 18, true);
    check_both({21, 320, 21}, 19, 18, true);
    check_both({90, 44, 2239, 3, 146}, 19, 18, true);
    check_both({30, 392, 30}, 17, 16, true);
    // the largest sequences and the most ranges there are
    for (int slots : {384, 768, kMaxRanges}) {
        check_both({5700000, 5700000}, slots, kMaxRanges + 2, false);
        check_both({(1 << 24) - 1, (1 << 24) - 1}, slots, kMaxRanges + 2, false);
        check_both({(1 << 24) - 1, 1, 16000000, 12345678}, slots, kMaxRanges + 2, false);
    }
    // one long dialogue between two short ones, every slot count and part limit near each other
    for (int slots = 3; slots <= 40; ++slots)
        for (int max_parts = 3; max_parts <= 18; ++max_parts)
            for (int k = 0; k < 40; ++k) {
                const int most = uni(8 * max_parts, 200 * max_parts), side = uni(0, most / 4);
                check_both({side, most, uni(0, 1) ? side : uni(0, most / 4)}, slots, max_parts, true);
            }
    for (int c = 0; c < cases; ++c) {
        const int B = uni(1, kInlineBatch), style = uni(0, 4), slots = uni(1, style == 3 ? 1500 : 64);
        std::vector<int> U(B);
        for (int& u : U) {
            u = uni(0, 60);
            if (style == 1) u = uni(0, 2) ? 0 : uni(1, 900);
            if (style == 2) u = 1;
            if (style == 3) u = uni(0, 30000);
            if (style == 4) u = uni(1, 1 << uni(1, 24));
        }
        if (style == 0) U[uni(0, B - 1)] = uni(1, 5000);
        check_both(U, slots, uni(3, 18), uni(0, 3) > 0);
        check_both(U, style == 4 ? uni(65, kMaxRanges) : slots, uni(3, 1200), uni(0, 3) > 0);
        check_parts(U, slots, uni(0, 40));
    }
    // ranges handed to a launch that fills the chip: one at least, all at the same time, or a whole number of rounds to within
    // an eighth
    for (int deep = 2; deep <= 3; ++deep)
        for (int inner = 1; inner <= 3000; ++inner) {
            const int cu = 256, s = question_slots(inner, deep * cu, cu, deep == 2), at_once = deep * cu / inner > 1 ? deep * cu / inner : 1;
            const long long busiest = ((long long)s * inner + cu - 1) / cu;
            if (s < at_once || (s > at_once && busiest * cu * 8 > 9ll * s * inner)) ++bad;
        }
    std::printf("%s: %lld cuts (%d with unequal ranges, %d by sequence), seed %u, %d failed checks\n", bad ? "FAILED" : "ok", n_checked, weighted, apart, seed, bad);
    return bad ? 1 : 0;
}
