// Cut of the key tiles of a question's batch into ranges, one per group of workgroups (question prefill and its round
// scores, paper Sec. 3.2 steps 2 to 4), for at most kInlineBatch sequences.
//
// The tiles of all sequences form one list, and a range may end inside a sequence and go on with the next: cutting every
// sequence by itself leaves pieces of unequal size (four pieces a sequence: a quarter of a sequence too much here and
// there), and the longest one is the launch.
// The ranges are sized by how the hardware serves the workgroups that stream them.  Of the C workgroups that share a
// compute unit the one dispatched first is the older one on every SIMD and gets the issue port first for the whole
// kernel; with equal ranges it ends early and the last one runs alone, with nothing left to overlap its softmax with
// (128-token question over four dialogues of 32 000 tokens: the classes of the score kernel ended after 118, 140 and
// 187 microseconds, of the attention kernel after 121 and 154).  A launch that fills the chip C deep therefore deals the
// ranges out to C classes in turn (class k = the k-th workgroup to land on a unit) and sizes them by `weight`.
// That holds if every class has as many ranges as the others: with one range more in the first class its last workgroups
// land second on their units and are the longest of all (200 tokens, 9 ranges of the attention kernel: 118.7 microseconds
// by weight, 109.0 equal; the score kernel with 5, 8, 19 ranges: 305, 204, 163 and 285, 182, 150; with 48 ranges 156 and
// 169, attention kernel with 2 ranges of 1000 tokens 249 and 277, at the watershed layer with 16 399 and 414).  Launches
// over paged blocks, which wait for their table entries, and of the fp16 mode are not served that way: attention kernel
// 179 microseconds by weight and 171 equal paged, 485 and 469 at the watershed layer, 132 and 127 in the fp16 mode; score
// kernel, paged, 192 and 190.
//
// Plain arithmetic usable on host and device; tests/host_model/tile_ranges.cpp runs it on the CPU.
#pragma once

#include "range_schedule.hpp"

#ifndef RA_HD
#ifdef __HIPCC__
#define RA_HD __host__ __device__
#else
#define RA_HD
#endif
#endif

namespace ra {

// Launches that plan themselves, questions and decode alike: a lane for every sequence, the lists in one pass of 256 threads.
constexpr int kInlineBatch = 64;     // most sequences
constexpr int kInlineRounds = 1024;  // most sequences times R_max
static_assert(kInlineBatch <= 64 && kInlineRounds % 256 == 0, "what the planning code reads in one pass");
constexpr int kMaxRanges = 1024;  // most ranges, whatever the launch

// First tile of piece j of n <= kMaxRanges equal pieces of U tiles: floor(U j / n), whose product would leave 32 bits (a sequence
// has up to 2^24 tiles), by the quotient and the remainder of U / n.
RA_HD inline int piece_begin(int U, int j, int n) {
    const int q = U / n;
    return q * j + (int)small_div((unsigned)((U - q * n) * j), (unsigned)n);
}
static_assert((long long)kMaxRanges * kMaxRanges < 1ll << 21, "what small_div takes");

template <int C>
struct RangeWeights {
    int w[C];  // in 1/1000 of an equal range
};
RA_HD constexpr RangeWeights<3> score_range_weights() { return {{1370, 1080, 550}}; }
RA_HD constexpr RangeWeights<2> attn_range_weights() { return {{1180, 820}}; }

constexpr int kShortRange = 8;     // longest ranges that sequences cut by themselves may exceed
constexpr int kWeightedTiles = 8;  // shortest ranges that are cut by weight (and none of which a light class leaves without a tile)

// Most ranges of a launch of `grid` workgroups, `inner` of which stream each range (its KV heads and blocks of query rows).
// A range's workgroups lie on consecutive units, and the launch lasts as long as the unit with the most of them.  As many
// ranges as run at the same time, if that leaves no more than an eighth of the units' time unused; otherwise the fewest
// more for which it does, by workgroups that stream several ranges one after the other.  With `partials`, whose number
// grows with the ranges, only if that takes a sixth off.  (Attention kernel, 600 tokens of 64 heads, inner 304: 1 range 450
// microseconds, 3 335; 1500 tokens, inner 376: 1 range 336, 2 291; 2500, inner 632: 1 range 649, 2 542; 200 of 64 heads,
// inner 104: 4 ranges 211, 7 212.  Score kernel, 2500 tokens, inner 320: 2 ranges 426, 3 381.)
inline int question_slots(int inner, long long grid, int num_cu, bool partials) {
    const int at_once = (int)(grid / inner) < 1 ? 1 : (int)(grid / inner);
    if (grid < num_cu) return at_once;
    auto busiest = [&](int s) { return ((long long)s * inner + num_cu - 1) / num_cu; };  // workgroups' worth of ranges on a unit
    for (int s = at_once; s <= 4 * at_once + 4; ++s) {
        if (busiest(s) * num_cu * 8 > (long long)s * inner * 9) continue;
        return partials && busiest(s) * at_once * 6 > busiest(at_once) * s * 5 ? at_once : s;
    }
    return at_once;
}

// Parts of a sequence that the values and the partial results of a row have room for: those of the launch's shortest ranges
// (`most`) as far as twice a sequence's share of the ranges goes, at least those of ranges of eight tiles (`of_eight`); no sequence
// meets more than `slots`.  Rows with more room than that are longer to write and read (122 tokens of 64 heads over nine dialogues
// of 27 short rounds, 24 ranges of scores and 8 of attention: 144.7 microseconds with the parts of eight tiles, 154.0 with room for
// 24 and 18).
inline int question_parts(long long most, long long of_eight, int slots, int n_sequences) {
    const long long share = 2ll * ((slots + n_sequences - 1) / n_sequences) + 2;
    const long long room = of_eight > share ? of_eight : share, parts = most < room ? most : room;
    return (int)(parts < slots ? parts : slots);
}

// At most `slots` ranges of about `len` tiles, at least min_tiles, such that at most max_parts (> 2) of them meet one
// sequence: the partial results of a row have room for that many.  A sequence that meets max_parts + 1 ranges holds the
// max_parts - 1 between its first and its last one whole, and at least a tile of each of those two.
//   * Equal ranges: len >= most / (max_parts - 2) and total > (n_ranges - 1) len, so max_parts - 1 of them hold more than
//     `most` tiles as long as there are that many, and rounding the ends down takes less than one.
//   * Ranges by weight: a run that begins and ends with the lightest class holds less than its share.  They are taken if
//     there are no more than max_parts, or if the lightest run of max_parts - 1 holds `most` tiles all the same.
template <int C>
struct TileCut {
    int total, len, n_ranges, w[C], sum;  // sum: weight of a turn of the classes

    // most: tiles of the longest sequence; full: by weight, if there are as many ranges as the launch may have
    RA_HD TileCut(int total_, int most, int slots, int min_tiles, int max_parts, bool full, const RangeWeights<C>& weights) {
        total = total_;
        len = (total + slots - 1) / slots;
        if (len < min_tiles) len = min_tiles;
        const int fewest = (most + max_parts - 3) / (max_parts - 2);
        if (len < fewest) len = fewest;
        n_ranges = (total + len - 1) / len;
        if (n_ranges < 1) n_ranges = 1;
        sum = 0;
        for (int k = 0; k < C; ++k) sum += w[k] = weights.w[k];
        const bool fits = n_ranges <= max_parts ||
                          (long long)lightest_run(max_parts - 1) * total >= (long long)most * weight_before(n_ranges % C, n_ranges / C);
        if (!(full && len >= kWeightedTiles && n_ranges == slots && n_ranges % C == 0 && fits)) {
            for (int k = 0; k < C; ++k) w[k] = 1000;
            sum = 1000 * C;
        }
    }
    RA_HD int lightest_run(int n) const {  // of n consecutive ranges
        int least = sum;
        for (int k = 0; k < C; ++k) {
            int x = 0;
            for (int j = 0; j < C; ++j) x += j < n % C ? w[(k + j) % C] : 0;
            least = x < least ? x : least;
        }
        return n / C * sum + (n % C ? least : 0);
    }
    RA_HD bool by_weight() const { return w[0] != 1000; }
    RA_HD int weight_before(int k, int turns) const {  // of the first k classes, and of so many whole turns of the classes
        int x = turns * sum;
        for (int j = 0; j < C; ++j) x += j < k ? w[j] : 0;
        return x;
    }
    RA_HD double tiles_per_weight() const { return (double)total / (double)weight_before(n_ranges % C, n_ranges / C); }
    // first tile of range r, 0 <= r <= n_ranges: monotone, as the rounding of the product is (in double: a batch has up to
    // 2^30 tiles, and a float's rounding could move the ends by several)
    RA_HD int begin(int r, double per_weight) const {
        const int t = (int)((double)weight_before(r % C, r / C) * per_weight);
        return r == n_ranges || t > total ? total : t;
    }
    // Every sequence by itself if that takes no more ranges than there may be, or, while they are short, with pieces up to two
    // tiles longer: a range that crosses from one sequence into the next starts twice, which takes as long as one to three
    // tiles.  (Whole calls: 38 tokens over 9 dialogues 73.3 -> 70.9 microseconds, 19 over three paged ones, no tile longer, 71.2
    // -> 68.0; with three tiles longer at any length 10 dialogues of 48 tiles a range 146.0 -> 148.0, three of 10 at the
    // watershed layer 43.6 -> 45.2.)
    // The lengths `len` .. longest_apart() are tried in turn; the first for which apart() holds is taken, with piece_begin() of
    // the cuts() pieces of every sequence as the ends.  None of them meets more than max_parts: they are no shorter than `len`.
    RA_HD int longest_apart(int n_sequences) const {
        if (n_sequences < 2 || by_weight()) return 0;
        return len + (len <= kShortRange ? 2 : 0);
    }
    RA_HD static int cuts(int U, int length) { return U > 0 ? (U + length - 1) / length : 0; }
    RA_HD static bool apart(int n_apart, int slots) { return n_apart <= slots && n_apart > 0; }  // n_apart: the sum of cuts()
};

}  // namespace ra
