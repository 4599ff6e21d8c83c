// Schedule of the matrix-core decode kernel: an equal split of the batch's key tiles over wavefronts, and the
// hand-over of the partial results of a sequence that was cut (round-sparse decode, paper Sec. 3.2 step 5).
//
// The key tiles (32 tokens, never crossing a round) of all sequences of the batch form one list per KV head:
// sequence 0's tiles, then sequence 1's, ...; tile_begin[b] is the index of sequence b's first tile and
// tile_begin[B] = total.  The list is cut into n_ranges ranges of equal size (to within one tile; see RangeCut for
// the one exception): with total = n_ranges * q + rem, the first rem ranges have q + 1 tiles and the others q,
//     range r = [ r * q + min(r, rem) , (r + 1) * q + min(r + 1, rem) ),
// and one wavefront streams one range for one (KV head, block of 16 query rows).  A range may end inside a
// sequence and may cover the tails and heads of several: the part of sequence b inside range r is a SEGMENT, and
// a sequence that lies in more than one range has one partial result ("record") per segment.  Along the list
// both r and b only grow, so  record(r, b) = r + b  is unique over all segments, and the records of one
// sequence are consecutive: record_first(b) .. + n_parts(b) - 1.
//
// Hand-over without waiting: a wave stores the record of its segment and is done; a second, small kernel, launched
// behind the first on the same stream, reads the n_parts records of every sequence that was cut and writes its
// output.  No wave ever waits for another, so every wave exits whatever the order of execution.
//
// Everything here is plain 32-bit integer arithmetic usable on host and device (the GPU has no fast 64-bit
// divide); the host model in tests/host_model/ runs the same functions with one thread per wave.
#pragma once

#ifndef RA_HD
#ifdef __HIPCC__
#define RA_HD __host__ __device__
#else
#define RA_HD
#endif
#endif

namespace ra {

// a / b for a < 2^21, b >= 1.  On the device by a reciprocal: (a + 1/2) / b is at least 1 / (2 b) away from a whole number, and
// the product is off by less than that.
RA_HD inline unsigned small_div(unsigned a, unsigned b) {
#ifdef __HIP_DEVICE_COMPILE__
    return (unsigned)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
#else
    return a / b;
#endif
}

// n / d, 0 <= n <= n_max, by one multiplication with a number made on the host, which is exact while n_max d < 2^31.  A division
// is about 35 dependent instructions, 0.1 microseconds for a wave that is alone on its SIMD, and the decode kernel had a dozen
// between its lists and its first tile.  (In the question kernels, which have scalar registers to spare for neither the numbers
// nor the way out, the same change costs 1 %.)
struct Divisor {
    unsigned magic;  // ceil(2^31 / d), 0: divide
    int d;
    RA_HD int divide(int n) const { return magic ? (int)((unsigned long long)(2u * (unsigned)n) * magic >> 32) : n / d; }
};
inline Divisor divisor(int d, long long n_max) {
    return {n_max * d < 0x80000000ll ? (unsigned)((0x80000000ull + (unsigned)d - 1) / (unsigned)d) : 0u, d};
}

// Row / G for the query rows of the many-row kernels, G <= 16, by one multiplication: exact below 2^27 rows, of whose partial
// results a workspace would hold terabytes.  (A division is twenty instructions, and a question kernel had a dozen of them
// in front of its first tile and in every store of scores.)
struct RowsPerToken {
    unsigned magic;  // ceil(2^31 / G)
    RA_HD explicit RowsPerToken(int G) : magic((0x80000000u + (unsigned)G - 1) / (unsigned)G) {}
    RA_HD int token(int row) const { return (int)((unsigned long long)(2u * (unsigned)row) * magic >> 32); }
};

// Number of ranges for a batch of `total` tiles: never more than `max_ranges` (the wavefronts of the launch
// divided by the work items per range) and no range shorter than `min_units` tiles.
RA_HD inline unsigned range_count(unsigned total, int min_units, int max_ranges) {
    unsigned n = total / (unsigned)(min_units > 0 ? min_units : 1);
    if (n > (unsigned)max_ranges) n = (unsigned)max_ranges;
    return n < 1 ? 1 : n;
}

// The cut of a batch, prepared once.  total < 2^30.
//
// With skew = 0 all ranges are equal to within one tile.  With skew > 0 (in 1/1000) and a launch that fills the
// chip (as many ranges as it may have, an even number, and long ones) the first half of the ranges, which the
// workgroups dispatched first stream, get (1 + skew/1000) / 2 of the tiles and the second half the rest: the
// hardware serves the waves that came first on a compute unit a little faster for the whole kernel, and ranges
// in proportion let both halves end together.  Inside each half the ranges are again equal to within one tile:
// the first rem_x ranges of a half have q_x + 1 tiles, the others q_x.
struct RangeCut {
    unsigned total, n_ranges;
    unsigned n_a, total_a, q_a, rem_a;  // first class: ranges 0 .. n_a - 1 cover tiles [0, total_a)
    unsigned q_b, rem_b;                // second class: ranges n_a .. n_ranges - 1 cover the rest
};
constexpr unsigned kSkewMinTiles = 16;  // ranges shorter than this are not skewed: their start dominates
RA_HD inline RangeCut range_cut(unsigned total, int min_units, int max_ranges, int skew = 0) {
    RangeCut c;
    c.total = total;
    c.n_ranges = range_count(total, min_units, max_ranges);
    c.n_a = c.n_ranges;
    c.total_a = total;
    if (skew > 0 && c.n_ranges == (unsigned)max_ranges && c.n_ranges >= 2 && (c.n_ranges & 1) == 0 &&
        total / c.n_ranges >= kSkewMinTiles) {
        const unsigned w = 1000u + (unsigned)(skew > 500 ? 500 : skew);
        c.n_a = c.n_ranges / 2;
        c.total_a = total / 2000u * w + total % 2000u * w / 2000u;  // total * w / 2000 without leaving 32 bits
    }
    const unsigned n_b = c.n_ranges - c.n_a, total_b = total - c.total_a;
    c.q_a = c.total_a / c.n_a;
    c.rem_a = c.total_a - c.q_a * c.n_a;
    c.q_b = n_b ? total_b / n_b : 1;
    c.rem_b = n_b ? total_b - c.q_b * n_b : 0;
    return c;
}
RA_HD inline unsigned range_begin(const RangeCut& c, unsigned r) {
    if (r <= c.n_a) return r * c.q_a + (r < c.rem_a ? r : c.rem_a);
    const unsigned k = r - c.n_a;
    return c.total_a + k * c.q_b + (k < c.rem_b ? k : c.rem_b);
}

// The range that holds tile t, 0 <= t < total.
RA_HD inline unsigned range_of_tile(const RangeCut& c, unsigned t) {
    if (t < c.total_a) {
        const unsigned big = c.rem_a * (c.q_a + 1);  // tiles in the ranges of q_a + 1
        return t < big ? t / (c.q_a + 1) : c.rem_a + (t - big) / c.q_a;
    }
    const unsigned u = t - c.total_a, big = c.rem_b * (c.q_b + 1);
    return c.n_a + (u < big ? u / (c.q_b + 1) : c.rem_b + (u - big) / c.q_b);
}

// The other cut, for few sequences and short ranges: every sequence by itself, into pieces of at most `len` tiles that are equal
// to within one.  A range that goes on with the next sequence starts twice, queries, segment table and first tile one memory
// round trip behind the other, and with a few tiles a range that is the longest wave of the launch.  Piece j of sequence b is
// range first(b) + j, first(b) being the number of pieces of the sequences before b; records as above.
struct SeqCut {
    int n, q, rem;  // pieces; the first rem of them have q + 1 tiles, the others q
};
RA_HD inline SeqCut seq_cut(int tiles, int len) {
    SeqCut c;
    c.n = (int)small_div((unsigned)tiles + (unsigned)len - 1, (unsigned)len);
    c.q = c.n > 0 ? (int)small_div((unsigned)tiles, (unsigned)c.n) : 0;
    c.rem = tiles - c.q * c.n;
    return c;
}
RA_HD inline int seq_cut_begin(const SeqCut& c, int j) { return j * c.q + (j < c.rem ? j : c.rem); }
// The lengths to try, *len and up to two of them, until there are no more pieces than ranges; 0: the batch is cut as one list.
// The first is that of the one list's longest range: as many pieces as there may be ranges, if every sequence were a whole
// number of them.  A tile more is worth it while it costs less than a second start.  (Whole decode call, batch cut as one list
// and by sequence, tiles per range in brackets, 128 channels.  At the first length: 8 dialogues [4.2] 23.4 and 22.5 microseconds,
// [6.2] 27.4 and 26.4, [8.3] 32.2 and 32.1; 10 of 64 heads [8.3] 34.4 and 33.2, [12.5] 42.7 and 42.3; 42 of 2 KV heads [4.2] 26.4
// and 24.3, [13] 45.5 and 45.1; longer ones alike or slower, 8 dialogues [18] 55.6 and 56.0.  At the second: 8 dialogues [5] 25.1
// and 24.2, [8.9] 33.5 and 34.0, [15] 47.8 and 48.5.  And a length that does not fit costs 0.3 in the prologue.  64 channels:
// 42 dialogues [4.2] 25.4 and 23.9; 16 [5.3] 24.6 and 24.6, [7.5] 29.1 and 29.6, [11.3] 39.5 and 40.3.  With less than twelve
// possible ranges for a sequence the pieces come out uneven, and the launch waits for the longest: 16 dialogues, 128 ranges,
// 121.6 -> 122.7; 24, 256 ranges, 56.8 -> 58.0; 40 of a few tiles 16.0 -> 17.5.)
constexpr int kSeqCutTries = 2;
constexpr int kSeqCutRanges = 12;      // ranges there may be for every sequence, at least
constexpr int kSeqCutTwice = 5;        // longest first length with a second
RA_HD constexpr int seq_cut_longest(int d) { return d == 64 ? 5 : 12; }  // longest first length
RA_HD inline int seq_cut_lengths(int B, int d, unsigned total, int min_units, int max_ranges, int* len) {
    if (B * kSeqCutRanges > max_ranges || total > (unsigned)(seq_cut_longest(d) * max_ranges)) return 0;
    *len = (int)small_div(total + (unsigned)max_ranges - 1, (unsigned)max_ranges);  // (total is at most twelve times max_ranges)
    if (*len < min_units) *len = min_units;
    return *len > kSeqCutTwice ? 1 : 2;
}

// Records of a sequence with tiles [t_lo, t_hi), t_hi > t_lo.
struct SeqParts {
    int first_range, n_parts;
};
RA_HD inline SeqParts seq_parts(const RangeCut& c, unsigned t_lo, unsigned t_hi) {
    SeqParts p;
    p.first_range = (int)range_of_tile(c, t_lo);
    p.n_parts = (int)range_of_tile(c, t_hi - 1) - p.first_range + 1;
    return p;
}
RA_HD inline int record_index(int r, int b) { return r + b; }
// Upper bound of record_index + 1 for a launch.
RA_HD inline int record_capacity(int max_ranges, int B) { return max_ranges + B; }

// The second step: 256 threads merge `rows` rows of a (sequence, KV head, block of up to 16 query rows), d / 4 threads a row; the
// groups of threads that this leaves take the records in turn, with `flight` of them in flight in every group.
// A workgroup for every row while they are at most four to a compute unit: few sequences are cut into many records each, and
// one workgroup walking them for eight rows took most of the call (whole decode call, in microseconds: one dialogue of 100
// rounds of 600 tokens, 30 % kept, 2 KV heads of 16 rows 87.5 -> 19.1, of 200 rounds, 8 KV heads of 4 rows 49.3 -> 35.0;
// four of 20 rounds 25.9 -> 20.6).  More rows than that have few records each, and a workgroup per row is mostly
// its own start: 64 dialogues, 512 blocks of 8 rows, 30.5 with a workgroup for 8 rows, 34.3 with one per row; 80 blocks of 16
// rows 37.3 and 38.0; 128 blocks of 8 rows 79.1 and 78.8.
struct MergeShape {
    int rows, flight;
};
RA_HD inline MergeShape merge_shape(int blocks, int rows, int num_cu) {
    if ((long long)blocks * rows <= 4ll * num_cu) return {1, 8};
    return {rows <= 1 ? 1 : rows <= 2 ? 2 : rows <= 4 ? 4 : 8, 4};
}
// Ranges are as short as two tiles (kMfmaSpreadUnits) while no sequence has more tiles than this: twice as many records as with
// four must not cost the merge more than the shorter ranges save, and it walks them the more slowly the more rows a workgroup has.
// (Whole call, ranges of four and of two tiles.  A workgroup for every row, one dialogue: 65 tiles of 8 rows 15.6 and 13.1
// microseconds, 193 16.5 and 15.5, 241 16.6 and 16.4; of 16 rows 65 tiles 15.5 and 12.8, 241 16.3 and 14.7, 481 17.5 and 17.0,
// twice 481 18.2 and 18.9, 801 19.6 and 20.9; 64 channels, 97 tiles of 4 rows 12.9 and 11.4.  Eight rows to one, a long dialogue
// among short ones: 17 dialogues of 8 rows, 64 tiles 20.4 and 17.9, 96 21.8 and 20.5, 128 23.0 and 23.0, 240 28.8 and 32.9; 34 of
// 16 rows, 64 tiles 17.8 and 17.5, 96 19.5 and 20.3, 384 30.8 and 43.3; 64 channels, 17 of 8 rows, 96 tiles 14.6 and 14.7, 384
// 21.3 and 28.5, 64 of 8 rows, 128 18.5 and 17.1, 240 21.0 and 21.7.  Four: 64 dialogues, 192 tiles 24.1 and 23.3; 64 channels,
// 192 18.2 and 16.6, 240 18.9 and 19.4, 384 21.2 and 22.6.)
RA_HD inline int spread_longest(const MergeShape& m) { return m.rows <= 2 ? 384 : 768 / m.rows; }

// Largest b in [0, n) with begin[b] <= t, for begin[0] <= t < begin[n] (begin non-decreasing).
template <typename T>
RA_HD inline int upper_slot(const T* begin, int n, long long t) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((long long)begin[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

}  // namespace ra
