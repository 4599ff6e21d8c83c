// Where the many-row kernels (question scores; question attention at the watershed layer) leave their log-sum-exps.
//
// The key tiles of a sequence, segment behind segment (history rounds in order, then the current round), are cut into parts
// that may begin and end anywhere.  Every (segment, part) that meet leave one value per query row, at index segment + part
// of the row: unique, since from one tile to the next of the list the segment, the part or both go up by one.  A row of
// segments + parts - 1 values holds them; an index where both went up at once stays unwritten and is not read.
//
// The streaming kernel notes for every segment with tokens its first and its last part: the workgroup that streams its first
// (last) tile for the first KV head and row block.  The finishing kernels read the notes.  Those of the history rounds lie in
// the caller's [B][R_max] score output, which the last finishing kernel overwrites with the scores, those of the current
// round in the workspace's head: no scratch of their own.
#pragma once

#include "common.hpp"

namespace ra {

struct PlaceNote {
    unsigned short first, last;  // parts
};
static_assert(sizeof(PlaceNote) == sizeof(float), "a note takes the place of a score");
struct ScorePlaces {
    PlaceNote* round;  // [B][R_max]
    PlaceNote* cur;    // [B]
    int chunk_limit;   // most 256-token chunks of a sequence by the caller's max_tokens: one with more gets NaN scores
};
constexpr size_t kWsPlacesOff = 4096;  // behind n_parts[kMaxBatch]
static_assert(kMaxBatch * sizeof(int) <= kWsPlacesOff && kWsPlacesOff + kMaxBatch * sizeof(PlaceNote) <= kWsSmallState,
              "what the head of the workspace has room for");

// By a wave, for the segments first .. last that part `part` meets, which holds the tiles [t_lo, t_hi) of sequence b; cum: prefix
// of the segments' tiles.
__device__ __forceinline__ void note_places(const ScorePlaces& pl, int b, int R_max, int n_hist, const int* cum, int first, int last,
                                            int part, int t_lo, int t_hi) {
    for (int i = first + (int)(threadIdx.x & 63); i <= last; i += 64) {
        const int begin = cum[i], end = cum[i + 1];
        if (begin == end) continue;
        PlaceNote* n = i >= n_hist ? pl.cur + b : pl.round + (size_t)b * R_max + i;
        if (begin >= t_lo && end <= t_hi) *n = PlaceNote{(unsigned short)part, (unsigned short)part};
        else if (begin >= t_lo) n->first = (unsigned short)part;
        else if (end <= t_hi) n->last = (unsigned short)part;
    }
}

}  // namespace ra
