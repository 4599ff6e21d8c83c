// Round selection (paper Sec. 3.3) for one sequence by one workgroup, on a score vector that already lies in LDS.
// Shared by the stand-alone selection kernel and by the score pass's finishing kernel when a call asks for the
// scores and the selection together.
//
// Every strategy reduces to "keep the n best rounds" (higher score first, then lower index):
//   ADAPTIVE / THRESHOLD  n = number of scores above the cut (those are exactly the n best)
//   TOP_FRACTION          n = ceil(fraction * R)
// then n is clamped by min_rounds / max_rounds.  Ranks are found by counting, the kept rounds are compacted in
// ascending order with wavefront ballots and a prefix over the waves.
// keep_first / keep_last (an optional policy, not the paper's) add the first and the most recent rounds to
// whatever the rule kept; the rule itself is evaluated as without them.
#pragma once

#include "stream_kv.hpp"

namespace ra {

constexpr int kSelectWaves = 16;  // most waves a selecting workgroup has

// LDS a selecting workgroup needs beside the score vector itself.
struct SelectShared {
    double cut;
    double terms[kMaxRounds];          // terms of a sequential sum, zeros up to a multiple of 16
    int part[kSelectWaves * 64];       // ranks of the rounds; up to 64 rounds: every wave's share of them
    int wave_cnt[kSelectWaves], wave_pass[kSelectWaves];
};

// ((t[0] + t[1]) + t[2]) + ... in that order.  The additions are the only serial part: sixteen terms at a time come
// from LDS while the sixteen before them are added.
#pragma clang fp contract(off)
__device__ static double sequential_sum(const double* t, int n) {
    double v[16], total = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = t[j];
    for (int j0 = 0; j0 < n; j0 += 16) {
        const int next = j0 + 16 < n ? j0 + 16 : j0;
        double w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = t[next + j];
#pragma unroll
        for (int j = 0; j < 16; ++j) total = total + v[j];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = w[j];
    }
    return total;
}

// The cut of the adaptive rule in IEEE double, sums taken sequentially in round order with separate
// multiply and add (no contraction), so that a host reference doing the same steps gets the same bits (the zeros
// behind the last term leave a sum that starts at +0.0 as it is).  Called by one whole wave, whose lanes convert the
// scores and square the deviations side by side.
#pragma clang fp contract(off)
__device__ static double adaptive_cut(const float* s, int R, double lambda, int ddof, double* terms) {
    const int lane = threadIdx.x & 63, R16 = (R + 15) & ~15;
    for (int r = lane; r < R16; r += 64) terms[r] = r < R ? (double)s[r] : 0.0;
    __builtin_amdgcn_wave_barrier();  // same wave: LDS operations complete in program order
    const double mean = sequential_sum(terms, R) / (double)R;
    __builtin_amdgcn_wave_barrier();
    for (int r = lane; r < R16; r += 64) {
        const double dev = r < R ? (double)s[r] - mean : 0.0;
        terms[r] = dev * dev;
    }
    __builtin_amdgcn_wave_barrier();
    const double ss = sequential_sum(terms, R);
    const int den = R - ddof;
    const double sd = den > 0 ? __builtin_sqrt(ss / (double)den) : 0.0;
    return mean + lambda * sd;
}

// Number of rounds preferred over round r with score x (higher score first, then lower index).  Sixteen scores at a
// time come from LDS; the rounds of a wave are r_wave .. r_wave + 63, so only those 64 need both comparisons.
__device__ __forceinline__ int rank_of(const float* s, int R, float x, int r, int r_wave) {
    int rank = 0;
    auto block = [&](int j0, auto preferred) {
        float4 y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = *reinterpret_cast<const float4*>(s + j0 + 4 * i);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            rank += preferred(y[i].x, j0 + 4 * i) + preferred(y[i].y, j0 + 4 * i + 1) + preferred(y[i].z, j0 + 4 * i + 2) +
                    preferred(y[i].w, j0 + 4 * i + 3);
    };
    const int own_end = min(r_wave + 64, R & ~15), end = R & ~15;
    int j = 0;
    for (; j < r_wave; j += 16) block(j, [&](float y, int) { return y >= x ? 1 : 0; });
    for (; j < own_end; j += 16) block(j, [&](float y, int jj) { return (y > x || (y == x && jj < r)) ? 1 : 0; });
    for (; j < end; j += 16) block(j, [&](float y, int) { return y > x ? 1 : 0; });
    for (; j < R; ++j) rank += (s[j] > x || (s[j] == x && j < r)) ? 1 : 0;
    return rank;
}

// s[0..R): the sequence's scores in LDS, 16-byte aligned (complete: a barrier lies between their last write and this
// call).  out[0..R_max): the sequence's row of sel_idx; *n_sel_out: its count.  Must be called by all threads of a
// workgroup of 4 to kSelectWaves waves.
// The last wave takes the cut while the others rank.  Up to 64 rounds (the usual dialogue) they share the comparisons
// of every round, and after the one barrier the first wave, a lane per round, finishes.  (Stand-alone selection by the
// adaptive rule, one lane walking the scores for the cut and every thread for its rank before: 60 rounds 5.7 -> 3.6
// microseconds, 200 rounds 12.2 -> 9.6, 1000 rounds 125 -> 71.)
__device__ inline void select_rounds_block(const float* s, int R, int R_max, const ra_select_params& p, int32_t* out,
                                           int32_t* n_sel_out, SelectShared& sh) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int NT = blockDim.x, NW = NT >> 6;
    const bool by_cut = p.strategy != RA_SEL_TOP_FRACTION;
    auto rounds_kept = [&](int n_pass) {
        int n_keep = n_pass;
        if (!by_cut) {
            const double want = __builtin_ceil(p.fraction * (double)R);
            n_keep = want < 1.0 ? 1 : (want > (double)R ? R : (int)want);
        }
        if (n_keep < p.min_rounds) n_keep = p.min_rounds;
        if (p.max_rounds > 0 && n_keep > p.max_rounds) n_keep = p.max_rounds;
        return n_keep > R ? R : n_keep;
    };
    // keep[r] <=> rank(r) < n_keep, rank = number of rounds preferred over r
    auto keeps = [&](int r, int rank, int n_keep) { return rank < n_keep || r < p.keep_first || r >= R - p.keep_last; };
    const int n_rank_waves = by_cut ? NW - 1 : NW;
    if (by_cut && wave == NW - 1 && R > 0) {
        const double cut = p.strategy == RA_SEL_ADAPTIVE ? adaptive_cut(s, R, p.lambda, p.ddof, sh.terms) : p.threshold;
        if (lane == 0) sh.cut = cut;
    }
    if (R <= 64) {
        const float x = lane < R ? s[lane] : 0.f;
        if (wave < n_rank_waves) {
            int rank = 0;
#pragma unroll 4
            for (int j = wave; j < R; j += n_rank_waves) {
                const float y = s[j];
                rank += (y > x || (y == x && j < lane)) ? 1 : 0;
            }
            sh.part[wave * 64 + lane] = rank;
        }
        lds_barrier();
        for (int r = 64 + tid; r < R_max; r += NT) out[r] = -1;
        if (wave != 0) return;
        int rank = 0;
#pragma unroll 4
        for (int w = 0; w < n_rank_waves; ++w) rank += sh.part[w * 64 + lane];
        const int n_pass = by_cut && R > 0 ? __popcll(__ballot(lane < R && (double)x > sh.cut)) : 0;
        const unsigned long long mask = __ballot(lane < R && keeps(lane, rank, rounds_kept(n_pass)));
        const int n = __popcll(mask);
        if (mask >> lane & 1) out[__popcll(mask & ((1ull << lane) - 1ull))] = lane;
        if (lane >= n && lane < R_max) out[lane] = -1;
        if (lane == 0) *n_sel_out = n;
        return;
    }
    for (int r0 = wave * 64; r0 < R; r0 += NT) {
        const int r = r0 + lane;
        const float x = r < R ? s[r] : 0.f;
        sh.part[r] = rank_of(s, R, x, r, r0);  // read by this thread alone
    }
    lds_barrier();
    int n_pass = 0;
    if (by_cut) {
        const double cut = sh.cut;
        int cnt = 0;
        for (int r0 = wave * 64; r0 < R; r0 += NT) cnt += __popcll(__ballot(r0 + lane < R && (double)s[min(r0 + lane, R - 1)] > cut));
        if (lane == 0) sh.wave_pass[wave] = cnt;
        lds_barrier();
        for (int w = 0; w < NW; ++w) n_pass += sh.wave_pass[w];
    }
    const int n_keep = rounds_kept(n_pass);
    // the kept rounds in ascending order: ballots and a prefix over the waves, NT rounds at a time
    int base = 0;
    for (int r0 = 0; r0 < R; r0 += NT) {
        const int r = r0 + tid;
        const bool keep = r < R && keeps(r, sh.part[min(r, R - 1)], n_keep);
        const unsigned long long mask = __ballot(keep);
        if (lane == 0) sh.wave_cnt[wave] = __popcll(mask);
        lds_barrier();
        int before = base, all = 0;
        for (int w = 0; w < NW; ++w) {
            if (w < wave) before += sh.wave_cnt[w];
            all += sh.wave_cnt[w];
        }
        if (keep) out[before + __popcll(mask & ((1ull << lane) - 1ull))] = r;
        base += all;
        lds_barrier();
    }
    for (int r = base + tid; r < R_max; r += NT) out[r] = -1;
    if (tid == 0) *n_sel_out = base;
}

// Host-side check of the selection parameters shared by the entry points; `who` prefixes the error text.
int check_select_params(const ra_select_params* params, const char* who);

}  // namespace ra
