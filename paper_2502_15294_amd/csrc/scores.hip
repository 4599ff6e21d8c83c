// Round scores at the watershed layer (paper Sec. 3.1, Eq. 1 and the normalisation after it): the generic
// streaming kernel, the finishing kernels and the entry point.
//
// (1) A streaming pass over the watershed layer's keys, HBM-bandwidth bound like decode attention but
//     without values, leaves one log-sum-exp per (query row, 256-token chunk of a round).  For bf16 / d = 128
//     it runs on the matrix cores (scores_mfma.hip, scores_prefill_mfma.hip); the kernel below serves fp32 and
//     d = 64: workgroup (c, g, b*q_len+i) owns chunk c of sequence b for KV head g and query token i, each of
//     its four waves issues the loads of its four 16-token units up front (16 KB in flight per workgroup), then
//     reduces the logits of the chunk to one log-sum-exp per query head.  Equal-sized work items keep long
//     rounds from becoming the tail of the launch.
// (2) Finishing kernels turn the per-chunk log-sum-exps into Eq. 1: per round the log-sum-exp over its chunks,
//     per query token the softmax normaliser over all rounds and the visible part of the current round, the
//     probability mass of every history round summed over the query tokens, normalisation over history
//     rounds, mean over query heads.  One kernel does all of it for a single query token; for several query
//     tokens the work of a head is split over several workgroups and a second small kernel normalises.
#include "scores_common.hpp"
#include "select_common.hpp"
#include "stream_kv.hpp"

namespace ra {

template <typename T, int D, int G, bool PAGED>
__global__ __launch_bounds__(256) void scores_stream_kernel(ScoreArgs a) {
    constexpr int EPL = D / 16;
    using Ops = RowOps<T, EPL>;
    constexpr int WORDS = Ops::WORDS;
    constexpr int EB = Ops::ELEM_BYTES;
    __shared__ float sm[4][G], sl[4][G];
    extern __shared__ __align__(16) char smem[];

    const DevView& vw = a.view;
    const int c = blockIdx.x, g = blockIdx.y;
    const int b = blockIdx.z / a.q_len, i = blockIdx.z - b * a.q_len;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, grp = lane >> 4, sub = lane & 15;
    const int Hkv = vw.Hkv;

    // ---- which round does chunk c belong to? -------------------------------------------------------
    const int n_hist = min(max(vw.n_rounds[b], 0), vw.R_max);
    const int cur_vis = a.cur_k ? cur_visible(a.cur_len, a.q_len, i) : 0;
    // the current round is chunked by its full length (the same for every query token); what a query
    // token may see of it is applied as a mask
    const int n_slots = n_hist + (a.cur_k && a.cur_len > 0 ? 1 : 0);
    const int cap = vw.R_max + 1;
    long long* t_off = reinterpret_cast<long long*>(smem);
    int* t_len = reinterpret_cast<int*>(t_off + cap);
    int* t_cum = t_len + cap;
    for (int s = tid; s < n_slots; s += 256) {
        int len = a.cur_len;
        long long off = 0;
        if (s < n_hist) {
            len = max(vw.seg_len[(size_t)b * vw.R_max + s], 0);
            off = vw.seg_off[(size_t)b * vw.R_max + s];
        }
        t_len[s] = len;
        t_off[s] = off;
        t_cum[s] = chunks_of(len);
    }
    exclusive_scan_units(t_cum, n_slots);
    const int total = n_slots > 0 ? t_cum[n_slots] : 0;
    if (c >= total) return;
    const int slot = find_slot(t_cum, n_slots, c);
    const int len = t_len[slot];
    const long long off = t_off[slot];
    const bool is_cur = slot >= n_hist;
    const int vis = is_cur ? cur_vis : len;  // tokens of this segment the query token may see
    const int chunk_tok0 = (c - t_cum[slot]) * kChunkTokens;

    uint32_t qw[G][WORDS];
    {
        const char* qp = reinterpret_cast<const char*>(a.q) +
                         ((((size_t)b * a.q_len + i) * a.Hq) + (size_t)g * G) * D * EB;
#pragma unroll
        for (int h = 0; h < G; ++h) {
            Frag<WORDS> f = load_frag<WORDS>(qp + ((size_t)h * D + sub * EPL) * EB);
#pragma unroll
            for (int e = 0; e < WORDS; ++e) qw[h][e] = f.w[e];
        }
    }

    // ---- issue every load of this wave's four units, then do the arithmetic ---------------------------
    const char* kbase = reinterpret_cast<const char*>(vw.k);
    Frag<WORDS> kf[4][4];
    int ntok[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int tok0 = chunk_tok0 + (j * 4 + wave) * kUnitTokens;  // the four waves read adjacent units
        ntok[j] = min(kUnitTokens, vis - tok0);
        if (ntok[j] > 0) {
            const char* kp;
            size_t stride;
            if (is_cur) {
                kp = reinterpret_cast<const char*>(a.cur_k) + ((((size_t)b * a.cur_len + tok0) * Hkv + g) * D) * EB;
                stride = (size_t)Hkv * D * EB;
            } else if (PAGED) {
                long long si = off + tok0 / kUnitTokens;
                si = si < 0 ? 0 : (si >= vw.max_blocks ? vw.max_blocks - 1 : si);
                int blk = vw.block_table[(size_t)b * vw.max_blocks + si];
                if (blk < 0) { blk = 0; ntok[j] = 0; }
                kp = kbase + ((((size_t)blk * Hkv + g) * kUnitTokens) * D) * EB;
                stride = (size_t)D * EB;
            } else {
                kp = kbase + (((size_t)off * Hkv + (size_t)g * len + tok0) * D) * EB;
                stride = (size_t)D * EB;
            }
            const int last = max(ntok[j] - 1, 0);
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4) {
                const int t = min(t4 * 4 + grp, last);  // rows past the round's end re-read its last row
                kf[j][t4] = load_frag<WORDS>(kp + (size_t)t * stride + (size_t)sub * EPL * EB);
            }
        }
    }

    // ---- logits: lane (grp, sub) ends with those of token 4 (sub % 4) + grp of every unit ------------------------------
    float sc[4][G];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (ntok[j] > 0) {
            const bool valid = 4 * (lane & 3) + grp < ntok[j];
#pragma unroll
            for (int h = 0; h < G; ++h) {
                float d[4];
#pragma unroll
                for (int t4 = 0; t4 < 4; ++t4) d[t4] = Ops::dot(kf[j][t4].w, qw[h]);
                const float all = row16_sums(d);
                sc[j][h] = valid ? all : -__builtin_inff();
            }
        } else {
#pragma unroll
            for (int h = 0; h < G; ++h) sc[j][h] = -__builtin_inff();
        }
    }

    // ---- a lane's four tokens, then the wave's 16 token lanes, then the four waves -----------------------
    // (With an online softmax unit by unit, its four tokens in every lane of a row, the kernel was bound by the vector ALU:
    // 16 dialogues of 14 400 tokens, four heads per KV head, step 255 -> 247 microseconds, eight 350 -> 327; 24 with 64 channels,
    // eight heads 290 -> 227.)
#pragma unroll
    for (int h = 0; h < G; ++h) {
        const float m = vmax(vmax(vmax(sc[0][h], sc[1][h]), vmax(sc[2][h], sc[3][h])), kNegBig), mc = m * a.c;
        float lv = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (ntok[j] > 0) lv += fast_exp2(__builtin_fmaf(sc[j][h], a.c, -mc));
        float M = vmax(m, dpp_mov<0xB1>(m));
        M = xrow_max4(vmax(M, dpp_mov<0x4E>(M)));
        lv *= fast_exp2((m - M) * a.c);
        lv += dpp_mov<0xB1>(lv);
        lv += dpp_mov<0x4E>(lv);
        lv = xrow_sum4(lv);
        if (lane == 0) {
            sm[wave][h] = M;
            sl[wave][h] = lv;
        }
    }
    __syncthreads();
    if (tid < G) {
        const int h = tid;
        const float M = fmaxf(fmaxf(sm[0][h], sm[1][h]), fmaxf(sm[2][h], sm[3][h]));
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) den = __builtin_fmaf(sl[w][h], fast_exp2((sm[w][h] - M) * a.c), den);
        const size_t idx = ((((size_t)b * a.Hq + (size_t)g * G + h) * a.q_len) + i) * a.n_chunks_max + c;
        // natural log of sum_j exp(scale * logit_j) = ln2 * (M * c + log2(den))
        a.part[idx] = den > 0.f ? kLn2 * __builtin_fmaf(M, a.c, fast_log2(den)) : -__builtin_inff();
    }
}

// Reductions over every SEG consecutive lanes (16, 32 or 64) of a wavefront, every lane ends with its segment's result:
// DPP inside the 16-lane rows, then lane-permute swaps across the rows; no LDS traffic.
template <int SEG = 64>
__device__ __forceinline__ float wave_max(float v) {
    v = vmax(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
    v = vmax(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
    v = vmax(v, dpp_mov<0x141>(v));  // row_half_mirror
    v = vmax(v, dpp_mov<0x140>(v));  // row_mirror
    if constexpr (SEG == 16) return v;
    if constexpr (SEG == 64) return xrow_max4(v);
    auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
    return vmax(as_f32(a[0]), as_f32(a[1]));
}
template <int SEG = 64>
__device__ __forceinline__ float wave_sum(float v) {
    v = row16_sum(v);
    if constexpr (SEG == 16) return v;
    if constexpr (SEG == 64) return xrow_sum4(v);
    auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
    return as_f32(a[0]) + as_f32(a[1]);
}
// Sum of the lanes of equal index in the wave's segments of SEG lanes.
template <int SEG>
__device__ __forceinline__ float sum_segments(float v) {
    if constexpr (SEG == 16) v = xrow_sum4(v);
    if constexpr (SEG == 32) {
        auto a = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
        v = as_f32(a[0]) + as_f32(a[1]);
    }
    return v;
}
// log-sum-exp of x[lo .. hi).  A round of up to four values (1024 tokens in the score pass's chunks; four parts of any length
// where the many-row kernels noted them) is read in one go.
__device__ __forceinline__ float lse_range(const float* x, int lo, int hi) {
    if (hi <= lo) return -__builtin_inff();
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = x[min(lo + j, hi - 1)];
    float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
    for (int k = lo + 4; k < hi; ++k) mx = fmaxf(mx, x[k]);
    if (hi - lo == 1 || mx == -__builtin_inff()) return mx;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) s += lo + j < hi ? __expf(v[j] - mx) : 0.f;
    for (int k = lo + 4; k < hi; ++k) s += __expf(x[k] - mx);
    return mx + __logf(s);
}

// The finishing kernels.  They are latency: a few kilobytes per sequence on one compute unit, and what they cost is the
// chain of memory and LDS round trips one behind the other and the instructions of that unit's sixteen waves.  So
//   * a wave asks for the rows of all the heads (or query tokens) it finishes at once, before the round lengths have
//     arrived, and finds the rounds' places by a prefix sum over its own lanes (up to 64 rounds): no barrier;
//   * a lane owns a round, and short dialogues (up to 32, up to 16 rounds) put two or four heads into one wave, in
//     segments of SEG lanes;
//   * the barriers are for LDS only: they do not wait for the stores of the per-head scores.
// With one head per wave at a time, its row asked for when its turn came, the one-token kernel took 8.4 microseconds for
// one sequence of 12 rounds and 32 heads and 16.7 for 64 of 50 rounds and 64 heads (with the selection, which had 2 and 6
// of them); now 4.4 and 12.8, and the head kernel of a 128-token question 13.6 -> 7.0 microseconds.

// f(k) for the rounds per lane that a view of R_max rounds has, k < KPL, four at a time: a group past R_max is skipped by a
// scalar branch, which also keeps the compiler from fetching all sixteen ahead.  (With every one of sixteen unrolled, and
// sixteen waves a workgroup, the one-token and head kernels spilled 70 to 176 registers: 300 rounds, the head kernel 53.1
// microseconds for 8 dialogues of one token and 68.6 for 4 of 128 tokens, now 7.5 and 20.8.)
template <int KPL, typename F>
__device__ __forceinline__ void for_rounds(int R_max, F f) {
#pragma unroll
    for (int k0 = 0; k0 < KPL; k0 += 4)
        if (k0 == 0 || 64 * k0 < R_max) {
#pragma unroll
            for (int k = k0; k < (KPL < 4 ? KPL : k0 + 4); ++k) f(k);
        }
}

// Where the values of the rounds r = (lane mod SEG) + SEG k lie in a row: [lo[k], hi[k]), empty for r >= R.  `cum` is LDS
// for the prefix sum over more than 64 rounds.  Returns the values of all history rounds.  Called by all threads.
template <int SEG, int KPL>
__device__ __forceinline__ int round_places(const FinishArgs& a, int b, int& R, int* cum, int (&lo)[KPL], int (&hi)[KPL]) {
    const int j = threadIdx.x & (SEG - 1);
    const int round_up = (1 << a.chunk_shift) - 1;
    if constexpr (KPL == 1) {
        const int len = j < a.R_max ? a.seg_len[(size_t)b * a.R_max + j] : 0;  // asked for before R has arrived
        R = min(max(a.n_rounds[b], 0), a.R_max);
        const int nc = j < R ? (max(len, 0) + round_up) >> a.chunk_shift : 0;
        hi[0] = wave_inclusive_sum<SEG>(nc);
        lo[0] = hi[0] - nc;
        return __builtin_amdgcn_readlane(hi[0], SEG - 1);
    } else {
        static_assert(KPL == 1 || SEG == 64, "more than 64 rounds take whole waves");
        R = min(max(a.n_rounds[b], 0), a.R_max);
        for (int r = threadIdx.x; r < a.R_max; r += blockDim.x) {
            const int len = a.seg_len[(size_t)b * a.R_max + r];
            if (r < R) cum[r] = (max(len, 0) + round_up) >> a.chunk_shift;
        }
        exclusive_scan_units(cum, R);
#pragma unroll
        for (int k = 0; k < KPL; ++k) lo[k] = hi[k] = 0;
        for_rounds<KPL>(a.R_max, [&](int k) {
            const int r = j + 64 * k;
            lo[k] = r < R ? cum[r] : 0;
            hi[k] = r < R ? cum[r + 1] : 0;
        });
        return R > 0 ? cum[R] : 0;
    }
}

// The same by the streaming kernel's notes: the rounds' values and the current round's.  Returns whether the caller's
// max_tokens was too small for the sequence.
template <int SEG, int KPL>
__device__ __forceinline__ bool noted_places(const FinishArgs& a, int b, int& R, int (&lo)[KPL], int (&hi)[KPL], int& cur_lo, int& cur_hi) {
    const int j = threadIdx.x & (SEG - 1);
    auto ask = [&](int k, int& len, PlaceNote& note) {
        const int r = j + SEG * k;
        len = r < a.R_max ? a.seg_len[(size_t)b * a.R_max + r] : 0;
        note = r < a.R_max ? a.places.round[(size_t)b * a.R_max + r] : PlaceNote{0, 0};
    };
    int chunks = 0;
    auto place = [&](int k, int len, PlaceNote note) {
        const int r = j + SEG * k;
        const bool some = r < R && len > 0;
        lo[k] = some ? r + note.first : 0;
        hi[k] = some ? r + note.last + 1 : 0;
        chunks += some ? (len + 255) >> 8 : 0;
    };
    PlaceNote cur = {0, 0};
    if (a.has_cur) cur = a.places.cur[b];
    if constexpr (KPL == 1) {
        int len;
        PlaceNote note;
        ask(0, len, note);  // before R has arrived
        R = min(max(a.n_rounds[b], 0), a.R_max);
        place(0, len, note);
    } else {
        R = min(max(a.n_rounds[b], 0), a.R_max);
#pragma unroll
        for (int k = 0; k < KPL; ++k) lo[k] = hi[k] = 0;
        for_rounds<KPL>(a.R_max, [&](int k) {
            int len;
            PlaceNote note;
            ask(k, len, note);
            place(k, len, note);
        });
    }
    cur_lo = R + cur.first;
    cur_hi = R + cur.last + 1;
    chunks = __builtin_amdgcn_readlane(wave_inclusive_sum<SEG>(chunks), SEG - 1);
    return chunks + (a.has_cur ? (a.cur_len + 255) >> 8 : 0) > a.places.chunk_limit;
}

// n consecutive floats of memory into the wave's LDS strip, 512 of them in flight at a time.
__device__ __forceinline__ void stage_floats(const float* src, int n, float* strip) {
    const int lane = threadIdx.x & 63;
    for (int c0 = 0; c0 < n; c0 += 512) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + 64 * u + lane;
            v[u] = c < n ? src[c] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + 64 * u + lane;
            if (c < n) strip[c] = v[u];
        }
    }
}

// Probability mass of the rounds (lane mod SEG) + SEG k for one query token and head from its row of log-sum-exps:
// softmax over the history rounds and, if has_cur, the current round's values behind them.  Zeros where the token sees
// no key; groups of rounds past R_max are left as they are.
template <int SEG, int KPL>
__device__ __forceinline__ void round_masses(int R_max, const float* row, const int (&lo)[KPL], const int (&hi)[KPL],
                                             bool has_cur, int cur_lo, int cur_hi, float (&e)[KPL]) {
    float mx = -__builtin_inff();
    if constexpr (KPL > 4) {
        // Dialogues of so many rounds have one value for most of them, two where a range of tiles ends inside: all of those
        // are fetched before any is used (behind a branch per round every one is a round trip of its own).
        // Four rounds' at a time: all sixteen, and registers spill.
        bool more = false;
#pragma unroll
        for (int k0 = 0; k0 < KPL; k0 += 4) {
            if (k0 > 0 && 64 * k0 >= R_max) continue;
            float a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = row[lo[k0 + j]];
                b[j] = row[max(hi[k0 + j] - 1, 0)];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = hi[k0 + j] - lo[k0 + j];
                const float top = fmaxf(a[j], b[j]), two = top + __logf(1.f + __expf(fminf(a[j], b[j]) - top));
                e[k0 + j] = n <= 0 ? -__builtin_inff() : (n == 1 || top == -__builtin_inff() ? a[j] : two);
                more |= n > 2;
            }
        }
        if (__any(more))
            for_rounds<KPL>(R_max, [&](int k) {
                if (hi[k] - lo[k] > 2) e[k] = lse_range(row, lo[k], hi[k]);
            });
        for_rounds<KPL>(R_max, [&](int k) { mx = fmaxf(mx, e[k]); });
    } else {
        for_rounds<KPL>(R_max, [&](int k) {
            e[k] = lse_range(row, lo[k], hi[k]);
            mx = fmaxf(mx, e[k]);
        });
    }
    const float lc = has_cur ? lse_range(row, cur_lo, cur_hi) : -__builtin_inff();
    mx = fmaxf(wave_max<SEG>(mx), lc);
    const bool none = mx == -__builtin_inff();
    float sum = 0.f;
    for_rounds<KPL>(R_max, [&](int k) {
        e[k] = none ? 0.f : __expf(e[k] - mx);
        sum += e[k];
    });
    const float z = wave_sum<SEG>(sum) + (none ? 1.f : __expf(lc - mx));
    const float inv = 1.f / z;
    for_rounds<KPL>(R_max, [&](int k) { e[k] *= inv; });
}

// One query token per sequence: grid (B), 4 to 16 waves.  A wave takes groups of P = 64 / SEG consecutive heads: group w,
// w + W, ..., with the rows of HB groups asked for together.  P goes to p_out [B][Hq][R_max] if wanted; the head mean
// is accumulated per wave in registers and reduced over the waves through LDS in a fixed order.
constexpr int kFinishWaves = 8;              // of the kernels that finish a head per workgroup
// Most waves of the kernels that finish a sequence per workgroup.  With sixteen a wave has 128 registers, too few for sixteen
// rounds per lane.
__host__ __device__ constexpr int most_head_waves(int KPL) { return KPL > 4 ? 8 : kSelectWaves; }
constexpr size_t kFinishLdsMax = 96 * 1024;  // dynamic LDS of a finishing kernel (the selection's 13 KB come on top)

template <int SEG, int KPL, int HB, bool STAGED>
__global__ __launch_bounds__(most_head_waves(KPL) * 64) void scores_finish_kernel(FinishArgs a) {
    constexpr int P = 64 / SEG;
    extern __shared__ __align__(16) char smem[];
    int* cum = reinterpret_cast<int*>(smem);                       // [R_max + 2] chunk prefix of the history rounds
    float* hs = reinterpret_cast<float*>(smem) + (a.R_max + 2);    // [W][R_max] per-wave head sums
    const int W = blockDim.x >> 6;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int seg = lane / SEG, rl = lane & (SEG - 1);
    const int n = a.n_chunks_max;
    float* strip = hs + W * a.R_max + (size_t)wave * HB * P * n;  // [HB][P][n] of this wave if staged
    const float* part_b = a.part + (size_t)b * a.Hq * n;
    float av[HB][KPL];  // running masses of earlier calls
    auto fetch = [&](int h0) {
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int hj = h0 + j * W * P, h = hj + seg;
            for_rounds<KPL>(a.R_max, [&](int k) {
                const int r = rl + SEG * k;
                av[j][k] = a.acc && h < a.Hq && r < a.R_max ? a.acc[((size_t)b * a.Hq + h) * a.R_max + r] : 0.f;
            });
            if constexpr (STAGED)
                if (hj < a.Hq) stage_floats(part_b + (size_t)hj * n, min(P, a.Hq - hj) * n, strip + j * P * n);
        }
        __builtin_amdgcn_wave_barrier();  // same wave: LDS operations complete in program order
    };
    fetch(wave * P);
    int R, lo[KPL], hi[KPL];
    const int hist_chunks = round_places<SEG, KPL>(a, b, R, cum, lo, hi);
    const int cur_chunks = a.has_cur ? (a.cur_len + (1 << a.chunk_shift) - 1) >> a.chunk_shift : 0;
    const bool overflow = hist_chunks + cur_chunks > n;

    float hsum[KPL];
#pragma unroll
    for (int k = 0; k < KPL; ++k) hsum[k] = 0.f;
    for (int h0 = wave * P; h0 < a.Hq; h0 += HB * W * P) {
        if (h0 != wave * P) fetch(h0);
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int hj = h0 + j * W * P, h = hj + seg;
            if (hj >= a.Hq) continue;
            const bool mine = h < a.Hq;  // a segment past the last head repeats the group's first one, unused
            const int hs_in = mine ? seg : 0;
            float qatt[KPL];
            if (!overflow)
                round_masses<SEG>(a.R_max, STAGED ? strip + (j * P + hs_in) * n : part_b + (size_t)(hj + hs_in) * n, lo, hi, a.has_cur,
                                  hist_chunks, hist_chunks + cur_chunks, qatt);
            float tot = 0.f;
            for_rounds<KPL>(a.R_max, [&](int k) {
                const int r = rl + SEG * k;
                if (overflow) qatt[k] = 0.f;
                if (a.acc && !overflow && r < R && mine) {
                    qatt[k] += av[j][k];
                    a.acc[((size_t)b * a.Hq + h) * a.R_max + r] = qatt[k];
                }
                tot += qatt[k];
            });
            tot = wave_sum<SEG>(tot);
            const float inv = tot > 0.f ? 1.f / tot : 0.f;
            for_rounds<KPL>(a.R_max, [&](int k) {
                const int r = rl + SEG * k;
                // a max_tokens that understates the cache would leave chunks unscored: make that loud
                const float val = overflow ? __builtin_nanf("") : (r < R ? qatt[k] * inv : 0.f);
                hsum[k] += mine ? val : 0.f;
                if (a.p_out && mine && r < a.R_max) a.p_out[((size_t)b * a.Hq + h) * a.R_max + r] = val;
            });
        }
    }
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        const int r = rl + SEG * k;
        const float sum = sum_segments<SEG>(hsum[k]);
        if (seg == 0 && r < a.R_max) hs[wave * a.R_max + r] = sum;
    }
    lds_barrier();
    const float inv_h = 1.f / (float)a.Hq;
    float* svec = reinterpret_cast<float*>(cum);  // the sequence's scores, for the selection (cum is no longer read)
    for (int r = tid; r < a.R_max; r += W * 64) {
        float s = 0.f;
#pragma unroll 4
        for (int w = 0; w < W; ++w) s += hs[w * a.R_max + r];
        const float val = s * inv_h;
        a.s_out[(size_t)b * a.R_max + r] = val;
        if (a.with_select) svec[r] = val;
    }
    if (a.with_select) {  // Sec. 3.3 on the scores just written, same bits
        __shared__ SelectShared sh;
        lds_barrier();
        select_rounds_block(svec, R, a.R_max, a.sel, a.sel_idx + (size_t)b * a.R_max, a.n_sel + b, sh);
    }
}

// Several query tokens: grid (B, Hq, Z), eight waves.  Z workgroups per (sequence, head); wave w of workgroup z takes
// the groups of P = 64 / SEG consecutive query tokens 8 z + w, + 8 Z, ..., the rows of TB groups asked for together.  The
// per-wave round masses are summed over the waves in LDS in a fixed order and written, not yet normalised, to p_part
// [B][Hq][Z][R_max]; scores_heads_kernel finishes.
template <int SEG, int KPL, int TB, bool STAGED, bool NOTED>
__global__ __launch_bounds__(kFinishWaves * 64) void scores_finish_rows_kernel(FinishArgs a, float* p_part) {
    constexpr int P = 64 / SEG;
    extern __shared__ __align__(16) char smem[];
    int* cum = reinterpret_cast<int*>(smem);                        // [R_max + 2]
    float* hs = reinterpret_cast<float*>(smem) + (a.R_max + 2);     // [kFinishWaves][R_max]
    const int b = blockIdx.x, h = blockIdx.y;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int seg = lane / SEG, rl = lane & (SEG - 1);
    const int n = a.n_chunks_max;
    float* strip = hs + kFinishWaves * a.R_max + (size_t)wave * TB * P * n;  // [TB][P][n] if staged
    const float* part_h = a.part + ((size_t)b * a.Hq + h) * a.q_len * n;
    const int step = kFinishWaves * gridDim.z * P;
    auto fetch = [&](int i0) {
        if constexpr (STAGED) {
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                const int ij = i0 + j * step;
                if (ij < a.q_len) stage_floats(part_h + (size_t)ij * n, min(P, a.q_len - ij) * n, strip + j * P * n);
            }
            __builtin_amdgcn_wave_barrier();  // same wave: LDS operations complete in program order
        }
    };
    const int i_first = (blockIdx.z * kFinishWaves + wave) * P;
    fetch(i_first);
    int R, lo[KPL], hi[KPL], cur_lo, cur_hi;
    bool overflow;
    if constexpr (NOTED) {
        overflow = noted_places<SEG, KPL>(a, b, R, lo, hi, cur_lo, cur_hi);
    } else {
        cur_lo = round_places<SEG, KPL>(a, b, R, cum, lo, hi);
        cur_hi = cur_lo + (a.has_cur ? (a.cur_len + (1 << a.chunk_shift) - 1) >> a.chunk_shift : 0);
        overflow = cur_hi > n;
    }

    float qatt[KPL];
#pragma unroll
    for (int k = 0; k < KPL; ++k) qatt[k] = 0.f;
    for (int i0 = i_first; i0 < a.q_len && !overflow; i0 += TB * step) {
        if (i0 != i_first) fetch(i0);
        for (int j = 0; j < TB; ++j) {
            const int ij = i0 + j * step;
            if (ij >= a.q_len) break;
            const bool mine = ij + seg < a.q_len;  // a segment past the last token repeats the group's first one, unused
            const int in = mine ? seg : 0;
            float e[KPL];
            round_masses<SEG>(a.R_max, STAGED ? strip + (j * P + in) * n : part_h + (size_t)(ij + in) * n, lo, hi, a.has_cur,
                              cur_lo, cur_hi, e);
            for_rounds<KPL>(a.R_max, [&](int k) { qatt[k] += mine ? e[k] : 0.f; });
        }
    }
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        const int r = rl + SEG * k;
        const float sum = sum_segments<SEG>(qatt[k]);
        if (seg == 0 && r < a.R_max) hs[wave * a.R_max + r] = sum;
    }
    lds_barrier();
    for (int r = tid; r < a.R_max; r += kFinishWaves * 64) {
        float tot = 0.f;
        if (r < R)
#pragma unroll
            for (int w = 0; w < kFinishWaves; ++w) tot += hs[w * a.R_max + r];
        p_part[(((size_t)b * a.Hq + h) * gridDim.z + blockIdx.z) * a.R_max + r] = overflow ? __builtin_nanf("") : tot;
    }
}

// One query token whose heads have many values per round (the watershed layer's, one per 32-token tile): grid (B, Hq),
// eight waves share the rounds, four at a time each, and a wave folds a round's values with all its lanes.  The rounds'
// log-sum-exps meet in LDS, the first wave turns them into masses; output as above with Z = 1.
template <int KPL>
__global__ __launch_bounds__(kFinishWaves * 64) void scores_finish_tiles_kernel(FinishArgs a, float* p_part) {
    extern __shared__ __align__(16) char smem[];
    int* cum = reinterpret_cast<int*>(smem);                                // [R_max + 2]
    float* round_lse = reinterpret_cast<float*>(smem) + (a.R_max + 2);      // [R_max]
    const int b = blockIdx.x, h = blockIdx.y;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    int R, lo[KPL], hi[KPL];
    const int hist_chunks = round_places<64, KPL>(a, b, R, cum, lo, hi);
    const bool overflow = hist_chunks > a.n_chunks_max;
    if (!overflow) {
        const float* row = a.part + ((size_t)b * a.Hq + h) * a.n_chunks_max;
        for (int r0 = wave; r0 < R; r0 += 4 * kFinishWaves) {
            int first[4], end[4];
            float v[4], mx[4], sum[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = r0 + j * kFinishWaves;
                first[j] = end[j] = 0;
                if (r < R) {
                    if constexpr (KPL == 1) {
                        first[j] = __builtin_amdgcn_readlane(lo[0], r);
                        end[j] = __builtin_amdgcn_readlane(hi[0], r);
                    } else {
                        first[j] = cum[r];
                        end[j] = cum[r + 1];
                    }
                }
                v[j] = first[j] + lane < end[j] ? row[first[j] + lane] : -__builtin_inff();
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mx[j] = v[j];
                for (int c = first[j] + 64 + lane; c < end[j]; c += 64) mx[j] = fmaxf(mx[j], row[c]);
                mx[j] = wave_max(mx[j]);
                const bool none = mx[j] == -__builtin_inff();
                sum[j] = none ? 0.f : __expf(v[j] - mx[j]);
                if (!none)
                    for (int c = first[j] + 64 + lane; c < end[j]; c += 64) sum[j] += __expf(row[c] - mx[j]);
                sum[j] = wave_sum(sum[j]);
                if (lane == 0 && r0 + j * kFinishWaves < R)
                    round_lse[r0 + j * kFinishWaves] = none ? mx[j] : mx[j] + __logf(sum[j]);
            }
        }
    }
    lds_barrier();
    if (wave != 0) return;
    float lv[KPL], mx = -__builtin_inff(), sum = 0.f;
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        const int r = lane + 64 * k;
        lv[k] = !overflow && r < R ? round_lse[r] : -__builtin_inff();
        mx = fmaxf(mx, lv[k]);
    }
    mx = wave_max(mx);
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        lv[k] = mx == -__builtin_inff() ? 0.f : __expf(lv[k] - mx);
        sum += lv[k];
    }
    sum = wave_sum(sum);
    const float inv = sum > 0.f ? 1.f / sum : 0.f;
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        const int r = lane + 64 * k;
        if (r < a.R_max) p_part[((size_t)b * a.Hq + h) * a.R_max + r] = overflow ? __builtin_nanf("") : lv[k] * inv;
    }
}

// grid (B), 4 to 16 waves: per head, the Z partial round masses are added in order and normalised over the rounds
// (Eq. 1; written to p_out [B][Hq][R_max] if given); scores[b][r] is the mean over heads.  Heads go to waves and lanes as
// in the one-token kernel, so all sums run in a fixed order.
struct HeadsSelect {
    bool with_select;
    ra_select_params sel;
    const int32_t* n_rounds;
    int32_t* sel_idx;
    int32_t* n_sel;
};
constexpr int kMaxSplits = 8;  // most partial masses per head (scores_finish_splits)
template <int SEG, int KPL, int HB>
__global__ __launch_bounds__(most_head_waves(KPL) * 64) void scores_heads_kernel(const float* p_part, int Z, int R_max, int Hq, float* p_out,
                                                            float* s_out, float* acc, HeadsSelect hsel) {
    constexpr int P = 64 / SEG;
    extern __shared__ __align__(16) char smem[];
    float* sacc = reinterpret_cast<float*>(smem);  // [W][R_max]
    const int W = blockDim.x >> 6;
    const int b = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int seg = lane / SEG, rl = lane & (SEG - 1);
    float mine[KPL];  // this wave's sum over its heads of the normalised masses of this lane's rounds
#pragma unroll
    for (int k = 0; k < KPL; ++k) mine[k] = 0.f;
    for (int h0 = wave * P; h0 < Hq; h0 += HB * W * P) {
        float tot[HB][KPL];
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int h = h0 + j * W * P + seg;
            const float* ph = p_part + ((size_t)b * Hq + (h < Hq ? h : 0)) * Z * R_max;
            if constexpr (KPL <= 4) {  // every part of every round asked for at once
#pragma unroll
                for (int k = 0; k < KPL; ++k) {
                    const int r = rl + SEG * k;
                    const bool ok = h < Hq && r < R_max;
                    float v[kMaxSplits];
#pragma unroll
                    for (int z = 0; z < kMaxSplits; ++z) v[z] = ok && z < Z ? ph[(size_t)z * R_max + r] : 0.f;
                    tot[j][k] = 0.f;
#pragma unroll
                    for (int z = 0; z < kMaxSplits; ++z) tot[j][k] += v[z];
                }
            } else {
#pragma unroll
                for (int k = 0; k < KPL; ++k) tot[j][k] = 0.f;
                for (int z = 0; z < Z; ++z)
                    for_rounds<KPL>(R_max, [&](int k) {
                        const int r = rl + SEG * k;
                        tot[j][k] += h < Hq && r < R_max ? ph[(size_t)z * R_max + r] : 0.f;
                    });
            }
        }
#pragma unroll
        for (int j = 0; j < HB; ++j) {
            const int h = h0 + j * W * P + seg;
            float all = 0.f;
            for_rounds<KPL>(R_max, [&](int k) {
                const int r = rl + SEG * k;
                if (acc && h < Hq && r < R_max && tot[j][k] == tot[j][k]) {  // (an undersized pass leaves the running masses alone)
                    float* slot = acc + ((size_t)b * Hq + h) * R_max + r;
                    tot[j][k] += *slot;
                    *slot = tot[j][k];
                }
                all += tot[j][k];
            });
            all = wave_sum<SEG>(all);
            const float inv = all > 0.f ? 1.f / all : (all == all ? 0.f : all);  // (NaN marks an undersized pass)
            for_rounds<KPL>(R_max, [&](int k) {
                const int r = rl + SEG * k;
                const float p = tot[j][k] * inv;
                if (p_out && h < Hq && r < R_max) p_out[((size_t)b * Hq + h) * R_max + r] = p;
                mine[k] += p;  // (zero for a segment past the last head)
            });
        }
    }
#pragma unroll
    for (int k = 0; k < KPL; ++k) {
        const int r = rl + SEG * k;
        const float sum = sum_segments<SEG>(mine[k]);
        if (seg == 0 && r < R_max) sacc[wave * R_max + r] = sum;
    }
    lds_barrier();
    const float inv_h = 1.f / (float)Hq;
    for (int r = threadIdx.x; r < R_max; r += blockDim.x) {
        float s = 0.f;
#pragma unroll 4
        for (int w = 0; w < W; ++w) s += sacc[w * R_max + r];
        const float val = s * inv_h;
        s_out[(size_t)b * R_max + r] = val;
        if (hsel.with_select) sacc[r] = val;  // (a thread only ever touches its own column r of sacc)
    }
    if (hsel.with_select) {  // Sec. 3.3 on the scores just written, same bits
        __shared__ SelectShared sh;
        lds_barrier();
        const int R = min(max(hsel.n_rounds[b], 0), R_max);
        select_rounds_block(sacc, R, R_max, hsel.sel, hsel.sel_idx + (size_t)b * R_max, hsel.n_sel + b, sh);
    }
}

template <typename T, int D, int G>
static void launch_scores(bool paged, dim3 grid, size_t smem, hipStream_t st, const ScoreArgs& a) {
    if (paged)
        RA_LAUNCH_TIMED((scores_stream_kernel<T, D, G, true>), grid, dim3(256), smem, st, a);
    else
        RA_LAUNCH_TIMED((scores_stream_kernel<T, D, G, false>), grid, dim3(256), smem, st, a);
}

template <typename T, int D>
static int dispatch_scores(int G, bool paged, dim3 grid, size_t smem, hipStream_t st, const ScoreArgs& a) {
    switch (G) {
        case 1: launch_scores<T, D, 1>(paged, grid, smem, st, a); return RA_OK;
        case 2: launch_scores<T, D, 2>(paged, grid, smem, st, a); return RA_OK;
        case 4: launch_scores<T, D, 4>(paged, grid, smem, st, a); return RA_OK;
        case 8: launch_scores<T, D, 8>(paged, grid, smem, st, a); return RA_OK;
        default: return fail(RA_ERR_UNSUPPORTED, "round_scores: Hq / Hkv = %d not in {1, 2, 4, 8}", G);
    }
}

}  // namespace ra

using namespace ra;

namespace ra {
// Several query tokens: Z workgroups per (sequence, head) leave partial round masses in p_part
// [B][Hq][Z][R_max], a second kernel adds, normalises and averages them.
int scores_finish_splits(int q_len, int B, int Hq) {
    int Z = q_len / 32 < 1 ? 1 : (q_len / 32 > kMaxSplits ? kMaxSplits : q_len / 32);
    while (Z > 1 && (int64_t)B * Hq * Z > 2048) --Z;
    return Z;
}

// Lanes a head's rounds take in the finishing kernels, and rounds per lane.
#define RA_FINISH_SHAPE(R_max, LAUNCH)                            \
    do {                                                          \
        if ((R_max) <= 16) LAUNCH(16, 1);                         \
        else if ((R_max) <= 32) LAUNCH(32, 1);                    \
        else if ((R_max) <= 64) LAUNCH(64, 1);                    \
        else if ((R_max) <= 256) LAUNCH(64, 4);                   \
        else LAUNCH(64, kMaxRounds / 64);                         \
    } while (0)

// Waves of a workgroup that finishes `groups` groups of heads of one sequence: 4 to `most`, and as the LDS allows.
static int head_waves(int groups, int most, int R_max) {
    int W = groups < 4 ? 4 : (groups > most ? most : groups);
    while (W > 4 && (size_t)(W + 1) * (R_max + 2) * sizeof(float) > kFinishLdsMax) --W;
    return W;
}

template <int SEG, int KPL, int TB, bool NOTED>
static void launch_rows(const FinishArgs& f, int B, float* p_part, int Z, hipStream_t st) {
    const size_t base = (size_t)(f.R_max + 2) * sizeof(int) + (size_t)kFinishWaves * f.R_max * sizeof(float);
    const size_t staged = base + (size_t)kFinishWaves * TB * (64 / SEG) * f.n_chunks_max * sizeof(float);
    const dim3 grid(B, f.Hq, Z), block(kFinishWaves * 64);
    if (staged <= kFinishLdsMax / 2)  // two workgroups per compute unit
        hipLaunchKernelGGL((scores_finish_rows_kernel<SEG, KPL, TB, true, NOTED>), grid, block, staged, st, f, p_part);
    else if (TB > 1)
        launch_rows<SEG, KPL, 1, NOTED>(f, B, p_part, Z, st);
    else
        hipLaunchKernelGGL((scores_finish_rows_kernel<SEG, KPL, 1, false, NOTED>), grid, block, base, st, f, p_part);
}

template <int SEG, int KPL, int HB>
static void launch_heads(const FinishArgs& f, int B, const float* p_part, int Z, hipStream_t st) {
    HeadsSelect hsel;
    hsel.with_select = f.with_select;
    hsel.sel = f.sel;
    hsel.n_rounds = f.n_rounds;
    hsel.sel_idx = f.sel_idx;
    hsel.n_sel = f.n_sel;
    const int W = head_waves((f.Hq * SEG + 63) / 64, most_head_waves(KPL), f.R_max);
    hipLaunchKernelGGL((scores_heads_kernel<SEG, KPL, HB>), dim3(B), dim3(W * 64), (size_t)W * f.R_max * sizeof(float), st,
                       p_part, Z, f.R_max, f.Hq, f.p_out, f.s_out, f.acc, hsel);
}

void launch_scores_finish_rows(const FinishArgs& f, int B, float* p_part, int Z, hipStream_t st) {
    if (f.q_len == 1 && !f.has_cur) {
        const dim3 grid(B, f.Hq), block(kFinishWaves * 64);
        const size_t smem = (size_t)(2 * f.R_max + 2) * sizeof(int);
        if (f.R_max <= 64) hipLaunchKernelGGL((scores_finish_tiles_kernel<1>), grid, block, smem, st, f, p_part);
        else if (f.R_max <= 256) hipLaunchKernelGGL((scores_finish_tiles_kernel<4>), grid, block, smem, st, f, p_part);
        else hipLaunchKernelGGL((scores_finish_tiles_kernel<kMaxRounds / 64>), grid, block, smem, st, f, p_part);
    } else {
        const bool several = f.q_len > kFinishWaves * Z;  // a wave may have more than one group of tokens
#define RA_ROWS(SEG, KPL)                                                              \
    do {                                                                               \
        constexpr int several_tb = (KPL) == 1 ? 4 : 1;                                 \
        if (f.places.round && several) launch_rows<SEG, KPL, several_tb, true>(f, B, p_part, Z, st); \
        else if (f.places.round) launch_rows<SEG, KPL, 1, true>(f, B, p_part, Z, st);  \
        else if (several) launch_rows<SEG, KPL, several_tb, false>(f, B, p_part, Z, st); \
        else launch_rows<SEG, KPL, 1, false>(f, B, p_part, Z, st);                     \
    } while (0)
        RA_FINISH_SHAPE(f.R_max, RA_ROWS);
#undef RA_ROWS
    }
#define RA_HEADS(SEG, KPL) launch_heads<SEG, KPL, (SEG) == 64 && (KPL) == 1 ? 2 : 1>(f, B, p_part, Z, st)
    RA_FINISH_SHAPE(f.R_max, RA_HEADS);
#undef RA_HEADS
}

// One query token: the finishing kernel for B sequences (f.q_len must be 1).  As many of a wave's groups of heads
// fetched together as it has and as their rows fit into LDS; rows that do not fit even so are read from memory.
template <int SEG, int KPL, int HB>
static void launch_single(const FinishArgs& f, int B, hipStream_t st) {
    const int groups = (f.Hq * SEG + 63) / 64, W = head_waves(groups, most_head_waves(KPL), f.R_max);
    const size_t base = (size_t)(f.R_max + 2) * sizeof(int) + (size_t)W * f.R_max * sizeof(float);
    const size_t staged = base + (size_t)W * HB * (64 / SEG) * f.n_chunks_max * sizeof(float);
    if (HB > 1 && (groups <= W * (HB / 2) || staged > kFinishLdsMax))
        launch_single<SEG, KPL, (HB > 1 ? HB / 2 : 1)>(f, B, st);
    else if (staged <= kFinishLdsMax)
        hipLaunchKernelGGL((scores_finish_kernel<SEG, KPL, HB, true>), dim3(B), dim3(W * 64), staged, st, f);
    else
        hipLaunchKernelGGL((scores_finish_kernel<SEG, KPL, 1, false>), dim3(B), dim3(W * 64), base, st, f);
}
void launch_scores_finish_single(const FinishArgs& f, int B, hipStream_t st) {
#define RA_SINGLE(SEG, KPL) launch_single<SEG, KPL, (KPL) == 1 && (SEG) == 64 ? 4 : (KPL) <= 4 ? 2 : 1>(f, B, st)
    RA_FINISH_SHAPE(f.R_max, RA_SINGLE);
#undef RA_SINGLE
}
void launch_scores_finish(const FinishArgs& f, int B, float* p_part, hipStream_t st) {
    if (scores_finish_by_rows(f.q_len, f.Hq, f.n_chunks_max))
        launch_scores_finish_rows(f, B, p_part, scores_finish_splits(f.q_len, B, f.Hq), st);
    else
        launch_scores_finish_single(f, B, st);
}
}  // namespace ra

static int scores_impl(ra_ctx* ctx, void* stream, const void* q, int q_len, int Hq, const ra_kv_view* watershed,
                       const void* cur_k, int cur_len, float scale, float* acc, float* scores_head, float* scores,
                       const ra_select_params* sel = nullptr, int32_t* sel_idx = nullptr, int32_t* n_sel = nullptr) {
    RA_REQUIRE(ctx != nullptr, RA_ERR_INVALID_ARG, "round_scores: ctx is NULL");
    RA_REQUIRE(q != nullptr && scores != nullptr, RA_ERR_INVALID_ARG, "round_scores: q or scores is NULL");
    if (int rc = check_view(watershed, false, "round_scores")) return rc;
    RA_REQUIRE(q_len > 0, RA_ERR_INVALID_ARG, "round_scores: q_len must be positive");
    RA_REQUIRE(Hq > 0 && Hq % watershed->Hkv == 0, RA_ERR_INVALID_ARG,
               "round_scores: Hq %d is not a multiple of Hkv %d", Hq, watershed->Hkv);
    RA_REQUIRE(cur_len >= 0 && (cur_k != nullptr) == (cur_len > 0), RA_ERR_INVALID_ARG,
               "round_scores: cur_k and cur_len > 0 must be given together");
    RA_REQUIRE(cur_k == nullptr || cur_len >= q_len, RA_ERR_INVALID_ARG,
               "round_scores: the q_len query tokens are the tail of the current round, so cur_len >= q_len");
    RA_REQUIRE(scale > 0.f && scale == scale, RA_ERR_INVALID_ARG, "round_scores: scale must be positive");
    RA_REQUIRE(watershed->R_max > 0, RA_ERR_INVALID_ARG, "round_scores: R_max is 0, there is nothing to score");
    if (sel) {
        RA_REQUIRE(sel_idx != nullptr && n_sel != nullptr, RA_ERR_INVALID_ARG, "round_scores_select: sel_idx or n_sel is NULL");
        if (int rc = check_select_params(sel, "round_scores_select")) return rc;
    }
    const int G = Hq / watershed->Hkv, D = watershed->d, B = watershed->B, R_max = watershed->R_max;
    RA_REQUIRE(D == 64 || D == 128, RA_ERR_UNSUPPORTED, "round_scores: head_dim %d not in {64, 128}", D);
    RA_REQUIRE((int64_t)B * q_len <= 65535, RA_ERR_UNSUPPORTED, "round_scores: B * q_len exceeds 65535");

    // With a single query token the current round's share of the softmax cancels in the
    // normalisation over history rounds, so its keys need not be read at all -- unless the masses are
    // added to those of other tokens, each with its own share.
    const bool use_cur = cur_k != nullptr && (q_len > 1 || acc != nullptr);
    bool mfma = watershed->dtype == RA_BF16 && D == 128;
    const int chunk_tokens = kChunkTokens;
    const int64_t nc64 = watershed->max_tokens / chunk_tokens + R_max + (use_cur ? (cur_len + chunk_tokens - 1) / chunk_tokens : 0);
    RA_REQUIRE(nc64 <= (int64_t)1 << 24, RA_ERR_UNSUPPORTED, "round_scores: max_tokens too large");
    const int n_chunks_max = (int)(nc64 < 1 ? 1 : nc64);
    const size_t rows = (size_t)B * Hq * q_len;
    size_t part_bytes = align_up(rows * n_chunks_max * sizeof(float), 256);
    // several query tokens (or many chunks): Z workgroups per head leave partial round masses in a buffer
    const size_t p_bytes = scores_finish_part_bytes(q_len, B, Hq, R_max, n_chunks_max);
    // more than 16 query rows per KV head on the matrix cores: persistent kernel driven by segment tables
    const bool many_rows = mfma && q_len * G > 16;
    if (mfma) RA_REQUIRE(G <= 16, RA_ERR_UNSUPPORTED, "round_scores: Hq / Hkv = %d exceeds 16", G);
    if (many_rows) RA_REQUIRE(B <= kMaxBatch, RA_ERR_UNSUPPORTED, "round_scores: batch %d exceeds %d", B, kMaxBatch);
    const size_t plan_bytes = many_rows ? align_up((size_t)B * plan_stride(R_max + 1), 256) : 0;
    // few rows on the matrix cores: one 16-byte descriptor per (sequence, chunk)
    size_t desc_bytes = mfma && !many_rows ? align_up((size_t)B * n_chunks_max * 16, 256) : 0;
    // 64 channels run there too as long as there are few rows, the descriptors fit and the 16-byte loads are aligned
    // (16 dialogues of 12 000 tokens, 196 MB of keys: 63 -> 33 microseconds); the generic kernel takes what is left
    if (watershed->dtype == RA_BF16 && D == 64 && q_len * G <= 16 && (G & (G - 1)) == 0 && G <= 8 &&
        (((uintptr_t)q | (uintptr_t)watershed->k | (uintptr_t)cur_k) & 15) == 0) {
        const size_t bytes = align_up((size_t)B * n_chunks_max * 16, 256);
        mfma = ctx->ws.base != nullptr && ctx->ws.bytes >= kWsReserved + part_bytes + p_bytes + bytes;
        if (mfma) desc_bytes = bytes;
    }
    RA_REQUIRE(ctx->ws.base != nullptr && ctx->ws.bytes >= kWsReserved + part_bytes + p_bytes + plan_bytes + desc_bytes,
               RA_ERR_WORKSPACE, "round_scores: workspace has %zu bytes, this call needs %zu", ctx->ws.bytes,
               kWsReserved + part_bytes + p_bytes + plan_bytes + desc_bytes);

    ScoreArgs a;
    int row_len = n_chunks_max;
    a.view = to_dev(watershed);
    a.q_len = q_len;
    a.Hq = Hq;
    a.num_cu = ctx->num_cu;
    if (many_rows) {
        // A value for every round (and the current one) and for every further part that a sequence is cut into, no more
        // than the workspace has room for: the least that passed the check above has room for one part.
        a.max_tiles = watershed->max_tokens / 32 + R_max + (use_cur ? (cur_len + 31) / 32 : 0);
        const int slots = R_max + (use_cur ? 1 : 0);
        const size_t room = (ctx->ws.bytes - kWsReserved - p_bytes - plan_bytes) / 256 * 256 / (rows * sizeof(float));
        scores_prefill_shape(a, (long long)room - slots + 1);
        row_len = slots + a.S - 1;
        part_bytes = align_up(rows * row_len * sizeof(float), 256);
        a.places = {reinterpret_cast<PlaceNote*>(scores), reinterpret_cast<PlaceNote*>(ctx->ws.base + kWsPlacesOff), n_chunks_max};
    }
    a.q = q;
    a.cur_k = use_cur ? cur_k : nullptr;
    a.cur_len = use_cur ? cur_len : 0;
    a.n_chunks_max = row_len;
    a.chunk_tokens = chunk_tokens;
    a.c = scale * kLog2e;
    a.part = reinterpret_cast<float*>(ctx->ws.base + kWsReserved);
    a.plan = ctx->ws.base + kWsReserved + part_bytes + p_bytes;
    a.chunks = desc_bytes ? ctx->ws.base + kWsReserved + part_bytes + p_bytes + plan_bytes : nullptr;

    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const dim3 grid(n_chunks_max, watershed->Hkv, B * q_len);
    const size_t tab_bytes = (size_t)(R_max + 1) * 16 + 16;
    const bool paged = watershed->block_size != 0;
    int rc;
    {
        KernelTimer timer(ctx, st);
        if (many_rows)
            rc = launch_scores_prefill_mfma(a, paged, st);
        else if (mfma)
            rc = launch_scores_mfma(a, paged, ctx->num_cu, st);
        else if (watershed->dtype == RA_BF16)
            rc = dispatch_scores<BF16, 64>(G, paged, grid, tab_bytes, st, a);
        else
            rc = D == 128 ? dispatch_scores<F32, 128>(G, paged, grid, tab_bytes, st, a)
                          : dispatch_scores<F32, 64>(G, paged, grid, tab_bytes, st, a);
    }
    if (rc) return rc;

    FinishArgs f;
    f.part = a.part;
    f.n_rounds = watershed->n_rounds;
    f.seg_len = watershed->seg_len;
    f.R_max = R_max;
    f.Hq = Hq;
    f.q_len = q_len;
    f.cur_len = a.cur_len;
    f.n_chunks_max = row_len;
    f.chunk_shift = 8;
    f.places = a.places;
    f.has_cur = use_cur;
    f.p_out = scores_head;
    f.s_out = scores;
    f.acc = acc;
    if (sel) {
        f.with_select = true;
        f.sel = *sel;
        f.sel_idx = sel_idx;
        f.n_sel = n_sel;
    }
    launch_scores_finish(f, B, reinterpret_cast<float*>(ctx->ws.base + kWsReserved + part_bytes), st);
    RA_HIP_CHECK(hipGetLastError());
    return RA_OK;
}

extern "C" int ra_round_scores(ra_ctx* ctx, void* stream, const void* q, int q_len, int Hq,
                               const ra_kv_view* watershed, const void* cur_k, int cur_len, float scale,
                               float* scores_head, float* scores) {
    return scores_impl(ctx, stream, q, q_len, Hq, watershed, cur_k, cur_len, scale, nullptr, scores_head, scores);
}

extern "C" int ra_round_scores_accumulate(ra_ctx* ctx, void* stream, const void* q, int q_len, int Hq,
                                          const ra_kv_view* watershed, const void* cur_k, int cur_len, float scale,
                                          float* acc, float* scores_head, float* scores) {
    RA_REQUIRE(acc != nullptr, RA_ERR_INVALID_ARG, "round_scores_accumulate: acc is NULL");
    return scores_impl(ctx, stream, q, q_len, Hq, watershed, cur_k, cur_len, scale, acc, scores_head, scores);
}

extern "C" int ra_round_scores_select(ra_ctx* ctx, void* stream, const void* q, int q_len, int Hq,
                                      const ra_kv_view* watershed, const void* cur_k, int cur_len, float scale,
                                      const ra_select_params* params, float* scores_head, float* scores,
                                      int32_t* sel_idx, int32_t* n_sel) {
    RA_REQUIRE(params != nullptr, RA_ERR_INVALID_ARG, "round_scores_select: params is NULL");
    return scores_impl(ctx, stream, q, q_len, Hq, watershed, cur_k, cur_len, scale, nullptr, scores_head, scores, params,
                       sel_idx, n_sel);
}
