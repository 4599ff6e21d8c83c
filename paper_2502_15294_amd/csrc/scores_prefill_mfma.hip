// Round scores (paper Sec. 3.1, Eq. 1) for a question of many tokens: streaming pass over the watershed
// layer's keys for bf16 / head_dim 128 on the matrix cores, many query rows per KV head.
//
// Same roles as in the attention kernels: S^T[16 tokens x 16 rows] = K . Q^T, lane%16 is the query row, so a
// row's running (reference logit, sum of exponentials) stays in its lane.  What is produced is one
// log-sum-exp per query row and part of a round: the key tiles of the batch are cut into ranges, a range may end
// anywhere inside a round, and every (round, range) that meet leave one value a row (score_places.hpp says
// where).  The finishing kernels turn those into round masses.
//
//   * a work item is (range of the batch's key tiles, KV head, block of 256 query rows): four waves with
//     four 16-row tiles each walk the range's tiles in lockstep;
//   * every 32-token key tile (8 KB) is fetched from global memory once per workgroup, one tile ahead, with
//     whole-row coalesced loads that go straight into one of two LDS buffers (no registers, no LDS stores): the
//     tile's image there is row-major with the 16-byte chunks of row r rotated by r, so that the operand reads
//     (16 lanes = 16 rows, one chunk) touch every bank once; all four waves read it; one barrier per tile;
//   * the reference logit of a lane is only raised when the exponentials of a tile relative to it add up to more than
//     2^16, so the common tile costs one multiply-add, one exponential and one add per logit;
//   * persistent launch with the batch-wide balanced schedule used by the attention kernels, in units of key tiles.  (With
//     one value per 256-token chunk of a round a range had to begin and end with a chunk: ranges of eight tiles, as a short
//     question has them, then came out between none and seventeen tiles long, and their ends spread from 12 to 32
//     microseconds.  19 tokens over three dialogues of 23 rounds, whole call 76.1 -> 71.3 microseconds; 128 tokens over four
//     of 32 000 tokens 324.5 -> 313; 24 tokens over three of 17 rounds at the watershed layer 49.8 -> 43.7.)
#include "scores_common.hpp"
#include "score_places.hpp"
#include "mfma_util.hpp"
#include "stream_kv.hpp"

#include <type_traits>

namespace ra {

constexpr int kTileSP = 32;                      // tokens per key tile
constexpr int kNTS = 4;                          // 16-row tiles per wave
constexpr int kRowsPerItemS = 4 * kNTS * 16;     // 256
constexpr int kKTileBytes = 8192;
constexpr int kPiecesPerWorkgroupS = 1;  // measured on the 4 x 32 K-token question-prefill workload: 1: 167-172 us, 2: 174-180, 3: 176
constexpr int kWorkgroupsPerCuS = 3;

// Planning kernel, grid (B): the table of segments of sequence b (all history rounds, then the current round)
// in the layout the attention kernels use, with cum = prefix sum of the segments' key-tile counts and U = total key tiles.
__global__ __launch_bounds__(256) void scores_plan_kernel(ScoreArgs a, char* plan) {
    extern __shared__ __align__(16) char smem[];
    const DevView& vw = a.view;
    const int b = blockIdx.x, tid = threadIdx.x;
    const int cap = vw.R_max + 1;
    int* cum = reinterpret_cast<int*>(smem);  // [cap + 1] tiles
    char* plan_b = plan + (size_t)b * plan_stride(cap);
    long long* g_off_k = reinterpret_cast<long long*>(plan_b + sizeof(PlanHeader));
    long long* g_off_v = g_off_k + cap;
    int* g_len = reinterpret_cast<int*>(g_off_v + cap);
    int* g_cum = g_len + cap;
    const int n_hist = min(max(vw.n_rounds[b], 0), vw.R_max);
    const int n_slots = n_hist + (a.cur_k && a.cur_len > 0 ? 1 : 0);
    for (int i = tid; i < cap; i += 256) {
        int len = 0;
        long long ok = 0;
        if (i < n_hist) {
            len = max(vw.seg_len[(size_t)b * vw.R_max + i], 0);
            ok = vw.seg_off[(size_t)b * vw.R_max + i];
        } else if (i < n_slots) {
            len = a.cur_len;
        }
        g_len[i] = len;
        g_off_k[i] = ok;
        g_off_v[i] = 0;
        cum[i] = (len + kTileSP - 1) / kTileSP;
    }
    exclusive_scan_units(cum, cap);
    for (int i = tid; i <= cap; i += 256) g_cum[i] = cum[i];
    if (tid == 0) {
        PlanHeader h;
        h.n_slots = n_slots;
        h.n_hist = n_hist;
        h.U = cum[n_slots];
        h.S_eff = 1;
        *reinterpret_cast<PlanHeader*>(plan_b) = h;
    }
}

// INLINE_PLAN: the workgroup reads the batch's segment lists and plans itself (small batches, no planning kernel before).
// RAGGED: some wave of some row block has fewer than four row tiles.  (A variant of its own: with the choice of tile counts
// in its loop the kernel takes 205 instead of 194 microseconds for the 512 rows of a 128-token question, which need none.)
template <bool PAGED, bool INLINE_PLAN, bool RAGGED>
__global__ __launch_bounds__(256, kWorkgroupsPerCuS) void scores_prefill_mfma_kernel(ScoreArgs a, int n_rowblocks) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int sU[INLINE_PLAN ? kInlineBatch : kMaxBatch], sps[INLINE_PLAN ? 1 : kMaxBatch + 1];
    __shared__ typename std::conditional<INLINE_PLAN, TileRanges, int>::type ranges;
    const DevView& vw = a.view;
    const int Hkv = vw.Hkv;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, n = lane & 15, q4 = lane >> 4;
    const int G = a.Hq / Hkv, q_len = a.q_len;
    const int rows_total = q_len * G;
    const RowsPerToken per_token(G);

    const int cap = vw.R_max + 1;
    SlotTable tab;
    tab.carve(smem, cap);
    char* tiles = smem + ((SlotTable::bytes(cap) + 15) & ~(size_t)15);  // two key-tile buffers
    const unsigned tiles_lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(lptr_t)tiles);

    const int inner = Hkv * n_rowblocks;
    int P;
    BatchLists lists;
    if constexpr (INLINE_PLAN) {
        lists.load(tiles + 2 * kKTileBytes, vw, nullptr, nullptr, [&](int) { return a.cur_k ? a.cur_len : 0; });
        lists.count_tiles(vw.B, sU);
        P = cut_tiles<kWorkgroupsPerCuS>(ranges, sU, vw.B, a.slots, a.min_units, a.max_parts,
                                         !PAGED && gridDim.x >= kWorkgroupsPerCuS * (unsigned)a.num_cu &&
                                             a.slots * inner <= (int)gridDim.x,
                                         score_range_weights());
    } else {
        const int slots = max((int)gridDim.x * kPiecesPerWorkgroupS / inner, 1);
        P = build_schedule(a.plan, cap, vw.B, a.S, a.min_units, slots, sU, sps);
    }

    const char* kbase = reinterpret_cast<const char*>(vw.k);
    const char* ck = reinterpret_cast<const char*>(a.cur_k);
    const int n_items = P * inner;
    // The exponentials of a tile are taken against the reference as it stands and their sum tells whether it was too low (on a
    // range's first tile it is infinite); then the reference is raised and they are taken again.  A maximum of the logits
    // beforehand was a fifth of the common tile's vector instructions (16 dialogues, 40 tokens: whole call 171 -> 168.5
    // microseconds, one of 60 rounds, 200 tokens: 140 -> 137).
    constexpr float kRaise = 65536.f;
    // row blocks of equal size (to within one 16-row tile)
    const int row_tiles = (rows_total + 15) / 16, tiles_per_block = (row_tiles + n_rowblocks - 1) / n_rowblocks;
    auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    auto uni64 = [&](long long x) { return ((long long)uni((int)(x >> 32)) << 32) | (unsigned)uni((int)x); };

    // One pass per (item, sequence that its range meets); planned apart an item is a piece of one sequence.  A single loop:
    // with the passes in a loop of their own the compiler keeps what only depends on the item in registers all through.
    int reached = 0;  // tiles of the item's range that earlier passes took end here
    bool first = true;
    for (int item = blockIdx.x; item < n_items;) {
        const int piece = uni(item / inner), rest = item - piece * inner;
        const int rowblock = uni(rest / Hkv), g = rest - rowblock * Hkv;
        int b, part, t_lo, t_hi;  // the pass: tiles [t_lo, t_hi) of sequence b, its part-th piece
        if constexpr (INLINE_PLAN) {
            const int r = range_at<kWorkgroupsPerCuS>(piece, P);
            const LaneSequence sq = lane_sequence(sU, vw.B);
            const int g_lo = max(uni(ranges.bound[r]), reached), g_hi = uni(ranges.bound[r + 1]);
            if (g_lo >= g_hi) {  // (an empty range)
                item += gridDim.x;
                continue;
            }
            b = sequence_of_tile(sq, vw.B, g_lo);
            part = r - first_part_of(ranges, P, sq, b);
            const int seq_lo = __builtin_amdgcn_readlane(sq.tile0, b), end = min(g_hi, seq_lo + __builtin_amdgcn_readlane(sq.U, b));
            t_lo = g_lo - seq_lo;
            t_hi = end - seq_lo;
            reached = end < g_hi ? end : 0;
        } else {
            b = uni(find_slot(sps, vw.B, piece));
            part = piece - sps[b];
            t_lo = piece_begin(sU[b], part, sps[b + 1] - sps[b]);
            t_hi = piece_begin(sU[b], part + 1, sps[b + 1] - sps[b]);
        }
        if (reached == 0) item += gridDim.x;

        // The block's 16-row tiles are dealt out to the waves in turn: row nt of this lane is row0 + 64 nt (whatever else is
        // needed of it is recomputed where it is used).
        const int wv = (wave + rowblock + piece) & 3;  // not always the same SIMD gets the odd tile
        const int row0 = (rowblock * tiles_per_block + wv) * 16 + n;
        const int my_tiles = !RAGGED ? 4 : (min(tiles_per_block, row_tiles - rowblock * tiles_per_block) - wv + 3) >> 2;
        uint4 qf[kNTS][4];  // asked for before the table is built
#pragma unroll
        for (int nt = 0; nt < kNTS; ++nt) {
            if (nt >= my_tiles) continue;
            const int row = row0 + nt * 64;
            const int rr = row < rows_total ? row : 0;
            const int qtok = per_token.token(rr);
            const size_t qrow = ((size_t)b * q_len + qtok) * a.Hq + (size_t)g * G + (rr - qtok * G);
            const uint4* qp = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.q) + qrow * 256);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qf[nt][kk] = qp[kk * 4 + q4];  // rows past the last repeat row 0, unused
        }
        float m[kNTS], l[kNTS];  // reference logit times a.c, sum of the exponentials relative to it
#pragma unroll
        for (int nt = 0; nt < kNTS; ++nt) {
            m[nt] = kNegBig;
            l[nt] = 0.f;
        }

        int n_slots, n_hist;
        if (!INLINE_PLAN || !first) __syncthreads();  // the previous pass's readers of the table and the tile buffers are done
        first = false;
        if constexpr (INLINE_PLAN) {
            n_hist = uni(lists.meta[3 * b + 1]);
            n_slots = n_hist + (uni(lists.meta[3 * b + 2]) > 0 ? 1 : 0);
            lists.table(b, tab);
        } else {
            const PlanHeader hdr = load_plan(a.plan + (size_t)b * plan_stride(cap), cap, tab);
            n_slots = uni(hdr.n_slots);
            n_hist = uni(hdr.n_hist);
            __syncthreads();
        }
        if (t_lo >= t_hi) continue;  // (a sequence without keys)

        // Uniform state of the loader: the segment it stands in (the table in LDS is read on entry only), and
        // inside it the next tile: the address of its first token's keys (head g) and the tokens left from there.
        int seg_len = 0, seg_end = 0, rows_left = 0;
        bool seg_cur = false;
        const char *seg_k = nullptr, *tile_k = nullptr;  // contiguous history / current round
        long long seg_tab = 0;                           // paged history: first block-table slot
        unsigned kstride = 256;                          // bytes from one token's keys to the next
        BlockWindow blocks;
        if constexpr (PAGED) blocks.open(vw, b);
        // This wave fills rows 8 wave .. + 7 of the tile's LDS image (row = token of the tile, 256 bytes) with two
        // loads of four whole rows each, 16 lanes per row; lane L's 16 bytes land at position L % 16 of its row,
        // where chunk (L % 16 - row) mod 16 belongs.
        const int row_a = 8 * wave + q4;                 // this lane helps to load tile rows row_a and row_a + 4
        const unsigned chunk_a = (unsigned)((n - row_a) & 15) * 16u, chunk_b = (unsigned)((n - row_a - 4) & 15) * 16u;
        unsigned off_a = 0, off_b = 0;                   // byte offsets from tile_k for a full tile
        auto open_seg = [&](int slot, int t) {  // ... and stand at its tile of the sequence's tile t
            seg_len = uni(tab.len[slot]);
            const int tok0 = (t - uni(tab.cum[slot])) * kTileSP;
            seg_end = uni(tab.cum[slot + 1]);
            seg_cur = slot >= n_hist;
            kstride = seg_cur ? (unsigned)Hkv * 256u : 256u;
            if (seg_cur)
                seg_k = ck + ((size_t)b * a.cur_len * Hkv + g) * 256;
            else if (PAGED)
                seg_tab = uni64(tab.off_k[slot]);
            else
                seg_k = kbase + ((size_t)uni64(tab.off_k[slot]) * Hkv + (size_t)g * seg_len) * 256;
            off_a = (unsigned)row_a * kstride + chunk_a;
            off_b = (unsigned)(row_a + 4) * kstride + chunk_b;
            rows_left = seg_len - tok0;
            tile_k = reinterpret_cast<const char*>(uni64(reinterpret_cast<long long>(seg_k + (size_t)tok0 * kstride)));
        };
        // This wave's quarter (rows 8*wave .. +7) of the next key tile goes to the buffer at LDS address `buf_lds`;
        // afterwards the loader stands at the tile that follows.  Rows past the segment's end re-read its last row
        // (their scores are masked).
        auto load_tile = [&](unsigned buf_lds) {
            const unsigned kd = buf_lds + 8 * wave * 256;
            if (!seg_cur && PAGED) {
                const int tok0 = seg_len - rows_left;
                const int blk = min((tok0 >> 4) + (wave >> 1), (seg_len - 1) >> 4);
                const int pb = blocks.block(seg_tab + blk);
                const char* kb = reinterpret_cast<const char*>(uni64(reinterpret_cast<long long>(kbase + ((size_t)pb * Hkv + g) * 4096)));
                const int last_row = seg_len - 1 - blk * 16;
                const int r0 = min(8 * (wave & 1) + q4, last_row), r1 = min(8 * (wave & 1) + 4 + q4, last_row);
                load_to_lds(kb, (unsigned)r0 * 256u + chunk_a, kd);
                load_to_lds(kb, (unsigned)r1 * 256u + chunk_b, kd + 1024);
            } else if (rows_left >= kTileSP) {
                load_to_lds(tile_k, off_a, kd);
                load_to_lds(tile_k, off_b, kd + 1024);
            } else {
                load_to_lds(tile_k, (unsigned)min(row_a, rows_left - 1) * kstride + chunk_a, kd);
                load_to_lds(tile_k, (unsigned)min(row_a + 4, rows_left - 1) * kstride + chunk_b, kd + 1024);
            }
            rows_left -= kTileSP;
            tile_k += (size_t)kTileSP * kstride;
        };
        // N: row tiles of this wave (1 .. 4)
        auto consume = [&](auto n_tiles, const char* buf, int tok0, int len, bool is_cur) {
            constexpr int N = decltype(n_tiles)::value;
            const bool full = !is_cur && (len - tok0 >= kTileSP);
            const uint4* kb = reinterpret_cast<const uint4*>(buf);
            floatx4_t sc[N][2];
            uint4 kf[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) kf[h][kk] = kb[(h * 16 + n) * 16 + ((kk * 4 + q4 + n) & 15)];
            asm volatile("" ::: "memory");  // all eight fragment reads are in flight before the first product is issued
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)  // the four row tiles' chains interleaved: no instruction waits for the one before
#pragma unroll
                    for (int nt = 0; nt < N; ++nt)
                        sc[nt][h] = mfma16(kf[h][kk], qf[nt][kk], kk ? sc[nt][h] : floatx4_t{0.f, 0.f, 0.f, 0.f});
            if (!full) {
#pragma unroll
                for (int nt = 0; nt < N; ++nt) {
                    // tokens of this segment the row may see (causal inside the current round)
                    const int lim = is_cur ? cur_visible(len, q_len, per_token.token(min(row0 + nt * 64, rows_total - 1))) : len;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (tok0 + h * 16 + q4 * 4 + i >= lim) sc[nt][h][i] = -__builtin_inff();
                }
            }
            auto masses = [&](int nt) {  // sum of the exponentials of this lane's eight logits of row tile nt
                float p[8];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) p[h * 4 + i] = fast_exp2(__builtin_fmaf(sc[nt][h][i], a.c, -m[nt]));
                return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
            };
            float sum[N];
            bool raise = false;
#pragma unroll
            for (int nt = 0; nt < N; ++nt) {
                sum[nt] = masses(nt);
                raise |= sum[nt] > kRaise;
            }
            if (__any(raise)) {  // each lane keeps its own reference: the four lane groups of a row are merged per chunk
#pragma unroll
                for (int nt = 0; nt < N; ++nt) {
                    const float m_new = vmax(m[nt], max8(sc[nt][0], sc[nt][1]) * a.c);
                    l[nt] *= fast_exp2(m[nt] - m_new);
                    m[nt] = m_new;
                    sum[nt] = masses(nt);
                }
            }
#pragma unroll
            for (int nt = 0; nt < N; ++nt) l[nt] += sum[nt];
        };
        // End of a segment or of the range: merge the four lane groups of every row into the log-sum-exp of what the range
        // has of the segment.  It is stored behind the request for the tile after next (store_place): at once, the wait for
        // that tile's loads, which counts stores too, would sit out the whole trip of the stores.  The reference logit
        // stays: a later part's sum underflows only where its share of the row's softmax is below 2^-126.
        float done[kNTS];
        int done_slot = -1;
        auto finish_place = [&](int slot) {
#pragma unroll
            for (int nt = 0; nt < kNTS; ++nt) {
                const float M = xrow_max4(m[nt]);
                const float lv = xrow_sum4(l[nt] * fast_exp2(m[nt] - M));
                done[nt] = lv > 0.f ? kLn2 * (M + fast_log2(lv)) : -__builtin_inff();
                l[nt] = 0.f;
            }
            done_slot = slot;
        };
        auto store_place = [&]() {
            if (done_slot < 0) return;
            int first_row = row0;
            asm volatile("" : "+v"(first_row));  // the four rows' addresses are made here, not kept in eight registers all through
#pragma unroll
            for (int nt = 0; nt < kNTS; ++nt) {
                const int row = first_row + nt * 64;
                if (nt < my_tiles && row < rows_total && q4 == 0) {
                    const int qtok = per_token.token(row);
                    const size_t rowid = ((size_t)b * a.Hq + (size_t)g * G + (row - qtok * G)) * q_len + qtok;  // [B][Hq][q_len]
                    a.part[rowid * a.n_chunks_max + done_slot + part] = done[nt];
                }
            }
            done_slot = -1;
        };
        // ---- walk the key tiles [t_lo, t_hi): the whole workgroup in lockstep ----------------------------------
        int slot = find_slot_wave(tab.cum, n_slots, t_lo);
        const int slot_lo = slot;
        open_seg(slot, t_lo);
        int c_tok0 = seg_len - rows_left;
        load_tile(tiles_lds);
        int bufsel = 0;
        for (int t = t_lo; t < t_hi; ++t) {
            char* buf = tiles + bufsel * kKTileBytes;
            wait_for_direct_loads();  // this wave's quarter of the tile has landed in LDS
            // the tile just stored, as the consumer needs it
            const int c_len = seg_len, c_t = c_tok0, c_slot = slot;
            const bool c_cur = seg_cur, c_last = t + 1 == seg_end || t + 1 == t_hi;
            __syncthreads();
            if (t + 1 < t_hi) {
                if (t + 1 >= seg_end) {
                    do ++slot; while (t + 1 >= uni(tab.cum[slot + 1]));
                    open_seg(slot, t + 1);
                }
                c_tok0 = seg_len - rows_left;
                load_tile(tiles_lds + (bufsel ^ 1) * kKTileBytes);
            }
            store_place();
            if (!RAGGED || my_tiles == 4) consume(std::integral_constant<int, 4>(), buf, c_t, c_len, c_cur);
            else if (my_tiles == 3) consume(std::integral_constant<int, 3>(), buf, c_t, c_len, c_cur);
            else if (my_tiles == 2) consume(std::integral_constant<int, 2>(), buf, c_t, c_len, c_cur);
            else if (my_tiles == 1) consume(std::integral_constant<int, 1>(), buf, c_t, c_len, c_cur);
            if (c_last) finish_place(c_slot);
            bufsel ^= 1;
        }
        store_place();
        if (rest == 0 && wave == 0) note_places(a.places, b, vw.R_max, n_hist, tab.cum, slot_lo, slot, part, t_lo, t_hi);
    }
}


static void launch_scores_plan(const ScoreArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(scores_plan_kernel, dim3(a.view.B), dim3(256), (size_t)(a.view.R_max + 2) * sizeof(int), st, a,
                       const_cast<char*>(a.plan));
}

// A launch that plans itself cuts down to two tiles a range, so that small questions spread over the chip (25 rounds of 50
// tokens, 32 tokens of 64 heads, whole call 49.5 -> 43.0 microseconds against ranges of at least eight, 45.1 with four; 5 short
// rounds, 102 tokens of 8 heads 47.7 -> 41.0).  Planned apart the batch is large and shorter ranges only add starts (100
// dialogues, 16 tokens: 8 tiles 263.6, 2 tiles 268.0).
constexpr int kMinTilesInline = 2, kMinTilesPlanned = 8;

static size_t scores_prefill_lds(int B, int R_max, bool plan_inline) {
    return align_up(SlotTable::bytes(R_max + 1), 16) + 2 * kKTileBytes + (plan_inline ? BatchLists::bytes(B, R_max) : 0);
}

void scores_prefill_shape(ScoreArgs& a, long long room) {
    const int B = a.view.B, rows_total = a.q_len * (a.Hq / a.view.Hkv);
    a.n_rowblocks = (rows_total + kRowsPerItemS - 1) / kRowsPerItemS;
    const int inner = a.view.Hkv * a.n_rowblocks;
    for (int plan_inline = 1; plan_inline >= 0; --plan_inline) {
        a.plan_inline = plan_inline;
        a.min_units = plan_inline ? kMinTilesInline : kMinTilesPlanned;
        const long long most = B + B * a.max_tiles / a.min_units;  // ranges
        long long grid = (long long)kWorkgroupsPerCuS * a.num_cu;
        if (grid > most * inner) grid = most * inner;
        if (grid < 1) grid = 1;
        a.grid = (int)grid;
        a.slots = plan_inline ? question_slots(inner, grid, a.num_cu, false)
                              : (int)(grid * kPiecesPerWorkgroupS / inner < 1 ? 1 : grid * kPiecesPerWorkgroupS / inner);
        if (a.slots > kMaxRanges) a.slots = kMaxRanges;
        const long long of_eight = (a.max_tiles + kMinTilesPlanned - 1) / kMinTilesPlanned + 2;
        const long long parts = question_parts(a.max_tiles / a.min_units + 2, of_eight, a.slots, plan_inline ? B : 1);
        a.S = (int)(parts > room ? room : parts);
        a.max_parts = a.S >= a.slots ? kMaxRanges + 2 : a.S;
        if (plan_inline && a.max_parts > 2 && prefill_plans_inline(B, a.view.R_max, scores_prefill_lds(B, a.view.R_max, true), grid, a.num_cu))
            return;
    }
}

int launch_scores_prefill_mfma(const ScoreArgs& a, bool paged, hipStream_t st) {
    const int rows_total = a.q_len * (a.Hq / a.view.Hkv), n_rowblocks = a.n_rowblocks, grid = a.grid;
    const bool plan_inline = a.plan_inline != 0;
    const size_t smem = scores_prefill_lds(a.view.B, a.view.R_max, plan_inline);
    if (!plan_inline) launch_scores_plan(a, st);
    const int row_tiles = (rows_total + 15) / 16;
    const bool ragged = row_tiles != n_rowblocks * 4 * kNTS;
#define RA_SCORES_CASE(P_, I_, R_)                                                                                   \
    if (paged == P_ && plan_inline == I_ && ragged == R_)                                                            \
        RA_LAUNCH_TIMED((scores_prefill_mfma_kernel<P_, I_, R_>), dim3((unsigned)grid), dim3(256), smem, st, a, n_rowblocks);
    RA_SCORES_CASE(false, false, false) RA_SCORES_CASE(false, true, false) RA_SCORES_CASE(true, false, false)
    RA_SCORES_CASE(true, true, false) RA_SCORES_CASE(false, false, true) RA_SCORES_CASE(false, true, true)
    RA_SCORES_CASE(true, false, true) RA_SCORES_CASE(true, true, true)
#undef RA_SCORES_CASE
    return RA_OK;
}

}  // namespace ra
