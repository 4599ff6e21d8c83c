// Device-side building blocks of the bandwidth-bound streaming kernels (decode attention and
// decode-shape round scores): the per-workgroup table of round segments, the lane layout that
// reads K/V rows with full 16-byte-per-lane coalescing, and the wavefront-level reductions.
//
// Lane layout inside a 64-wide wavefront: the wave is four rows of 16 lanes.  Row `grp` works on
// one token at a time and lane `sub` of the row owns d/16 consecutive channels of that token, so
// one load instruction of the wave covers four consecutive token rows (1 KB for bf16, d = 128).
// A dot product is finished with four DPP adds inside the 16-lane row; nothing goes through LDS.
#pragma once

#include "common.hpp"
#include "tile_ranges.hpp"

#include <type_traits>

namespace ra {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float as_f32(uint32_t x) { return __builtin_bit_cast(float, x); }
__device__ __forceinline__ uint32_t as_u32(float x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
    return as_f32((uint32_t)__builtin_amdgcn_update_dpp(0, (int)as_u32(v), CTRL, 0xf, 0xf, false));
}
// Sum over the 16 lanes of a DPP row; every lane of the row ends with the total.
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);  // row_half_mirror
    v += dpp_mov<0x140>(v);  // row_mirror
    return v;
}
// Four sums over the 16 lanes of a row at once: lane i of the row ends with the total of d[i mod 4].  Eleven operations, where
// four sums that end in every lane take sixteen, and what follows is one value a lane, not four.
__device__ __forceinline__ float row16_sums(const float (&d)[4]) {
    const bool odd = threadIdx.x & 1, upper = threadIdx.x & 2;
    const float a = (odd ? d[1] : d[0]) + dpp_mov<0xB1>(odd ? d[0] : d[1]);  // quad_perm [1,0,3,2]
    const float b = (odd ? d[3] : d[2]) + dpp_mov<0xB1>(odd ? d[2] : d[3]);
    float v = (upper ? b : a) + dpp_mov<0x4E>(upper ? a : b);  // quad_perm [2,3,0,1]
    v += dpp_mov<0x124>(v);                                    // row_ror:4
    v += dpp_mov<0x128>(v);                                    // row_ror:8
    return v;
}
// Maxima are ordinary float code on purpose.  The compiler inserts the wait states that the hardware leaves to
// software (a vector instruction that reads the result of a matrix-core product still in flight, a DPP or lane-swap
// instruction that reads a register just written), and it does so only for instructions it can see: an asm
// statement with v_max_f32 inside gets none.  Such a statement here once read the previous tile's logits (on a
// wave's first tile: whatever the registers held before) whenever the scheduler happened to put it within a few
// instructions of the products: a reference logit that was still valid but differed from launch to launch, and with
// it the last bits of the outputs.  The price is a few copies that quiet signalling NaNs in front of some maxima.
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_fmaxf(a, b); }
// Reductions over the four 16-lane rows of a wavefront (lanes l, l^16, l^32, l^48); every lane ends with the
// result.  v_permlane16_swap / v_permlane32_swap applied to two copies of a value hand each lane the values of
// both rows of a pair (of both halves of the wave), so the exchange stays in the vector ALU.
__device__ __forceinline__ float xrow_max4(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
    v = vmax(as_f32(a[0]), as_f32(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
    return vmax(as_f32(b[0]), as_f32(b[1]));
}
__device__ __forceinline__ float xrow_sum4(float v) {
    auto a = __builtin_amdgcn_permlane16_swap(as_u32(v), as_u32(v), false, false);
    v = as_f32(a[0]) + as_f32(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(as_u32(v), as_u32(v), false, false);
    return as_f32(b[0]) + as_f32(b[1]);
}

// Element-type specific pieces.  A lane's share of one K or V row is WORDS 32-bit words.
struct F32 {};
struct BF16 {};
template <typename T, int EPL>
struct RowOps;

template <int EPL>
struct RowOps<F32, EPL> {
    static constexpr int WORDS = EPL;
    static constexpr int ELEM_BYTES = 4;
    __device__ static __forceinline__ float dot(const uint32_t* k, const uint32_t* q) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < WORDS; ++e) acc = __builtin_fmaf(as_f32(k[e]), as_f32(q[e]), acc);
        return acc;
    }
    __device__ static __forceinline__ void widen(const uint32_t* w, float* f) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) f[e] = as_f32(w[e]);
    }
};

template <int EPL>
struct RowOps<BF16, EPL> {
    static constexpr int WORDS = EPL / 2;
    static constexpr int ELEM_BYTES = 2;
    // Both operands are bf16, so every product is exact in fp32; accumulation is fp32.
    __device__ static __forceinline__ float dot(const uint32_t* k, const uint32_t* q) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < WORDS; ++e)
            acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, k[e]), __builtin_bit_cast(bf16x2_t, q[e]),
                                                  acc, false);
        return acc;
    }
    __device__ static __forceinline__ void widen(const uint32_t* w, float* f) {
#pragma unroll
        for (int e = 0; e < WORDS; ++e) {
            f[2 * e] = as_f32(w[e] << 16);
            f[2 * e + 1] = as_f32(w[e] & 0xffff0000u);
        }
    }
};

// Loads of data that a kernel reads exactly once, marked non-temporal so that the lines do not displace anything
// in the caches on their way through.  It pays where one load instruction of a wave covers whole cache lines: a
// plain read of 4 GiB reaches 7.0-7.1 TB/s this way against 5.9-6.2 TB/s with ordinary loads on the same MI355X (each
// wave streaming its own span, 16- or 8-byte loads, 512 or 1024 contiguous bytes per instruction), and the decode
// kernel's value tiles, which have that shape, took it from 212 to 194 microseconds on the large paged workload.
// It does not pay for key tiles read in the operand layout of the matrix cores (16 rows x 64 bytes per instruction,
// two instructions to a cache line): no change in the decode kernel, 738 -> 878 microseconds in the score kernel, which
// reads nothing else.  The score kernel therefore loads its keys as whole rows (four rows, eight cache lines per
// instruction) and turns them into the operand layout through LDS: 738 -> 732 microseconds for itself, and the
// kernels that follow find their tables still in the caches (decode at 6 % kept 95 -> 85 microseconds, the whole
// small-batch step 70 -> 66).  And the hint must not sit behind a run-time condition: written as `flag ? load_once(p) : *p`
// the decode kernel ran at 320 instead of 212 microseconds (the loads of a tile then sit in separate branches, and
// the two tiles the kernel keeps in flight no longer overlap).
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once(const uint4* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 load_once(const uint2* p) {
    const u32x2_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
    return make_uint2(v.x, v.y);
}

template <int WORDS>
struct Frag {
    uint32_t w[WORDS];
};

template <int WORDS>
__device__ __forceinline__ Frag<WORDS> load_frag(const char* p) {
    Frag<WORDS> f;
    if constexpr (WORDS == 2) {
        uint2 t = *reinterpret_cast<const uint2*>(p);
        f.w[0] = t.x;
        f.w[1] = t.y;
    } else {
#pragma unroll
        for (int i = 0; i < WORDS / 4; ++i) {
            uint4 t = reinterpret_cast<const uint4*>(p)[i];
            f.w[4 * i + 0] = t.x;
            f.w[4 * i + 1] = t.y;
            f.w[4 * i + 2] = t.z;
            f.w[4 * i + 3] = t.w;
        }
    }
    return f;
}

// ---- per-workgroup table of the round segments it may touch ------------------------------------
// slot i < n_hist is a history round, slot n_hist (if present) is the current round.  `cum` is the
// exclusive prefix sum of the segments' unit counts (a unit = 16 tokens, never crossing a segment).
struct SlotTable {
    long long* off_k;  // [cap]   segment start: tokens (contiguous) or block-table slots (paged)
    long long* off_v;  // [cap]
    int* len;          // [cap]
    int* cum;          // [cap + 1]
    __host__ __device__ static size_t bytes(int cap) { return (size_t)cap * 24 + 4; }
    __device__ void carve(char* smem, int cap) {
        off_k = reinterpret_cast<long long*>(smem);
        off_v = off_k + cap;
        len = reinterpret_cast<int*>(off_v + cap);
        cum = len + cap;
    }
};

// The table is built once per call and sequence by a small planning kernel and kept in global memory
// (header, then the four arrays with `cap` entries each, cum with cap + 1); the streaming kernels
// copy it to LDS with independent loads, so their workgroups start after a single memory round trip.
struct PlanHeader {
    int n_slots, n_hist, U, S_eff;  // U = total work units, S_eff = pieces the sequence is cut into
};
__host__ __device__ inline size_t plan_stride(int cap) { return (sizeof(PlanHeader) + SlotTable::bytes(cap) + 15) & ~(size_t)15; }

__device__ __forceinline__ PlanHeader load_plan(const char* plan_b, int cap, SlotTable& tab) {
    const PlanHeader hdr = *reinterpret_cast<const PlanHeader*>(plan_b);
    const long long* g_off_k = reinterpret_cast<const long long*>(plan_b + sizeof(PlanHeader));
    const long long* g_off_v = g_off_k + cap;
    const int* g_len = reinterpret_cast<const int*>(g_off_v + cap);
    const int* g_cum = g_len + cap;
    for (int i = threadIdx.x; i < cap; i += blockDim.x) {  // entries past n_slots are zero and unused
        tab.off_k[i] = g_off_k[i];
        tab.off_v[i] = g_off_v[i];
        tab.len[i] = g_len[i];
        tab.cum[i] = g_cum[i];
    }
    if (threadIdx.x == 0) tab.cum[cap] = g_cum[cap];
    return hdr;
}

// Inclusive prefix sum over every SEG consecutive lanes (16, 32 or 64) of a wave: shifts inside the rows of 16 lanes
// (zeros come in at a row's start), then the totals of the rows before added from scalar registers; no trip through LDS.
template <int SEG = 64>
__device__ __forceinline__ int wave_inclusive_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    const int lane = threadIdx.x & 63;
    if constexpr (SEG == 16) return v;
    const int t0 = __builtin_amdgcn_readlane(v, 15), t2 = __builtin_amdgcn_readlane(v, 47);
    if constexpr (SEG == 32) return v + (lane & 16 ? (lane & 32 ? t2 : t0) : 0);
    const int t1 = __builtin_amdgcn_readlane(v, 31);
    return v + (lane < 16 ? 0 : (lane < 32 ? t0 : (lane < 48 ? t0 + t1 : t0 + t1 + t2)));
}

// Barrier of a workgroup for what it exchanges through LDS: unlike __syncthreads it does not wait for outstanding
// global loads and for the acknowledgement of global stores, which no other wave of the workgroup reads.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exclusive prefix sum, in place, of cum[0..n) by the first wavefront; cum[n] receives the total.
// Must be called by all threads of the workgroup (it synchronises).
__device__ inline void exclusive_scan_units(int* cum, int n) {
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const int per = (n + 63) >> 6;
        const int base = lane * per;
        int sum = 0;
        for (int j = 0; j < per; ++j)
            if (base + j < n) sum += cum[base + j];
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            int t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        int excl = incl - sum;
        for (int j = 0; j < per; ++j)
            if (base + j < n) {
                int u = cum[base + j];
                cum[base + j] = excl;
                excl += u;
            }
        if (lane == 63) cum[n] = incl;
    }
    __syncthreads();
}

// ---- loads from global memory straight into LDS -----------------------------------------------------
typedef void __attribute__((address_space(3)))* lptr_t;
// 16 bytes per lane from global memory straight into LDS (global_load_lds_dwordx4): lane L's piece lands at
// lds + 16 * L, `lds` being an LDS byte address that is the same in all lanes (it travels in M0).  Written as
// instructions of their own because the compiler, given its builtin for them, makes every later LDS read wait for
// the load to land (it cannot tell the two tile buffers apart), which exposes the whole memory latency once per
// tile (measured: 180 against 157 microseconds); here the one wait sits where it belongs, before the barrier that
// publishes the buffer (wait_for_direct_loads).  The compiler's own vector-memory counts do not see these loads,
// which can only make one of its waits longer, never shorter: loads complete in order.
// An asm statement is opaque to the compiler's hazard handling, so the wait states the hardware leaves to software
// are written out here: a scalar write of M0 needs one before an instruction that takes its LDS address from M0
// (the compiler puts the same s_nop behind its own M0 writes), and an SGPR written by a vector instruction
// (v_readfirstlane, or v_readlane when the compiler reloads a spilled SGPR) needs five before a vector-memory
// instruction reads it as its base address: the form with a uniform base therefore waits s_nop 3, which with the
// M0 write makes five whatever came right before the statement.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is named as clobbered; the compiler sets it anew before each of its own uses
__device__ __forceinline__ void load_to_lds(const void* src, unsigned lds) {  // per-lane 64-bit address
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds) : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds(const char* base, unsigned off, unsigned lds) {  // uniform base + lane offset
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory", "m0");
}
// s_waitcnt vmcnt(0) (the other counters at their maxima: expcnt 7, lgkmcnt 15)
__device__ __forceinline__ void wait_for_direct_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }
// The same wait, for a load that is issued only on some paths and used after they meet.  Left to the compiler, the
// wait lands after the join and is a wait for everything (with a conditional load in between, the number of younger
// loads is no constant), on every pass; written into the branch, right behind the load, it is paid only there.
__device__ __forceinline__ void wait_for_loads_so_far() { __builtin_amdgcn_s_waitcnt(0x0f70); }
#pragma clang diagnostic pop

// Paged storage: the physical blocks of the tiles ahead, 64 block-table entries at a time in a wave's registers.  A look-up
// per tile is one more memory round trip before every tile's loads, in a wave that has nothing else to do meanwhile (question
// of 101 tokens over four paged dialogues of 32 000: score kernel 184 -> 175 microseconds, attention kernel 166 -> 155; of 128
// tokens over 16 of 8 500: 266 -> 246 and 222 -> 212).
struct BlockWindow {
    const int* table;  // the sequence's row of the block table
    int max_blocks;
    long long lo;  // slot of lane 0's entry
    int n, mine;
    __device__ __forceinline__ void open(const DevView& vw, int b) {
        table = vw.block_table + (size_t)b * vw.max_blocks;
        max_blocks = vw.max_blocks;
        lo = 0;
        n = 0;
    }
    __device__ __forceinline__ int block(long long slot) {  // uniform
        slot = min(max(slot, 0ll), (long long)max_blocks - 1);
        if (slot < lo || slot >= lo + n) {
            lo = slot;
            n = 64;
            mine = table[min(slot + (threadIdx.x & 63), (long long)max_blocks - 1)];
            wait_for_loads_so_far();  // here, once per window, not after the join on every tile
        }
        return max(__builtin_amdgcn_readlane(mine, (int)(slot - lo)), 0);
    }
};

// ---- balanced schedule of a whole batch ------------------------------------------------------------
// Every workgroup of a persistent attention launch derives the same schedule from the per-sequence
// unit counts U_b the planning kernel left in the plan headers: sequence b is cut into
//   n_b = clamp(ceil(U_b / T), 1, S)   pieces of about equal size whatever the selection sizes are.
// T is the smallest piece (>= min_units) for which the batch has no more than `slots` pieces: one piece more than the
// launch has workgroups for would run after all the others, alone on its compute unit and as long as they took
// together (T = ceil(sum U_b / slots) leaves up to B - 1 such pieces: score kernel of a 128-token question over 4 dialogues
// of 300 rounds 209 -> 171 microseconds, 16 of 100 rounds 240 -> 227, 24 of 50 rounds 247 -> 205).  With fewer than two
// slots a sequence the smallest such T is the length of a whole sequence, and T = ceil(sum U_b / slots) is taken (32
// dialogues of 40 rounds, 48 slots: 302 -> 222; 64 of 20 rounds, 96 slots: 159 -> 133), as above 64 sequences.
// sU[b] = U_b, sps = exclusive prefix of n_b (sps[B] = number of pieces).  Must be called by all threads of the
// workgroup.
__device__ inline int build_schedule(const char* plan, int cap, int B, int S, int min_units, int slots, int* sU, int* sps) {
    __shared__ int s_fit;
    const size_t stride = plan_stride(cap);
    if (threadIdx.x == 0) s_fit = 0x7fffffff;
    for (int b = threadIdx.x; b < B; b += blockDim.x)
        sps[b] = sU[b] = reinterpret_cast<const PlanHeader*>(plan + (size_t)b * stride)->U;
    exclusive_scan_units(sps, B);
    const int total = sps[B];
    auto pieces = [&](int U, int T) {
        const int nb = (int)(((unsigned)U + (unsigned)T - 1) / (unsigned)T);
        return nb < 1 ? 1 : (nb > S ? S : nb);
    };
    int T = (int)(((unsigned)total + (unsigned)slots - 1) / (unsigned)slots);
    if (T < min_units) T = min_units;
    if (B > 1 && B <= 64 && slots >= 2 * B) {
        // every thread tries one T between that and the one that fits for certain; the smallest that fits is taken
        const int most = (int)(((unsigned)total + (unsigned)(slots - B) - 1) / (unsigned)(slots - B));
        const int mine = T + (int)((unsigned)max(most - T, 0) * threadIdx.x / (blockDim.x - 1));
        int n = 0;
        for (int b = 0; b < B; ++b) n += pieces(sU[b], mine);
        if (n <= slots) atomicMin(&s_fit, mine);
        __syncthreads();
        if (s_fit != 0x7fffffff) T = s_fit;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += blockDim.x) sps[b] = pieces(sU[b], T);
    exclusive_scan_units(sps, B);
    return sps[B];
}

// Largest slot with cum[slot] <= u, for 0 <= u < cum[n].
template <typename T>
__device__ __forceinline__ int find_slot(const T* cum, int n, T u) {
    int lo = 0, hi = n;  // invariant: cum[lo] <= u < cum[hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (cum[mid] <= u) lo = mid; else hi = mid;
    }
    return lo;
}

// ---- planning inside a launch, for small batches ------------------------------------------------------
// The segment lists of the whole batch in LDS, read in one memory round trip: a kernel that has them needs no planning
// kernel before it and no second trip for the tables that one would have written.
// A launch that plans itself must still hold as many workgroups on a compute unit as it has for one: the lists, 24 bytes per
// (sequence, round), come on top of the table's.  (128-token question, one dialogue of 619 rounds: the score kernel, three
// to a unit, 78.9 microseconds behind the planning kernel and 109.4 with its own plan while only two of that fitted; 618
// rounds, of which three did, 84.3.  917 rounds: the attention kernel 93.5 and 114.2, two to a unit and one; 914: 74.6.)
constexpr size_t kLdsPerUnit = 160 * 1024, kLdsGranule = 1280;
__device__ constexpr int align16(int x) { return (x + 15) & ~15; }
struct BatchLists {
    long long *ok, *ov;  // [B][R_max] starts of the rounds' keys / values, by round index
    int *len, *sel;      // [B][R_max] tokens of the rounds; the listed rounds
    int* meta;           // [B][3] rounds of the sequence, listed rounds, length of the current round
    int R_max;
    __host__ __device__ static size_t bytes(int B, int R_max) { return ((size_t)B * R_max * 24 + (size_t)B * 12 + 15) & ~(size_t)15; }
    // sel_idx null: every round; cur_len(b): the current round's tokens.  All threads (256) call it; ends with a barrier.
    // One memory round trip: everything a thread reads is asked for before any of it is used.
    template <typename CurLen>
    __device__ __forceinline__ void load(char* smem, const DevView& vw, const int32_t* sel_idx, const int32_t* n_sel,
                                         CurLen cur_len) {
        R_max = vw.R_max;
        listed = sel_idx != nullptr;
        const int n = vw.B * R_max, tid = threadIdx.x;
        ok = reinterpret_cast<long long*>(smem);
        ov = ok + n;
        len = reinterpret_cast<int*>(ov + n);
        sel = len + n;
        meta = sel + n;
        int c_rounds = 0, c_sel = 0;
        if (tid < vw.B) {
            c_rounds = vw.n_rounds[tid];
            if (sel_idx) c_sel = n_sel[tid];
        }
        auto read = [&](auto per_thread) {
            constexpr int N = decltype(per_thread)::value;
            int l[N], s[N];
            long long k[N], v[N];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int i = min(tid + 256 * j, n - 1);
                l[j] = vw.seg_len[i];
                k[j] = vw.seg_off[i];
                v[j] = vw.seg_off_v[i];
                s[j] = sel_idx ? sel_idx[i] : 0;
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int i = tid + 256 * j;
                if (i < n) {
                    len[i] = l[j];
                    ok[i] = k[j];
                    ov[i] = v[j];
                    sel[i] = s[j];
                }
            }
        };
        if (n > 256) read(std::integral_constant<int, kInlineRounds / 256>());
        else if (n > 0) read(std::integral_constant<int, 1>());
        if (tid < vw.B) {
            const int n_rounds = min(max(c_rounds, 0), R_max);
            meta[3 * tid] = n_rounds;
            meta[3 * tid + 1] = sel_idx ? min(max(c_sel, 0), R_max) : n_rounds;
            meta[3 * tid + 2] = cur_len(tid);
        }
        __syncthreads();
    }
    // Segment i of sequence b's table, as the planning kernel defines it: the i-th listed round (entries that are not
    // rounds of the sequence count as empty), then the current round.
    __device__ __forceinline__ int entry(int b, int i, long long& k, long long& v) const {
        k = v = 0;
        if (i < meta[3 * b + 1]) {
            const int r = listed ? sel[b * R_max + i] : i;
            if (r < 0 || r >= meta[3 * b]) return 0;
            k = ok[b * R_max + r];
            v = ov[b * R_max + r];
            return max(len[b * R_max + r], 0);
        }
        return i == meta[3 * b + 1] ? max(meta[3 * b + 2], 0) : 0;
    }
    // Key tiles of every sequence into sU[0..B): a wave per sequence.  Ends with a barrier.
    __device__ __forceinline__ void count_tiles(int B, int* sU) const {
        const int lane = threadIdx.x & 63;
        for (int b = threadIdx.x >> 6; b < B; b += blockDim.x >> 6) {
            int tiles = 0;
            for (int i = lane; i <= R_max; i += 64) {
                long long k, v;
                tiles += (entry(b, i, k, v) + 31) >> 5;
            }
            tiles = __builtin_amdgcn_readlane(wave_inclusive_sum(tiles), 63);
            if (lane == 0) sU[b] = tiles;
        }
        lds_barrier();
    }
    // Sequence b's table by the first wave, cum the prefix of the segments' key tiles.  Ends with a barrier.
    __device__ __forceinline__ void table(int b, const SlotTable& tab) const {
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x, cap = R_max + 1;
            int t0 = 0;
            for (int i0 = 0; i0 < cap; i0 += 64) {
                const int i = i0 + lane;
                long long k = 0, v = 0;
                const int n = i < cap ? entry(b, i, k, v) : 0;
                const int tiles = (n + 31) >> 5, t = wave_inclusive_sum(tiles);
                if (i < cap) {
                    tab.off_k[i] = k;
                    tab.off_v[i] = v;
                    tab.len[i] = n;
                    tab.cum[i] = t0 + t - tiles;
                }
                t0 += __builtin_amdgcn_readlane(t, 63);
            }
            if (lane == 0) tab.cum[cap] = t0;
        }
        lds_barrier();
    }
    bool listed;
};

// Largest slot with cum[slot] <= u, for 0 <= u < cum[n]: by all lanes of the wave at once.
__device__ __forceinline__ int find_slot_wave(const int* cum, int n, int u) {
    const int lane = threadIdx.x & 63;
    int c = 0;
    for (int i = lane; i - lane < n; i += 64) c += __popcll(__ballot(i < n && cum[min(i, n - 1)] <= u));
    return c - 1;
}
// The cut of the batch's key tiles into ranges (tile_ranges.hpp), in LDS: range r is the tiles bound[r] .. bound[r + 1] - 1 of
// the batch's list.  Which sequence a range begins in and which ranges a sequence meets is found by all lanes at once when a
// pass needs it (sequences in lanes, find_slot_wave), not looked up in further tables: filling those behind one more barrier,
// by two searches of a thread per sequence, was half of the 2 microseconds that the cut took of a question's start.
struct TileRanges {
    int bound[kMaxRanges + 1];
};
// lds: dynamic LDS of the launch that plans itself; grid: its workgroups.
inline bool prefill_plans_inline(int B, int R_max, size_t lds, long long grid, int num_cu) {
    const size_t all = align_up(lds + sizeof(TileRanges) + (kInlineBatch + 4) * sizeof(int), kLdsGranule);
    return B <= kInlineBatch && (long long)B * R_max <= kInlineRounds && (grid + num_cu - 1) / num_cu * all <= kLdsPerUnit;
}
// Lane b: the tiles of sequence b and the first of them.
struct LaneSequence {
    int U, tile0;
};
__device__ __forceinline__ LaneSequence lane_sequence(const int* sU, int B) {
    const int lane = threadIdx.x & 63, U = lane < B ? sU[lane] : 0;
    return {U, wave_inclusive_sum(U) - U};
}
// Fills `tr` from the sequences' tiles sU; returns the number of ranges.  All threads call it; no barrier behind the counts
// needed before it, one at its end.
template <int C>
__device__ __forceinline__ int cut_tiles(TileRanges& tr, const int* sU, int B, int slots, int min_tiles, int max_parts, bool full,
                                         const RangeWeights<C>& weights) {
    const int tid = threadIdx.x;
    const LaneSequence sq = lane_sequence(sU, B);
    const int total = __builtin_amdgcn_readlane(sq.tile0 + sq.U, 63);
    float top = (float)sq.U;  // (exact: a sequence has fewer than 2^24 tiles)
    top = vmax(top, dpp_mov<0xB1>(top));
    top = vmax(top, dpp_mov<0x4E>(top));
    top = vmax(top, dpp_mov<0x141>(top));
    top = xrow_max4(vmax(top, dpp_mov<0x140>(top)));
    const int most = __builtin_amdgcn_readfirstlane((int)top);
    if (slots > kMaxRanges) slots = kMaxRanges;
    const TileCut<C> cut(total, most, slots, min_tiles, max_parts, full, weights);
    int P = cut.n_ranges;
    for (int len = cut.len; len <= cut.longest_apart(B); ++len) {
        const int cuts = cut.cuts(sq.U, len), cuts_incl = wave_inclusive_sum(cuts);
        const int P_apart = __builtin_amdgcn_readlane(cuts_incl, 63);
        if (!cut.apart(P_apart, slots)) continue;
        for (int b = tid >> 6; b < B; b += 4) {  // a wave per sequence (a thread's loop over 96 ranges took 6 microseconds)
            const int n = __builtin_amdgcn_readlane(cuts, b), first = __builtin_amdgcn_readlane(cuts_incl, b) - n;
            const int U = __builtin_amdgcn_readlane(sq.U, b), t0 = __builtin_amdgcn_readlane(sq.tile0, b);
            for (int j = tid & 63; j < n; j += 64) tr.bound[first + j] = t0 + piece_begin(U, j, n);
        }
        if (tid == 0) tr.bound[P_apart] = total;
        lds_barrier();
        return P_apart;
    }
    const double per_weight = cut.tiles_per_weight();
    for (int r = tid; r <= P; r += blockDim.x) tr.bound[r] = cut.begin(r, per_weight);
    lds_barrier();
    return P;
}
// The sequence that tile t lies in: the last one that begins at or before it.
__device__ __forceinline__ int sequence_of_tile(const LaneSequence& sq, int B, int t) {
    return __popcll(__ballot((int)(threadIdx.x & 63) < B && sq.tile0 <= t)) - 1;
}
// Ranges that sequence b meets: the first of them and their number (uniform).
__device__ __forceinline__ int parts_of(const TileRanges& tr, int P, const LaneSequence& sq, int b, int& first) {
    const int U = __builtin_amdgcn_readlane(sq.U, b), t0 = __builtin_amdgcn_readlane(sq.tile0, b);
    first = 0;
    if (U <= 0) return 0;
    first = find_slot_wave(tr.bound, P, t0);
    return find_slot_wave(tr.bound, P, t0 + U - 1) - first + 1;
}
// The first of them, for a sequence with tiles.
__device__ __forceinline__ int first_part_of(const TileRanges& tr, int P, const LaneSequence& sq, int b) {
    return find_slot_wave(tr.bound, P, __builtin_amdgcn_readlane(sq.tile0, b));
}
// The range that the position-th group of workgroups takes: class 0's ranges first, then class 1's, ...
template <int C>
__device__ __forceinline__ int range_at(int position, int P) {
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int n = (P - k + C - 1) / C;
        if (position < n) return position * C + k;
        position -= n;
    }
    return P - 1;
}

}  // namespace ra
