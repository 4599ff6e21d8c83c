// Round-indexed KV store for the post-watershed layers (paper Sec. 3.2 and Fig. 1: the "upper half"
// u_m of every round stays in host memory as one tensor; the tensors of the selected rounds are
// moved to the GPU once the selection is known, each in one transfer or in one per group of layers).
//
// Mostly host side: a registry of pinned per-round tensors, a bump-allocated device pool, the index
// tables of the compact per-layer views, and the choreography of copies and events on a side
// stream.  The copied bytes keep the host layout: per layer the keys [Hkv][len][d] followed by the
// values in transposed 16-token tiles [Hkv][ceil(len/16)][d][16].  Every slice is therefore already a
// round block in the device layout and staging needs no repacking kernel.
//
// Large slices are moved by asynchronous copies, small ones by a kernel that reads the pinned host memory itself
// (stage_kernel).  The kernel at the end of a turn (Sec. 3.2, last step; Alg. 1, last line) gathers
// the new round's token-major keys and values of every post-watershed layer into that round layout
// behind the staged rounds in the pool, from where each sequence's new round leaves for host memory
// as a whole.  The registry also counts how often each round was staged, which is what KV-cache
// dropping (Sec. 3.4) decides on.
#include "common.hpp"

#include <algorithm>
#include <memory>
#include <new>
#include <vector>

namespace ra {
constexpr int kStageGroups = 5;  // most groups of layers of different size (grouped order)
// A round on its way between host memory and the pool.
struct StageJob {
    const char* src;      // its first layer
    char* dst;
    int64_t layer_bytes;  // of one layer, a multiple of 16
};
// Byte offsets of the tables in their block.
struct StoreTables {
    size_t off = 0, len = 0, n = 0, jobs = 0, units = 0, bytes = 0;
    void layout(const ra_store_cfg& c) {
        const size_t plane = (size_t)c.B * c.R_max;
        len = align_up(off + (size_t)c.n_layers * 2 * plane * sizeof(int64_t), 16);
        n = align_up(len + plane * sizeof(int32_t), 16);
        jobs = align_up(n + (size_t)c.B * sizeof(int32_t), 16);
        units = align_up(jobs + plane * sizeof(StageJob), 16);  // [kStageGroups][B * R_max + 1] prefix of the jobs' units
        bytes = align_up(units + kStageGroups * (plane + 1) * sizeof(int32_t), 16);
    }
};
// ... of the turn-end write-back.
struct SaveTables {
    size_t off = 0, len = 0, cur = 0, jobs = 0, units = 0, bytes = 0;
    void layout(const ra_store_cfg& c) {
        len = align_up(off + (size_t)c.B * sizeof(int64_t), 16);        // off [B]: start of the round's tensor in the pool, in tokens; -1 = skip
        cur = align_up(len + (size_t)c.B * sizeof(int32_t), 16);        // len [B]
        jobs = align_up(cur + (size_t)c.n_layers * 2 * sizeof(void*), 16);  // cur [2][n_layers]: keys and values of the current round
        units = align_up(jobs + (size_t)c.B * sizeof(StageJob), 16);
        bytes = align_up(units + ((size_t)c.B + 1) * sizeof(int32_t), 16);
    }
};
}  // namespace ra

struct ra_kv_store {
    using StoreTables = ra::StoreTables;
    using SaveTables = ra::SaveTables;
    ra_store_cfg cfg;
    size_t token_bytes = 0;  // bytes of one token of one layer of K (or V): Hkv * d * elem
    struct Round {
        const char* host = nullptr;
        bool direct = false;  // kernels may read the host tensor
        int len = -1;  // -1 = never registered
        uint32_t turns = 0, hits = 0;  // stage calls since registration / of those, the ones that selected it
        bool dropped = false;
    };
    std::vector<Round> rounds;  // [B][R_max]
    char* pool = nullptr;
    // index tables of the views and the staging kernel's: one block, host pinned mirror and device copy
    char *h_tab = nullptr, *d_tab = nullptr;
    StoreTables tab;
    int64_t* h_off = nullptr;  // [n_layers][2][B][R_max]
    int32_t* h_len = nullptr;  // [B][R_max]
    int32_t* h_n = nullptr;    // [B]
    int64_t* d_off = nullptr;
    int32_t* d_len = nullptr;
    int32_t* d_n = nullptr;
    std::vector<hipEvent_t> ready;
    bool staged = false;
    int64_t max_tokens = 0;
    size_t staged_tok = 0;  // pool cursor behind the staged rounds, in units of token_bytes
    // turn-end write-back of the new round: its tables (pinned mirror + device copy) and events
    char *h_wb = nullptr, *d_wb = nullptr;
    SaveTables wb;
    hipEvent_t wb_packed = nullptr, wb_done = nullptr;
    bool wb_pending = false;
    uint64_t saved_bytes = 0;
    uint64_t staged_bytes = 0, n_copies = 0;
};

using namespace ra;

// Tokens' worth of storage of one layer of one round: len rows of keys plus the values padded to
// whole 16-token tiles.
static inline size_t layer_tokens(int len) { return (size_t)len + (size_t)((len + 15) / 16) * 16; }

// Layers in group gi of the grouped staging order for L layers: first max(1, L / 8); last 1; the layers in
// between in three groups as equal as possible (fewer when there are fewer layers).
static int grouped_stage_size(int L, int gi) {
    const int first = L / 8 > 1 ? L / 8 : 1;
    if (gi == 0) return first < L ? first : L;
    const int middle = L - first - 1;                 // layers between the first group and the last layer
    const int n_mid = middle < 3 ? (middle > 0 ? middle : 0) : 3;
    if (gi <= n_mid) return middle / n_mid + (gi <= middle % n_mid ? 1 : 0);
    return 1;
}

// Whether an allocation of these flags is coherent for the kernels whatever HIP_HOST_COHERENT says, which decides for the ones
// that have other flags alone (hipHostMallocPortable).
static bool is_coherent(unsigned flags) {
    if (flags & (hipHostMallocNonCoherent | hipHostMallocUncached | hipHostMallocWriteCombined)) return false;
    return flags == hipHostMallocDefault || flags & (hipHostMallocCoherent | hipHostMallocMapped);
}
// Pinned memory.  `direct`: whether kernels may read and write `bytes` bytes of it: coherent, at the same address, and all in one
// allocation (of a tensor that is shorter than its round a copy reports an error, a kernel faults).
static bool is_pinned_host(const void* p, size_t bytes, bool* direct) {
    hipPointerAttribute_t attr;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    *direct = false;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();  // ordinary pageable memory: not an error of ours, clear the sticky code
        return false;
    }
    if (attr.type != hipMemoryTypeHost) return false;
    if (hipMemGetAddressRange(&base, &size, const_cast<void*>(p)) == hipSuccess) {
        const size_t at = (size_t)(static_cast<const char*>(p) - static_cast<const char*>(base));
        *direct = attr.devicePointer == p && is_coherent(attr.allocationFlags) && at <= size && bytes <= size - at;
    } else {
        (void)hipGetLastError();
    }
    return true;
}

namespace {
// ---- between host memory and the pool -----------------------------------------------------------------
// Slices of kStageCopyBytes (kSaveCopyBytes) and more are asynchronous copies: the copy engines leave the compute units to the
// work beside them.  Each costs 10 microseconds of its own on the stream, whatever its size (49 GB/s in copies of 4 MB, 44 of 2,
// 37 of 1, 18 of 256 KB; the link: 57).
// Smaller slices, of which a turn of short rounds has hundreds, are one launch of a kernel that reads (at a turn's end: writes)
// the pinned host memory itself, in units of 16 KB (a workgroup's four 16-byte loads a thread) that a small grid takes in turn:
// 57 GB/s with half a megabyte asked for.  While it runs the work beside it is slow: memory-bound products at 40 % of their rate,
// and beside the write-back at next to nothing, where a copy saves as much as it costs from 0.6 MB on.  While rounds are staged
// there is often nothing to compute yet, so the line lies higher there.  Microseconds with everything by copies, everything by
// the kernel, and staged so with copies from 2, 4 and 8 MB on (a copy of a layer of 425 tokens and 8 KV heads: 1.8 MB):
//   turn of 8 rounds of 425 tokens, 24 layers                   7 209   6 880   7 088   7 022   6 988
//   ... with 3.6 ms of memory-bound products behind the layers  8 068  10 280   8 057   8 171   8 452
//   turn of 16 such rounds, 6 layers                            4 590   3 800   4 231   3 891   3 822
//   ... with 5.8 ms of memory-bound products behind the layers  6 912   8 300   7 338   7 886   8 326
//   turn of one dialogue, 4 rounds of 350 tokens, 3 layers        639     514     520     521     525
//   turn of 5 x 7 rounds of 50 tokens, 5 layers                 2 750     943   1 000     987   1 003
//   save of 4 x 500 tokens, 6 layers, 2.6 ms of products of 4096^3 behind it: 2 721 and 3 526
// (Copies dealt out to two streams reach 55 GB/s in 2 MB, but 25 from a release of device memory on until the runtime next
// changes its mind, single ones 56 all the while.)
constexpr size_t kStageCopyBytes = 4 << 20, kSaveCopyBytes = 1 << 20;
constexpr int kStageThreads = 256, kStageLoads = 4, kStageGrid = 32, kSaveGrid = 64;
constexpr int kUnitBytes = kStageThreads * kStageLoads * 16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 global_u32x4;  // (a pointer out of a table would be a flat one)

// unit0[j]: first unit of job j, unit0[n_jobs] = n_units; a job without units is left out.  Layers [l0, l0 + n_l) of every job.
// TO_HOST: the destination is host memory.
template <bool TO_HOST>
__global__ __launch_bounds__(kStageThreads) void stage_kernel(const StageJob* jobs, const int32_t* unit0, int n_jobs, int n_units, int l0,
                                                             int n_l) {
    const int lane = threadIdx.x & 63;
    int j = 0;  // unit0[j] <= u
    for (int u = blockIdx.x; u < n_units; u += gridDim.x) {
        while (true) {
            const int at_or_before = __popcll(__ballot(j + lane < n_jobs && unit0[min(j + lane, n_jobs)] <= u));
            j += at_or_before - 1;
            if (at_or_before < 64) break;
        }
        const StageJob jb = jobs[j];
        const int64_t first = (int64_t)l0 * jb.layer_bytes, end = first + (int64_t)n_l * jb.layer_bytes;
        const int64_t at = first + (int64_t)(u - unit0[j]) * kUnitBytes + threadIdx.x * 16;
        u32x4 v[kStageLoads];
#pragma unroll
        for (int i = 0; i < kStageLoads; ++i) {
            const int64_t o = at + i * (kStageThreads * 16);
            if (o < end) v[i] = __builtin_nontemporal_load((const global_u32x4*)(jb.src + o));
        }
#pragma unroll
        for (int i = 0; i < kStageLoads; ++i) {
            const int64_t o = at + i * (kStageThreads * 16);
            if (o >= end) continue;
            if (TO_HOST) __builtin_nontemporal_store(v[i], (global_u32x4*)(jb.dst + o));
            else *(global_u32x4*)(jb.dst + o) = v[i];
        }
    }
}

// The tables, 16-byte pieces.
__global__ __launch_bounds__(kStageThreads) void copy_tables_kernel(const u32x4* src, u32x4* dst, int n) {
    for (int i = blockIdx.x * kStageThreads + threadIdx.x; i < n; i += gridDim.x * kStageThreads) dst[i] = src[i];
}

static int copy_tables(const char* host, char* device, size_t bytes, hipStream_t st) {
    const int n = (int)(bytes / 16), grid = (n + kStageThreads - 1) / kStageThreads;
    hipLaunchKernelGGL(copy_tables_kernel, dim3(grid < kStageGrid ? grid : kStageGrid), dim3(kStageThreads), 0, st,
                       reinterpret_cast<const u32x4*>(host), reinterpret_cast<u32x4*>(device), n);
    RA_HIP_CHECK(hipGetLastError());
    return RA_OK;
}
// Everything goes to the store's device, where its events are: a stream of another one is refused before anything is enqueued.
// (The handles that name a default stream mean the current device's; hipStreamGetDevice takes only the first of them.)
static int check_stream(const ra_kv_store* s, hipStream_t st, const char* who) {
    int device = -1;
    if (st == nullptr || st == hipStreamLegacy || st == hipStreamPerThread) RA_HIP_CHECK(hipGetDevice(&device));
    else RA_HIP_CHECK(hipStreamGetDevice(st, &device));
    RA_REQUIRE(device == s->cfg.device, RA_ERR_HIP, "%s: a stream of device %d, the store is on device %d", who, device, s->cfg.device);
    return RA_OK;
}
// The store's device while it enqueues.
struct OnDevice {
    int prev = -1;
    explicit OnDevice(int device) {
        if (hipGetDevice(&prev) != hipSuccess || prev == device || hipSetDevice(device) != hipSuccess) prev = -1;
    }
    ~OnDevice() {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

// Tensors on their way, all in one direction: the kernel's jobs (in the pinned mirror of a table) and which of them it can reach.
struct Moves {
    StageJob* jobs;
    std::vector<bool> direct;
    hipMemcpyKind kind;
    void add(const char* src, char* dst, size_t layer_bytes, bool reachable) {
        jobs[direct.size()] = {src, dst, (int64_t)layer_bytes};
        direct.push_back(reachable && ((uintptr_t)src | (uintptr_t)dst | layer_bytes) % 16 == 0);
    }
    int size() const { return (int)direct.size(); }
    // Prefix of the units of n_l layers of every job, none for the jobs that are copied.
    void units(int n_l, int32_t* row) const {
        const size_t copied = kind == hipMemcpyDeviceToHost ? kSaveCopyBytes : kStageCopyBytes;
        int64_t n = 0;
        for (int k = 0; k < size(); ++k) {
            const int64_t bytes = n_l * jobs[k].layer_bytes, more = (bytes + kUnitBytes - 1) / kUnitBytes;
            row[k] = (int32_t)n;
            if (direct[k] && (size_t)bytes < copied && n + more <= INT32_MAX / 2) n += more;
        }
        row[size()] = (int32_t)n;
    }
    // Enqueues layers [l0, l0 + n_l) of every tensor on `st`.  row, and its device copy: the units.
    int enqueue(const char* d_jobs, const int32_t* row, const char* d_row, int l0, int n_l, hipStream_t st) const {
        if (const int n_units = row[size()]; n_units > 0) {
            const bool to_host = kind == hipMemcpyDeviceToHost;
            const int most = to_host ? kSaveGrid : kStageGrid;
            const auto kernel = to_host ? stage_kernel<true> : stage_kernel<false>;
            hipLaunchKernelGGL(kernel, dim3(n_units < most ? n_units : most), dim3(kStageThreads), 0, st, reinterpret_cast<const StageJob*>(d_jobs),
                               reinterpret_cast<const int32_t*>(d_row), size(), n_units, l0, n_l);
            RA_HIP_CHECK(hipGetLastError());
        }
        for (int k = 0; k < size(); ++k) {
            const size_t o = (size_t)l0 * jobs[k].layer_bytes, bytes = (size_t)n_l * jobs[k].layer_bytes;
            if (row[k + 1] == row[k]) RA_HIP_CHECK(hipMemcpyAsync(jobs[k].dst + o, jobs[k].src + o, bytes, kind, st));
        }
        return RA_OK;
    }
};

constexpr int kRepackThreads = 256;

template <typename T>
union Vec16 {
    uint4 u;
    T e[16 / sizeof(T)];
};

// Turn-end gather of the new round (Sec. 3.2, last step), the layers from layer0 on in one launch.  A workgroup moves one
// 16-token tile of one layer and kv head of one sequence: the key rows go out unchanged to row t of head g,
// the value rows are turned through LDS into the [d][16] tile of the round layout, rows past the
// round's length as zeros.  Pure data movement in 16-byte pieces; T only fixes the element width.
template <typename T>
__global__ __launch_bounds__(kRepackThreads) void repack_round_kernel(const T* const* __restrict__ cur, int n_layers, int layer0, int n_tiles,
                                                                      int cur_cap, int Hkv, int d,
                                                                      const int64_t* __restrict__ wb_off,
                                                                      const int32_t* __restrict__ wb_len,
                                                                      T* __restrict__ pool) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int V = 16 / sizeof(T);  // elements per 16-byte piece; also the row padding in LDS
    T* tile = reinterpret_cast<T*>(smem);  // [16][d + V]
    const int local = blockIdx.x / n_tiles, tile16 = blockIdx.x - local * n_tiles, layer = layer0 + local;
    const int b = blockIdx.z, g = blockIdx.y, t0 = tile16 * 16;
    const int64_t off = wb_off[b];
    const int n = wb_len[b];
    if (off < 0 || t0 >= n) return;
    const T *cur_k = cur[layer], *cur_v = cur[n_layers + layer];
    const int tiles = (n + 15) / 16;
    const size_t layer_tok = (size_t)off + (size_t)layer * ((size_t)n + (size_t)tiles * 16);
    T* kdst = pool + (layer_tok * Hkv + (size_t)g * n) * d;
    T* vdst = pool + (layer_tok + n) * Hkv * d + ((size_t)g * tiles + tile16) * d * 16;
    const int pieces = d / V, pitch = d + V;
    for (int i = threadIdx.x; i < 16 * pieces; i += kRepackThreads) {
        const int j = i / pieces, c = (i % pieces) * V, t = t0 + j;
        uint4 vv = make_uint4(0, 0, 0, 0);
        if (t < n) {
            const size_t src = (((size_t)b * cur_cap + t) * Hkv + g) * d + c;
            *reinterpret_cast<uint4*>(kdst + (size_t)t * d + c) = *reinterpret_cast<const uint4*>(cur_k + src);
            vv = *reinterpret_cast<const uint4*>(cur_v + src);
        }
        *reinterpret_cast<uint4*>(tile + j * pitch + c) = vv;
    }
    __syncthreads();
    constexpr int per_channel = 16 / V;  // 16-byte pieces of one channel's 16 tokens
    for (int i = threadIdx.x; i < d * per_channel; i += kRepackThreads) {
        const int c = i / per_channel, j0 = (i % per_channel) * V;
        Vec16<T> x;
#pragma unroll
        for (int e = 0; e < V; ++e) x.e[e] = tile[(j0 + e) * pitch + c];
        *reinterpret_cast<uint4*>(vdst + c * 16 + j0) = x.u;
    }
}
}  // namespace

extern "C" {

int ra_kv_store_create(ra_kv_store** out, const ra_store_cfg* cfg) {
    RA_REQUIRE(out != nullptr && cfg != nullptr, RA_ERR_INVALID_ARG, "kv_store_create: NULL argument");
    *out = nullptr;
    RA_REQUIRE(cfg->n_layers > 0 && cfg->B > 0 && cfg->R_max > 0 && cfg->Hkv > 0 && cfg->d > 0, RA_ERR_INVALID_ARG,
               "kv_store_create: non-positive dimension");
    RA_REQUIRE(cfg->R_max <= kMaxRounds, RA_ERR_UNSUPPORTED, "kv_store_create: R_max %d exceeds %d", cfg->R_max,
               kMaxRounds);
    RA_REQUIRE(cfg->dtype == RA_F32 || cfg->dtype == RA_BF16, RA_ERR_UNSUPPORTED, "kv_store_create: unknown dtype");
    RA_REQUIRE(cfg->device_pool_bytes > 0, RA_ERR_INVALID_ARG, "kv_store_create: device_pool_bytes is 0");
    int ndev = 0, prev = 0;
    RA_HIP_CHECK(hipGetDeviceCount(&ndev));
    RA_REQUIRE(cfg->device >= 0 && cfg->device < ndev, RA_ERR_INVALID_ARG, "kv_store_create: device out of range");
    RA_HIP_CHECK(hipGetDevice(&prev));
    RA_HIP_CHECK(hipSetDevice(cfg->device));

    ra_kv_store* s = new (std::nothrow) ra_kv_store();
    RA_REQUIRE(s != nullptr, RA_ERR_OOM, "kv_store_create: out of host memory");
    s->cfg = *cfg;
    s->token_bytes = (size_t)cfg->Hkv * cfg->d * (cfg->dtype == RA_BF16 ? 2 : 4);
    s->rounds.resize((size_t)cfg->B * cfg->R_max);
    s->tab.layout(*cfg);
    hipError_t e = hipMalloc((void**)&s->pool, cfg->device_pool_bytes);
    if (e == hipSuccess) e = hipMalloc((void**)&s->d_tab, s->tab.bytes);
    if (e == hipSuccess) e = hipHostMalloc((void**)&s->h_tab, s->tab.bytes, hipHostMallocDefault);
    s->h_off = reinterpret_cast<int64_t*>(s->h_tab + s->tab.off);
    s->h_len = reinterpret_cast<int32_t*>(s->h_tab + s->tab.len);
    s->h_n = reinterpret_cast<int32_t*>(s->h_tab + s->tab.n);
    s->d_off = reinterpret_cast<int64_t*>(s->d_tab + s->tab.off);
    s->d_len = reinterpret_cast<int32_t*>(s->d_tab + s->tab.len);
    s->d_n = reinterpret_cast<int32_t*>(s->d_tab + s->tab.n);
    s->wb.layout(*cfg);
    if (e == hipSuccess) e = hipMalloc((void**)&s->d_wb, s->wb.bytes);
    if (e == hipSuccess) e = hipHostMalloc((void**)&s->h_wb, s->wb.bytes, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->wb_packed, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->wb_done, hipEventDisableTiming);
    if (e == hipSuccess) {
        s->ready.resize(cfg->n_layers, nullptr);
        for (int l = 0; l < cfg->n_layers && e == hipSuccess; ++l)
            e = hipEventCreateWithFlags(&s->ready[l], hipEventDisableTiming);
    }
    (void)hipSetDevice(prev);
    if (e != hipSuccess) {
        const bool oom = e == hipErrorOutOfMemory;
        (void)hipGetLastError();
        ra_kv_store_destroy(s);
        return fail(oom ? RA_ERR_OOM : RA_ERR_HIP, "kv_store_create: %s", hipGetErrorString(e));
    }
    *out = s;
    return RA_OK;
}

int ra_kv_store_destroy(ra_kv_store* s) {
    if (!s) return RA_OK;
    for (hipEvent_t ev : s->ready)
        if (ev) (void)hipEventDestroy(ev);
    if (s->pool) (void)hipFree(s->pool);
    if (s->d_tab) (void)hipFree(s->d_tab);
    if (s->h_tab) (void)hipHostFree(s->h_tab);
    if (s->wb_pending) (void)hipEventSynchronize(s->wb_done);  // host tensors may be freed right after this call
    if (s->d_wb) (void)hipFree(s->d_wb);
    if (s->h_wb) (void)hipHostFree(s->h_wb);
    if (s->wb_packed) (void)hipEventDestroy(s->wb_packed);
    if (s->wb_done) (void)hipEventDestroy(s->wb_done);
    delete s;
    return RA_OK;
}

size_t ra_kv_store_round_bytes(const ra_kv_store* s, int len) {
    if (!s || len < 0) return 0;
    return (size_t)s->cfg.n_layers * layer_tokens(len) * s->token_bytes;
}

int ra_kv_store_register_round(ra_kv_store* s, int seq, int round, const void* host_kv, int len) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_register_round: store is NULL");
    RA_REQUIRE(seq >= 0 && seq < s->cfg.B && round >= 0 && round < s->cfg.R_max, RA_ERR_INVALID_ARG,
               "kv_store_register_round: (seq %d, round %d) outside [0,%d) x [0,%d)", seq, round, s->cfg.B,
               s->cfg.R_max);
    RA_REQUIRE(len >= 0, RA_ERR_INVALID_ARG, "kv_store_register_round: negative length");
    RA_REQUIRE(len == 0 || host_kv != nullptr, RA_ERR_INVALID_ARG, "kv_store_register_round: host_kv is NULL");
    RA_REQUIRE(!s->staged, RA_ERR_STATE, "kv_store_register_round: rounds are staged; call ra_kv_store_release first");
    bool direct = false;
    if (len > 0)
        RA_REQUIRE(is_pinned_host(host_kv, ra_kv_store_round_bytes(s, len), &direct), RA_ERR_INVALID_ARG,
                   "kv_store_register_round: host_kv is not pinned host memory (use hipHostMalloc / pin_memory)");
    ra_kv_store::Round& r = s->rounds[(size_t)seq * s->cfg.R_max + round];
    r.host = static_cast<const char*>(host_kv);
    r.direct = direct;
    r.len = len;
    r.turns = r.hits = 0;
    r.dropped = false;
    return RA_OK;
}

int ra_kv_store_stage(ra_kv_store* s, const int32_t* sel_idx_host, const int32_t* n_sel_host, int order,
                      void* side_stream) {
    RA_REQUIRE(s != nullptr && sel_idx_host != nullptr && n_sel_host != nullptr, RA_ERR_INVALID_ARG,
               "kv_store_stage: NULL argument");
    RA_REQUIRE(order == RA_STAGE_ROUND_MAJOR || order == RA_STAGE_LAYER_MAJOR || order == RA_STAGE_GROUPED,
               RA_ERR_INVALID_ARG, "kv_store_stage: unknown order %d", order);
    RA_REQUIRE(!s->staged, RA_ERR_STATE, "kv_store_stage: already staged; call ra_kv_store_release first");
    const int B = s->cfg.B, R = s->cfg.R_max, L = s->cfg.n_layers;
    // ---- validate the selection and place every selected round in the pool ----------------------
    struct Job { const char* src; size_t dst_tok; int len; bool direct; };
    std::vector<Job> jobs;
    size_t tok = 0;  // pool cursor in units of token_bytes
    int64_t max_tokens = 0;
    for (int b = 0; b < B; ++b) {
        const int n = n_sel_host[b];
        RA_REQUIRE(n >= 0 && n <= R, RA_ERR_INVALID_ARG, "kv_store_stage: n_sel[%d] = %d outside [0, %d]", b, n, R);
        int64_t seq_tokens = 0;
        int prev = -1;
        for (int i = 0; i < n; ++i) {
            const int r = sel_idx_host[(size_t)b * R + i];
            RA_REQUIRE(r > prev && r < R, RA_ERR_INVALID_ARG,
                       "kv_store_stage: sel_idx[%d][%d] = %d is not an ascending round index below %d", b, i, r, R);
            prev = r;
            const ra_kv_store::Round& rd = s->rounds[(size_t)b * R + r];
            RA_REQUIRE(rd.len >= 0, RA_ERR_STATE, "kv_store_stage: round %d of sequence %d was never registered", r, b);
            jobs.push_back({rd.host, tok, rd.len, rd.direct});
            tok += (size_t)L * layer_tokens(rd.len);
            seq_tokens += rd.len;
        }
        if (seq_tokens > max_tokens) max_tokens = seq_tokens;
    }
    RA_REQUIRE(tok * s->token_bytes <= s->cfg.device_pool_bytes, RA_ERR_OOM,
               "kv_store_stage: selected rounds need %zu bytes, the device pool has %zu", tok * s->token_bytes,
               s->cfg.device_pool_bytes);
    hipStream_t st = reinterpret_cast<hipStream_t>(side_stream);
    if (int rc = check_stream(s, st, "kv_store_stage")) return rc;
    // ---- index tables of the compact views (round i of the view = i-th selected round) ----------
    const size_t plane = (size_t)B * R;
    for (size_t i = 0; i < (size_t)L * 2 * plane; ++i) s->h_off[i] = 0;
    for (size_t i = 0; i < plane; ++i) s->h_len[i] = 0;
    size_t j = 0;
    for (int b = 0; b < B; ++b) {
        s->h_n[b] = n_sel_host[b];
        for (int i = 0; i < n_sel_host[b]; ++i, ++j) {
            const Job& jb = jobs[j];
            s->h_len[(size_t)b * R + i] = jb.len;
            for (int l = 0; l < L; ++l) {
                s->h_off[((size_t)l * 2 + 0) * plane + (size_t)b * R + i] = (int64_t)(jb.dst_tok + (size_t)l * layer_tokens(jb.len));
                s->h_off[((size_t)l * 2 + 1) * plane + (size_t)b * R + i] =
                    (int64_t)(jb.dst_tok + (size_t)l * layer_tokens(jb.len) + jb.len);
            }
        }
    }
    // ---- activity counters (Sec. 3.4): every kept round was a candidate, the selected ones were hit --
    for (int b = 0; b < B; ++b) {
        for (int r = 0; r < R; ++r) {
            ra_kv_store::Round& rd = s->rounds[(size_t)b * R + r];
            if (rd.len >= 0 && !rd.dropped) ++rd.turns;
        }
        for (int i = 0; i < n_sel_host[b]; ++i) {
            ra_kv_store::Round& rd = s->rounds[(size_t)b * R + sel_idx_host[(size_t)b * R + i]];
            if (!rd.dropped) ++rd.hits;
        }
    }
    // ---- enqueue the copies ------------------------------------------------------------------------
    OnDevice on(s->cfg.device);
    // a round saved at the end of the last turn may be selected now, and its packed copy may still
    // sit where this selection is about to land: both wait for the write-back
    if (s->wb_pending) RA_HIP_CHECK(hipStreamWaitEvent(st, s->wb_done, 0));
    // Groups of consecutive layers [l0, l1) in the order they are copied, every round's layers of a group as one slice: a
    // round's layers are contiguous in its host tensor.  Grouped: a small first group lets the first post-watershed layer
    // start early, a last group of one layer leaves a single layer's attention to run after the last byte has arrived.
    std::vector<int> bounds{0};
    for (int gi = 0; bounds.back() < L; ++gi)
        bounds.push_back(order == RA_STAGE_ROUND_MAJOR ? L
                                                       : bounds.back() + (order == RA_STAGE_LAYER_MAJOR ? 1 : grouped_stage_size(L, gi)));
    const int n_groups = (int)bounds.size() - 1;
    Moves moves{reinterpret_cast<StageJob*>(s->h_tab + s->tab.jobs), {}, hipMemcpyHostToDevice};
    for (const Job& jb : jobs)
        if (jb.len > 0) moves.add(jb.src, s->pool + jb.dst_tok * s->token_bytes, layer_tokens(jb.len) * s->token_bytes, jb.direct);
    s->staged_bytes = (uint64_t)tok * s->token_bytes;
    s->n_copies = (uint64_t)n_groups * moves.size();
    // (the layer-major order's groups are all of one size)
    auto row_off = [&](int g) { return s->tab.units + (order == RA_STAGE_LAYER_MAJOR ? 0 : g) * (plane + 1) * sizeof(int32_t); };
    auto row = [&](int g) { return reinterpret_cast<int32_t*>(s->h_tab + row_off(g)); };
    for (int g = 0; g < n_groups; ++g) moves.units(bounds[g + 1] - bounds[g], row(g));
    if (int rc = copy_tables(s->h_tab, s->d_tab, s->tab.bytes, st)) return rc;
    for (int g = 0; g < n_groups; ++g) {
        const int l0 = bounds[g], n_l = bounds[g + 1] - l0;
        if (int rc = moves.enqueue(s->d_tab + s->tab.jobs, row(g), s->d_tab + row_off(g), l0, n_l, st)) return rc;
        for (int l = l0; l < l0 + n_l; ++l) RA_HIP_CHECK(hipEventRecord(s->ready[l], st));
    }
    s->max_tokens = max_tokens;
    s->staged_tok = tok;
    s->staged = true;
    return RA_OK;
}

int ra_kv_store_wait_layer(ra_kv_store* s, int layer, void* compute_stream) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_wait_layer: store is NULL");
    RA_REQUIRE(layer >= 0 && layer < s->cfg.n_layers, RA_ERR_INVALID_ARG, "kv_store_wait_layer: layer out of range");
    RA_REQUIRE(s->staged, RA_ERR_STATE, "kv_store_wait_layer: nothing is staged");
    RA_HIP_CHECK(hipStreamWaitEvent(reinterpret_cast<hipStream_t>(compute_stream), s->ready[layer], 0));
    return RA_OK;
}

int ra_kv_store_layer_view(ra_kv_store* s, int layer, ra_kv_view* out) {
    RA_REQUIRE(s != nullptr && out != nullptr, RA_ERR_INVALID_ARG, "kv_store_layer_view: NULL argument");
    RA_REQUIRE(layer >= 0 && layer < s->cfg.n_layers, RA_ERR_INVALID_ARG, "kv_store_layer_view: layer out of range");
    RA_REQUIRE(s->staged, RA_ERR_STATE, "kv_store_layer_view: nothing is staged");
    const size_t plane = (size_t)s->cfg.B * s->cfg.R_max;
    out->k = s->pool;
    out->v = s->pool;
    out->seg_off = s->d_off + ((size_t)layer * 2 + 0) * plane;
    out->seg_off_v = s->d_off + ((size_t)layer * 2 + 1) * plane;
    out->seg_len = s->d_len;
    out->n_rounds = s->d_n;
    out->block_table = nullptr;
    out->block_size = 0;
    out->max_blocks = 0;
    out->B = s->cfg.B;
    out->R_max = s->cfg.R_max;
    out->Hkv = s->cfg.Hkv;
    out->d = s->cfg.d;
    out->dtype = s->cfg.dtype;
    out->reserved = 0;
    out->max_tokens = s->max_tokens;
    return RA_OK;
}

int ra_kv_store_stats(const ra_kv_store* s, uint64_t* staged_bytes, uint64_t* registered_bytes, uint64_t* n_copies) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_stats: store is NULL");
    if (staged_bytes) *staged_bytes = s->staged_bytes;
    if (n_copies) *n_copies = s->n_copies;
    if (registered_bytes) {
        uint64_t t = 0;
        for (const auto& r : s->rounds)
            if (r.len > 0) t += (uint64_t)s->cfg.n_layers * layer_tokens(r.len) * s->token_bytes;
        *registered_bytes = t;
    }
    return RA_OK;
}

int ra_kv_store_save_round(ra_kv_store* s, const int32_t* round_host, const int32_t* len_host,
                           const void* const* cur_k_layers, const void* const* cur_v_layers, int cur_cap,
                           void* const* host_kv, void* compute_stream, void* side_stream) {
    RA_REQUIRE(s != nullptr && round_host != nullptr && len_host != nullptr && cur_k_layers != nullptr &&
                   cur_v_layers != nullptr && host_kv != nullptr,
               RA_ERR_INVALID_ARG, "kv_store_save_round: NULL argument");
    RA_REQUIRE(cur_cap > 0, RA_ERR_INVALID_ARG, "kv_store_save_round: cur_cap must be positive");
    const int B = s->cfg.B, R = s->cfg.R_max, L = s->cfg.n_layers;
    const size_t elem = s->cfg.dtype == RA_BF16 ? 2 : 4;
    RA_REQUIRE(((size_t)s->cfg.d * elem) % 16 == 0, RA_ERR_UNSUPPORTED,
               "kv_store_save_round: a row of d = %d elements is not a whole number of 16-byte pieces", s->cfg.d);
    size_t tok = s->staged ? s->staged_tok : 0;
    int max_len = 0;
    std::vector<int64_t> off(B, -1);
    std::unique_ptr<bool[]> direct(new bool[B]());
    for (int b = 0; b < B; ++b) {
        const int r = round_host[b];
        if (r == -1) continue;
        const int n = len_host[b];
        RA_REQUIRE(r >= 0 && r < R, RA_ERR_INVALID_ARG, "kv_store_save_round: round[%d] = %d outside [0, %d)", b, r, R);
        RA_REQUIRE(n >= 0 && n <= cur_cap, RA_ERR_INVALID_ARG, "kv_store_save_round: len[%d] = %d outside [0, %d]", b,
                   n, cur_cap);
        if (n > 0)
            RA_REQUIRE(host_kv[b] != nullptr && is_pinned_host(host_kv[b], ra_kv_store_round_bytes(s, n), &direct[b]), RA_ERR_INVALID_ARG,
                       "kv_store_save_round: host_kv[%d] is not pinned host memory", b);
        off[b] = (int64_t)tok;
        tok += (size_t)L * layer_tokens(n);
        if (n > max_len) max_len = n;
    }
    RA_REQUIRE(tok * s->token_bytes <= s->cfg.device_pool_bytes, RA_ERR_OOM,
               "kv_store_save_round: staged rounds plus the new round need %zu bytes, the device pool has %zu",
               tok * s->token_bytes, s->cfg.device_pool_bytes);
    if (max_len > 0)
        for (int l = 0; l < L; ++l) {
            RA_REQUIRE(cur_k_layers[l] != nullptr && cur_v_layers[l] != nullptr, RA_ERR_INVALID_ARG,
                       "kv_store_save_round: layer %d has a NULL key or value pointer", l);
            RA_REQUIRE(((uintptr_t)cur_k_layers[l] | (uintptr_t)cur_v_layers[l]) % 16 == 0, RA_ERR_INVALID_ARG,
                       "kv_store_save_round: layer %d pointers are not 16-byte aligned", l);
        }
    hipStream_t cs = reinterpret_cast<hipStream_t>(compute_stream);
    hipStream_t ss = reinterpret_cast<hipStream_t>(side_stream);
    if (max_len > 0) {
        if (int rc = check_stream(s, cs, "kv_store_save_round")) return rc;
        if (int rc = check_stream(s, ss, "kv_store_save_round")) return rc;
    }
    // the placement table's pinned mirror and the pool area behind the staged rounds are reused from
    // call to call: the previous write-back must have left them
    if (s->wb_pending) {
        RA_HIP_CHECK(hipEventSynchronize(s->wb_done));
        s->wb_pending = false;
    }
    s->saved_bytes = 0;
    if (max_len > 0) {
        int64_t* h_off = reinterpret_cast<int64_t*>(s->h_wb + s->wb.off);
        int32_t* h_len = reinterpret_cast<int32_t*>(s->h_wb + s->wb.len);
        const void** h_cur = reinterpret_cast<const void**>(s->h_wb + s->wb.cur);
        int32_t* h_units = reinterpret_cast<int32_t*>(s->h_wb + s->wb.units);
        Moves moves{reinterpret_cast<StageJob*>(s->h_wb + s->wb.jobs), {}, hipMemcpyDeviceToHost};
        for (int b = 0; b < B; ++b) {
            h_off[b] = off[b];
            h_len[b] = off[b] < 0 ? 0 : len_host[b];
            if (h_len[b] == 0) continue;
            const size_t bytes = (size_t)L * layer_tokens(h_len[b]) * s->token_bytes;
            moves.add(s->pool + (size_t)off[b] * s->token_bytes, static_cast<char*>(host_kv[b]), bytes, direct[b]);
            s->saved_bytes += (uint64_t)bytes;
        }
        moves.units(1, h_units);
        for (int l = 0; l < L; ++l) {
            h_cur[l] = cur_k_layers[l];
            h_cur[L + l] = cur_v_layers[l];
        }
        OnDevice on(s->cfg.device);
        if (int rc = copy_tables(s->h_wb, s->d_wb, s->wb.bytes, cs)) return rc;
        const int n_tiles = (max_len + 15) / 16;
        const int64_t* d_off = reinterpret_cast<const int64_t*>(s->d_wb + s->wb.off);
        const int32_t* d_len = reinterpret_cast<const int32_t*>(s->d_wb + s->wb.len);
        const char* d_cur = s->d_wb + s->wb.cur;
        const int at_once = std::max(1, (int)(UINT32_MAX / kRepackThreads) / n_tiles);  // layers: a launch has fewer than 2^32 threads
        for (int l = 0; l < L; l += at_once) {
            const dim3 grid((unsigned)n_tiles * std::min(at_once, L - l), s->cfg.Hkv, B), block(kRepackThreads);
            if (elem == 2)
                hipLaunchKernelGGL(repack_round_kernel<uint16_t>, grid, block, 16 * (size_t)(s->cfg.d + 8) * 2, cs,
                                   reinterpret_cast<const uint16_t* const*>(d_cur), L, l, n_tiles, cur_cap, s->cfg.Hkv, s->cfg.d, d_off, d_len,
                                   reinterpret_cast<uint16_t*>(s->pool));
            else
                hipLaunchKernelGGL(repack_round_kernel<uint32_t>, grid, block, 16 * (size_t)(s->cfg.d + 4) * 4, cs,
                                   reinterpret_cast<const uint32_t* const*>(d_cur), L, l, n_tiles, cur_cap, s->cfg.Hkv, s->cfg.d, d_off, d_len,
                                   reinterpret_cast<uint32_t*>(s->pool));
            RA_HIP_CHECK(hipGetLastError());
        }
        RA_HIP_CHECK(hipEventRecord(s->wb_packed, cs));
        RA_HIP_CHECK(hipStreamWaitEvent(ss, s->wb_packed, 0));
        if (int rc = moves.enqueue(s->d_wb + s->wb.jobs, h_units, s->d_wb + s->wb.units, 0, 1, ss)) return rc;
        RA_HIP_CHECK(hipEventRecord(s->wb_done, ss));
        s->wb_pending = true;
    }
    for (int b = 0; b < B; ++b) {
        if (off[b] < 0) continue;
        ra_kv_store::Round& r = s->rounds[(size_t)b * R + round_host[b]];
        r.host = len_host[b] > 0 ? static_cast<const char*>(host_kv[b]) : nullptr;
        r.direct = direct[b];
        r.len = len_host[b];
        r.turns = r.hits = 0;
        r.dropped = false;
    }
    return RA_OK;
}

int ra_kv_store_save_wait(ra_kv_store* s, uint64_t* saved_bytes) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_save_wait: store is NULL");
    if (s->wb_pending) {
        RA_HIP_CHECK(hipEventSynchronize(s->wb_done));
        s->wb_pending = false;
    }
    if (saved_bytes) *saved_bytes = s->saved_bytes;
    return RA_OK;
}

int ra_kv_store_round_activity(const ra_kv_store* s, int seq, int round, uint32_t* turns, uint32_t* hits) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_round_activity: store is NULL");
    RA_REQUIRE(seq >= 0 && seq < s->cfg.B && round >= 0 && round < s->cfg.R_max, RA_ERR_INVALID_ARG,
               "kv_store_round_activity: (seq %d, round %d) outside [0,%d) x [0,%d)", seq, round, s->cfg.B,
               s->cfg.R_max);
    const ra_kv_store::Round& r = s->rounds[(size_t)seq * s->cfg.R_max + round];
    RA_REQUIRE(r.len >= 0, RA_ERR_STATE, "kv_store_round_activity: round %d of sequence %d was never registered", round,
               seq);
    if (turns) *turns = r.turns;
    if (hits) *hits = r.hits;
    return RA_OK;
}

// A dropped round keeps its index as an empty round: selecting it stages nothing.
static void drop_one(ra_kv_store::Round& r) {
    r.host = nullptr;
    r.len = 0;
    r.dropped = true;
}

int ra_kv_store_drop_round(ra_kv_store* s, int seq, int round) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_drop_round: store is NULL");
    RA_REQUIRE(seq >= 0 && seq < s->cfg.B && round >= 0 && round < s->cfg.R_max, RA_ERR_INVALID_ARG,
               "kv_store_drop_round: (seq %d, round %d) outside [0,%d) x [0,%d)", seq, round, s->cfg.B, s->cfg.R_max);
    RA_REQUIRE(!s->staged, RA_ERR_STATE, "kv_store_drop_round: rounds are staged; call ra_kv_store_release first");
    ra_kv_store::Round& r = s->rounds[(size_t)seq * s->cfg.R_max + round];
    RA_REQUIRE(r.len >= 0, RA_ERR_STATE, "kv_store_drop_round: round %d of sequence %d was never registered", round, seq);
    if (s->wb_pending) {  // the caller frees the host tensor next: no copy may still be writing it
        RA_HIP_CHECK(hipEventSynchronize(s->wb_done));
        s->wb_pending = false;
    }
    drop_one(r);
    return RA_OK;
}

int ra_kv_store_drop_inactive(ra_kv_store* s, uint32_t min_turns, int32_t* dropped_idx, int32_t* n_dropped) {
    RA_REQUIRE(s != nullptr && dropped_idx != nullptr && n_dropped != nullptr, RA_ERR_INVALID_ARG,
               "kv_store_drop_inactive: NULL argument");
    RA_REQUIRE(!s->staged, RA_ERR_STATE, "kv_store_drop_inactive: rounds are staged; call ra_kv_store_release first");
    if (s->wb_pending) {
        RA_HIP_CHECK(hipEventSynchronize(s->wb_done));
        s->wb_pending = false;
    }
    const int B = s->cfg.B, R = s->cfg.R_max;
    for (int b = 0; b < B; ++b) {
        int n = 0;
        for (int r = 0; r < R; ++r) {
            dropped_idx[(size_t)b * R + r] = -1;
            ra_kv_store::Round& rd = s->rounds[(size_t)b * R + r];
            if (rd.len < 0 || rd.dropped || rd.hits != 0 || rd.turns < min_turns) continue;
            drop_one(rd);
            dropped_idx[(size_t)b * R + n++] = r;
        }
        n_dropped[b] = n;
    }
    return RA_OK;
}

int ra_kv_store_release(ra_kv_store* s) {
    RA_REQUIRE(s != nullptr, RA_ERR_INVALID_ARG, "kv_store_release: store is NULL");
    if (s->staged) {
        // the pinned mirrors of the index tables are rewritten by the next stage call: make sure the
        // copies that read them have finished
        RA_HIP_CHECK(hipEventSynchronize(s->ready[s->cfg.n_layers - 1]));
        s->staged = false;
        s->staged_tok = 0;
    }
    return RA_OK;
}

}  // extern "C"
