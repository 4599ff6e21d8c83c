// Which host tensors the store's kernels read and write themselves (fake_hip.hpp): those that lie in one allocation from their
// first byte to their last, allocated in a way that is coherent whatever the environment says.  Everything else is left to copies, which report an error where a kernel would fault.
//
// exit status 0 = every check passed
#include "fake_hip.hpp"
#include "round_attention.h"

static int bad = 0;
#define CHECK(x)                                                             \
    do {                                                                     \
        if (!(x)) {                                                          \
            ++bad;                                                           \
            std::fprintf(stderr, "line %d: %s  (%s)\n", __LINE__, #x, ra_last_error()); \
        }                                                                    \
    } while (0)

static fake::Stream side{0}, compute{0};

static ra_kv_store* make_store() {
    ra_store_cfg cfg = {};
    cfg.n_layers = 2;
    cfg.B = 1;
    cfg.R_max = 2;
    cfg.Hkv = 2;
    cfg.d = 64;
    cfg.dtype = RA_BF16;
    cfg.device_pool_bytes = 64 << 20;
    ra_kv_store* store = nullptr;
    CHECK(ra_kv_store_create(&store, &cfg) == RA_OK);
    return store;
}
static bool kernel_moved() {
    bool moved = false, copied = false;
    for (const fake::Op& op : fake::state().ops) {
        moved |= op.name.find("stage_kernel") != std::string::npos;
        copied |= op.what == "copy";
    }
    CHECK(moved != copied);
    return moved;
}
// Whether the kernel stages (then: saves) a tensor of `len` tokens at p.
static bool staged_by_kernel(void* p, int len) {
    ra_kv_store* store = make_store();
    const int32_t sel[2] = {0, -1}, n_sel = 1;
    CHECK(ra_kv_store_register_round(store, 0, 0, p, len) == RA_OK);
    fake::state().ops.clear();
    CHECK(ra_kv_store_stage(store, sel, &n_sel, RA_STAGE_GROUPED, fake::handle(side)) == RA_OK);
    const bool moved = kernel_moved();
    CHECK(ra_kv_store_destroy(store) == RA_OK);
    return moved;
}
static bool saved_by_kernel(void* p, int len) {
    ra_kv_store* store = make_store();
    void* cur = nullptr;
    (void)hipMalloc(&cur, 1 << 20);
    const void* layers[2] = {cur, cur};
    const int32_t round = 0, n = len;
    fake::state().ops.clear();
    CHECK(ra_kv_store_save_round(store, &round, &n, layers, layers, 100, &p, fake::handle(compute), fake::handle(side)) == RA_OK);
    const bool moved = kernel_moved();
    (void)hipFree(cur);
    CHECK(ra_kv_store_destroy(store) == RA_OK);
    return moved;
}
static void check_tensor(void* p, int len, bool by_kernel) {
    CHECK(staged_by_kernel(p, len) == by_kernel);
    CHECK(saved_by_kernel(p, len) == by_kernel);
}

int main() {
    ra_kv_store* store = make_store();
    const size_t bytes = ra_kv_store_round_bytes(store, 33);
    CHECK(ra_kv_store_destroy(store) == RA_OK);
    char* memory = nullptr;
    if (posix_memalign(reinterpret_cast<void**>(&memory), 4096, 8 * bytes)) return 2;
    // from the first byte of an allocation to its last, inside one, up to its end
    fake::place(memory, bytes, 0);
    check_tensor(memory, 33, true);
    fake::place(memory, 3 * bytes, 0);
    check_tensor(memory + 64, 33, true);
    check_tensor(memory + 2 * bytes, 33, true);
    // past its end: into nothing, and into another allocation behind a hole or right behind it
    check_tensor(memory + 2 * bytes + 16, 33, false);
    fake::place(memory + 3 * bytes + 16, bytes, 0);
    check_tensor(memory + 2 * bytes + 32, 33, false);
    fake::place(memory + 3 * bytes, 16, 0);
    check_tensor(memory + 2 * bytes + 32, 33, false);
    // Coherent whatever HIP_HOST_COHERENT says: allocations without flags, mapped ones and those that ask for it.  By the
    // environment: other flags alone.  Not, or not for kernels to read at speed: non-coherent, uncached and write-combined ones.
    char* other = memory + 5 * bytes;
    for (unsigned flags : {(unsigned)hipHostMallocDefault, (unsigned)hipHostMallocMapped, (unsigned)hipHostMallocCoherent,
                           (unsigned)(hipHostMallocPortable | hipHostMallocMapped), (unsigned)(hipHostMallocPortable | hipHostMallocCoherent)}) {
        fake::place(other, bytes, flags);
        check_tensor(other, 33, true);
    }
    for (unsigned flags : {(unsigned)hipHostMallocPortable, (unsigned)hipHostMallocNumaUser, (unsigned)hipHostMallocWriteCombined,
                           (unsigned)(hipHostMallocWriteCombined | hipHostMallocMapped), (unsigned)hipHostMallocNonCoherent,
                           (unsigned)(hipHostMallocNonCoherent | hipHostMallocMapped), (unsigned)(hipHostMallocUncached | hipHostMallocMapped)}) {
        fake::place(other, bytes, flags);
        check_tensor(other, 33, false);
    }
    std::printf("%s: %d failed checks\n", bad ? "FAILED" : "ok", bad);
    return bad ? 1 : 0;
}
