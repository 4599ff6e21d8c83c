// How the host store's bytes travel (fake_hip.hpp): slices of four megabytes and more (of the write-back: of one) by asynchronous
// copies, which leave the compute units to the work beside them, smaller ones by the kernel if it can reach the tensor.  Every
// byte of the selection goes exactly once, a layer's wait covers its copies, and the side stream ends behind all of them.
//
// exit status 0 = every check passed
#include <algorithm>

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

constexpr int kLayers = 6, kRounds = 8, kHkv = 8, kD = 128;
static size_t slice(int len, int layers) { return (size_t)(len + (len + 15) / 16 * 16) * kHkv * kD * 2 * layers; }
static bool is_mover(const fake::Op& op) { return op.what == "kernel" && op.name.find("stage_kernel") != std::string::npos; }

int main() {
    auto& s = fake::state();
    fake::Stream side{0}, compute{0};
    ra_store_cfg cfg = {};
    cfg.n_layers = kLayers;
    cfg.B = 2;
    cfg.R_max = kRounds;
    cfg.Hkv = kHkv;
    cfg.d = kD;
    cfg.dtype = RA_BF16;
    cfg.device_pool_bytes = (size_t)512 << 20;
    ra_kv_store* store = nullptr;
    CHECK(ra_kv_store_create(&store, &cfg) == RA_OK);
    auto host = [&](int len, size_t offset) {
        void* p = nullptr;
        (void)hipHostMalloc(&p, ra_kv_store_round_bytes(store, len) + offset, 0);
        return static_cast<char*>(p) + offset;
    };
    struct Case {
        int order;
        std::vector<int> len;   // the rounds of both sequences
        std::vector<size_t> at;  // bytes that each tensor begins behind its allocation
        bool kernel;             // is there anything for the kernel
    };
    const std::vector<int> groups[3] = {{6}, {1, 1, 1, 1, 1, 1}, {1, 2, 1, 1, 1}};  // layers of a group, by order
    const std::vector<Case> cases = {
        {RA_STAGE_GROUPED, {2000, 1200, 1024, 3000}, {0, 0, 0, 0}, false},
        {RA_STAGE_GROUPED, {2000, 900, 450, 3000}, {0, 0, 0, 0}, true},  // two of them copied in the group of two layers alone
        {RA_STAGE_LAYER_MAJOR, {2000, 1025, 1024, 3000}, {0, 0, 0, 0}, false},
        {RA_STAGE_LAYER_MAJOR, {2000, 1025, 1023, 3000}, {0, 0, 0, 0}, true},
        {RA_STAGE_ROUND_MAJOR, {700, 300, 2000}, {0, 0, 0}, false},
        {RA_STAGE_GROUPED, {700, 20, 3000, 0}, {0, 0, 0, 0}, true},
        {RA_STAGE_GROUPED, {1, 20, 33, 90}, {0, 0, 0, 0}, true},
        {RA_STAGE_GROUPED, {1, 20, 33, 90}, {0, 8, 0, 0}, true},  // one that the kernel cannot read in 16-byte pieces
        {RA_STAGE_GROUPED, {1, 20, 33, 90}, {8, 8, 8, 8}, false},
        {RA_STAGE_GROUPED, {1200}, {0}, false},
    };
    for (const Case& c : cases) {
        const int n = (int)c.len.size();
        std::vector<int32_t> sel(2 * kRounds, -1), n_sel(2, 0);
        std::vector<char*> tensor(n);
        std::vector<int64_t> left;  // bytes of every (group, round) still to come
        for (int r = 0; r < n; ++r) {
            const int b = r % 2;
            tensor[r] = host(c.len[r], c.at[r]);
            CHECK(ra_kv_store_register_round(store, b, r / 2, tensor[r], c.len[r]) == RA_OK);
            sel[b * kRounds + n_sel[b]++] = r / 2;
        }
        s.ops.clear();
        CHECK(ra_kv_store_stage(store, sel.data(), n_sel.data(), c.order, fake::handle(side)) == RA_OK);
        int movers = 0;
        for (const fake::Op& op : s.ops) movers += is_mover(op);
        CHECK((movers > 0) == c.kernel);
        for (int r = 0; r < n; ++r) {
            size_t at = 0;
            for (int n_l : groups[c.order]) {
                const size_t bytes = slice(c.len[r], n_l);
                int copies = 0;
                for (const fake::Op& op : s.ops) copies += bytes && op.what == "copy" && op.src == tensor[r] + at && op.bytes == bytes;
                CHECK(copies == (bytes && (bytes >= (size_t)4 << 20 || c.at[r] % 16) ? 1 : 0));
                at += bytes;
            }
        }
        // A layer's waits: an event recorded behind each of the streams that its copies are on, and the last one on the side
        // stream behind everything.
        const std::vector<fake::Op> enqueued = s.ops;
        int layer = 0;
        size_t at_layer[16] = {};
        for (int n_l : groups[c.order]) {
            for (int l = layer; l < layer + n_l; ++l) {
                s.ops.clear();
                CHECK(ra_kv_store_wait_layer(store, l, fake::handle(compute)) == RA_OK);
                for (int r = 0; r < n; ++r)
                    for (size_t i = 0; i < enqueued.size(); ++i) {
                        if (enqueued[i].what != "copy" || enqueued[i].src != tensor[r] + at_layer[r]) continue;
                        bool covered = false;
                        for (const fake::Op& w : s.ops) covered |= w.what == "wait" && fake::reaches(enqueued, w.event, i);
                        CHECK(covered);
                    }
            }
            for (int r = 0; r < n; ++r) at_layer[r] += slice(c.len[r], n_l);
            layer += n_l;
        }
        for (size_t i = 0; i < enqueued.size(); ++i)
            if (enqueued[i].what == "copy" || is_mover(enqueued[i])) CHECK(fake::reaches_end(enqueued, fake::handle(side), i));
        CHECK(ra_kv_store_release(store) == RA_OK);
    }
    // The write-back: every tensor once, behind the gather, and the side stream behind all of them.
    void* cur = nullptr;
    (void)hipMalloc(&cur, (size_t)2 * 2000 * kHkv * kD * 2);
    const void* layers[kLayers];
    std::fill(layers, layers + kLayers, cur);
    for (int len0 : {10, 2000}) {
        const int32_t round[2] = {0, 0}, len[2] = {len0, 900};
        void* to[2] = {host(len0, 0), host(900, 0)};
        s.ops.clear();
        CHECK(ra_kv_store_save_round(store, round, len, layers, layers, 2000, to, fake::handle(compute), fake::handle(side)) == RA_OK);
        int gather = -1;
        for (size_t i = 0; i < s.ops.size(); ++i)
            if (s.ops[i].name.find("repack") != std::string::npos) gather = (int)i;
        for (int b = 0; b < 2; ++b) {
            int copies = 0;
            for (size_t i = 0; i < s.ops.size(); ++i) {
                if (s.ops[i].what != "copy" || s.ops[i].dst != to[b]) continue;
                ++copies;
                CHECK(s.ops[i].bytes == slice(len[b], kLayers) && gather >= 0 && fake::before(s.ops, gather, i));
            }
            CHECK(copies == (slice(len[b], kLayers) >= (size_t)1 << 20));
        }
        for (size_t i = 0; i < s.ops.size(); ++i)
            if (s.ops[i].what == "copy" || is_mover(s.ops[i])) {
                CHECK(gather >= 0 && fake::before(s.ops, gather, i));
                CHECK(fake::reaches_end(s.ops, fake::handle(side), i));
            }
        CHECK(ra_kv_store_save_wait(store, nullptr) == RA_OK);
    }
    CHECK(ra_kv_store_destroy(store) == RA_OK);
    std::printf("%s: %d failed checks\n", bad ? "FAILED" : "ok", bad);
    return bad ? 1 : 0;
}
