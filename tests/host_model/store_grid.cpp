// The gather of a saved round over many layers (fake_hip.hpp): no launch has 2^32 threads or more in a dimension, which the
// runtime refuses, and the launches cover every layer and 16-token tile once.
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

int main() {
    auto& s = fake::state();
    fake::Stream side{0}, compute{0};
    struct Case {
        int layers, len;
    };
    for (const Case& c : {Case{3, 40}, Case{128, 100000}, Case{128, 2097153}, Case{80, 4000000}, Case{1, 4000000}}) {
        ra_store_cfg cfg = {};
        cfg.n_layers = c.layers;
        cfg.B = 1;
        cfg.R_max = 1;
        cfg.Hkv = 1;
        cfg.d = 8;
        cfg.dtype = RA_BF16;
        const size_t tiles = (c.len + 15) / 16, bytes = (c.len + tiles * 16) * 16 * (size_t)c.layers;
        cfg.device_pool_bytes = bytes;
        ra_kv_store* store = nullptr;
        CHECK(ra_kv_store_create(&store, &cfg) == RA_OK);
        CHECK(ra_kv_store_round_bytes(store, c.len) == bytes);
        void* host = reinterpret_cast<void*>((uintptr_t)1 << 45);  // (never read)
        fake::place(host, bytes, 0);
        std::vector<const void*> cur(c.layers, host);
        const int32_t round = 0, len = c.len;
        s.ops.clear();
        CHECK(ra_kv_store_save_round(store, &round, &len, cur.data(), cur.data(), c.len, &host, fake::handle(compute), fake::handle(side)) == RA_OK);
        size_t groups = 0;
        for (const fake::Op& op : s.ops) {
            if (op.what != "kernel") continue;
            CHECK((uint64_t)op.grid.x * op.block.x < (uint64_t)1 << 32);
            if (op.name.find("repack") != std::string::npos) groups += (size_t)op.grid.x * op.grid.y * op.grid.z;
        }
        CHECK(groups == tiles * c.layers);
        CHECK(ra_kv_store_destroy(store) == RA_OK);
    }
    std::printf("%s: %d failed checks\n", bad ? "FAILED" : "ok", bad);
    return bad ? 1 : 0;
}
