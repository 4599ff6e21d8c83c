// The host store's enqueueing calls where the current device is not the store's (fake_hip.hpp): on explicit streams of the
// store's device everything, waits included, goes to that device and the current one comes back; a stream of another device,
// the null stream of the current one among them, is refused before anything is enqueued.
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
    fake::Stream on0{0}, on1{1}, other1{1};
    ra_store_cfg cfg = {};
    cfg.device = 1;
    cfg.n_layers = 3;
    cfg.B = 2;
    cfg.R_max = 4;
    cfg.Hkv = 2;
    cfg.d = 64;
    cfg.dtype = RA_BF16;
    cfg.device_pool_bytes = 64 << 20;
    ra_kv_store* store = nullptr;
    CHECK(ra_kv_store_create(&store, &cfg) == RA_OK);
    CHECK(s.current == 0);
    void *cur = nullptr, *host[2];
    (void)hipMalloc(&cur, 1 << 20);
    const void* layers[3] = {cur, cur, cur};
    for (void*& h : host) (void)hipHostMalloc(&h, ra_kv_store_round_bytes(store, 40), 0);
    const int32_t sel[8] = {0, -1, -1, -1, 0, -1, -1, -1}, n_sel[2] = {1, 1}, round[2] = {0, 0}, len[2] = {40, 33};
    auto save = [&](void* compute, void* side) { return ra_kv_store_save_round(store, round, len, layers, layers, 40, host, compute, side); };
    auto stage = [&](void* side) { return ra_kv_store_stage(store, sel, n_sel, RA_STAGE_GROUPED, side); };
    auto all_on = [&](int device) {
        bool ok = !s.ops.empty();
        for (const fake::Op& op : s.ops) ok &= op.device == device;
        s.ops.clear();
        return ok;
    };
    for (int current : {0, 1}) {
        s.current = current;
        s.ops.clear();
        CHECK(save(fake::handle(on1), fake::handle(other1)) == RA_OK);
        CHECK(all_on(1) && s.current == current);
        CHECK(stage(fake::handle(other1)) == RA_OK);  // waits for the write-back
        CHECK(fake::count("wait") == 1);
        CHECK(all_on(1) && s.current == current);
        CHECK(ra_kv_store_release(store) == RA_OK);
        // streams of the other device
        CHECK(save(fake::handle(on0), fake::handle(other1)) != RA_OK);
        CHECK(save(fake::handle(on1), fake::handle(on0)) != RA_OK);
        CHECK(save(fake::handle(on1), fake::handle(other1)) == RA_OK);
        s.ops.clear();
        CHECK(stage(fake::handle(on0)) != RA_OK);
        CHECK(s.ops.empty() && s.current == current);
        // the default streams: the current device's
        for (hipStream_t st : {(hipStream_t) nullptr, hipStreamLegacy, hipStreamPerThread}) {
            CHECK(save(fake::handle(on1), fake::handle(other1)) == RA_OK);
            s.ops.clear();
            CHECK((stage(st) == RA_OK) == (current == 1));
            CHECK(current == 1 ? fake::count("wait") == 1 && all_on(1) : s.ops.empty());
            CHECK(ra_kv_store_release(store) == RA_OK);
            CHECK((save(st, st) == RA_OK) == (current == 1));
            CHECK(current == 1 ? all_on(1) : s.ops.empty());
            CHECK(s.current == current);
        }
    }
    CHECK(ra_kv_store_destroy(store) == RA_OK);
    std::printf("%s: %d failed checks\n", bad ? "FAILED" : "ok", bad);
    return bad ? 1 : 0;
}
