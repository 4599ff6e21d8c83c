// Which launches a question's attention is made of (fake_hip.hpp), by the size of the workspace: with room for the partial results
// of ranges of eight key tiles it plans itself, as with room for shorter ones, and no planning kernel runs.
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

static size_t up(size_t x) { return (x + 255) / 256 * 256; }

int main() {
    auto& s = fake::state();
    ra_ctx* ctx = nullptr;
    CHECK(ra_create(&ctx, 0) == RA_OK);
    void *memory = nullptr, *ws = nullptr;
    (void)hipMalloc(&memory, 1 << 20);  // (what the calls point to is never read)
    (void)hipMalloc(&ws, (size_t)256 << 20);
    for (int B : {1, 3})
        for (int R : {5, 40, 1000})
            for (int tokens : {300, 700, 2000, 9000})
                for (int form = 0; form < 4; ++form) {
                    if (B * R > 1024 || (R == 1000 && tokens == 9000)) continue;  // always planned apart; more ranges than LDS has room for
                    const bool watershed = form & 1;
                    const int q_len = form & 2 ? 40 : 20, Hq = 32, Hkv = 8, cur = q_len, d = 128;
                    ra_kv_view v = {};
                    v.k = v.v = memory;
                    v.seg_off = v.seg_off_v = static_cast<int64_t*>(memory);
                    v.seg_len = v.n_rounds = static_cast<int32_t*>(memory);
                    v.B = B;
                    v.R_max = R;
                    v.Hkv = Hkv;
                    v.d = d;
                    v.dtype = RA_BF16;
                    v.max_tokens = tokens;
                    float* out = static_cast<float*>(memory);
                    // number of planning kernels, -1: refused
                    auto plans = [&](size_t bytes) {
                        CHECK(ra_set_workspace(ctx, ws, bytes) == RA_OK);
                        s.ops.clear();
                        const int rc = watershed ? ra_watershed_attn_prefill(ctx, nullptr, memory, q_len, Hq, &v, memory, memory, cur, 0.1f, out, out, out, out)
                                                 : ra_round_sparse_attn_prefill(ctx, nullptr, memory, q_len, Hq, &v, nullptr, nullptr, memory, memory, cur, 0.1f, out, out);
                        if (rc != RA_OK) return -1;
                        int n = 0;
                        for (const fake::Op& op : s.ops) n += op.name.find("plan_kernel") != std::string::npos;
                        return n;
                    };
                    // head, tables, and of every row and part 128 sums, a maximum and a sum
                    const size_t rows = (size_t)B * q_len * Hq, tables = up((size_t)B * (((R + 1) * 24 + 4 + 16 + 15) / 16 * 16));
                    auto need = [&](int parts, int values) {  // values: in a row of the score output
                        const size_t scores = watershed ? up(rows * values * 4) + up((size_t)B * Hq * R * 4) : 0;
                        return 32768 + tables + up(rows * parts * d * 4) + 2 * up(rows * parts * 4) + scores;
                    };
                    const int eight = std::max(1, std::min(16, (tokens + cur) / 256)), chunks = tokens / 256 + R + cur / 256 + 1;
                    const size_t least = need(std::min(8, eight), chunks);
                    CHECK(plans(least - 256) == -1);
                    CHECK(plans(least) >= 0);
                    for (int parts = eight + 2; parts <= 20; ++parts) CHECK(plans(need(parts, std::max(chunks, R + parts))) == 0);
                    if (!watershed || eight > 1) CHECK(plans(need(eight + 2, chunks)) == 0);
                }
    std::printf("%s: %d failed checks\n", bad ? "FAILED" : "ok", bad);
    return bad ? 1 : 0;
}
