// The divisions of the kernels' schedules and query rows (range_schedule.hpp) against the compiler's: Divisor up to the largest
// numerator it is made for, RowsPerToken up to its last row, and the reciprocal that small_div takes on the device, off by a unit
// in its last place either way.
#include <cmath>
#include <cstdio>
#include <random>

#include "range_schedule.hpp"

int main() {
    long long bad = 0, n = 0;
    std::mt19937 rng(1);
    auto check = [&](unsigned got, unsigned a, unsigned b, const char* what) {
        ++n;
        if (got != a / b && ++bad <= 10) std::fprintf(stderr, "%s: %u / %u = %u\n", what, a, b, got);
    };
    auto by_reciprocal = [&](unsigned a, unsigned b) {
        const float r = 1.0f / (float)b;
        for (float x : {std::nextafterf(r, 0.f), r, std::nextafterf(r, 2.f)}) check((unsigned)(((float)a + 0.5f) * x), a, b, "reciprocal");
    };
    for (unsigned b = 1; b < (1u << 21); b += 1 + b / 300) {
        for (int k = 0; k < 200; ++k) {
            unsigned a = rng() % (1u << 21);
            if (k < 100) a = a / b * b - (k & 1);  // a multiple, or one short of it
            if (a < (1u << 21)) by_reciprocal(a, b);
        }
        by_reciprocal((1u << 21) - 1, b);
    }
    for (int d = 1; d < (1 << 30); d += 1 + d / 200)
        for (long long n_max : {(0x80000000ll - 1) / d, 0x80000000ll / d + 1, (long long)d}) {
            if (n_max > 0x3fffffff) n_max = 0x3fffffff;
            const ra::Divisor x = ra::divisor(d, n_max);
            for (int k = 0; k < 60; ++k) {
                long long a = rng() % (unsigned long long)(n_max + 1);
                if (k < 40) a = a / d * d - (k & 1);
                if (k == 59) a = n_max;
                if (a >= 0) check((unsigned)x.divide((int)a), (unsigned)a, (unsigned)d, "Divisor");
            }
        }
    for (int G = 1; G <= 16; ++G) {
        const ra::RowsPerToken per_token(G);
        for (unsigned row = 0; row < (1u << 27); row += row < 100000 ? 1 : 1 + rng() % 4000)
            for (unsigned r : {row, row / G * G, row / G * G + G - 1}) check((unsigned)per_token.token((int)r), r, (unsigned)G, "RowsPerToken");
        for (unsigned r = (1u << 27) - 100; r < (1u << 27); ++r) check((unsigned)per_token.token((int)r), r, (unsigned)G, "RowsPerToken");
    }
    std::printf("%s: %lld divisions, %lld wrong\n", bad ? "FAILED" : "ok", n, bad);
    return bad ? 1 : 0;
}
