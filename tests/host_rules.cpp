// Device rules that are plain arithmetic, run on the CPU (test_host_rules.py compiles this file for the
// host only).  Prints one line per rule: its name, then "ok" or what is wrong.
#include <cmath>
#include <cstdio>

#include "qvg_attn_tiles.hpp"
#include "qvg_kmeans.hpp"

using namespace qvg;

// every tile of the cache belongs to exactly one part, in order, and none lies past the end
static const char *tiles_of(int64_t n_kv, int64_t chunk_len, int parts, bool ends_only) {
    AttnArgs a{};
    a.n_kv = n_kv; a.chunk_len = chunk_len; a.n_chunks = (int)((n_kv - 1) / chunk_len + 1); a.parts = parts;
    const int64_t tpc = tiles_per_chunk(span_of(a, 0));
    for (int p = 0; p < parts; ++p) {
        const Span s = span_of(a, p);
        Tile t = first_tile(s);
        int64_t g = p;                                     // the tile's number in the cache
        if (ends_only && t.valid) {                        // start near the end instead
            const int64_t last = (int64_t)(a.n_chunks - 1) * tpc + (n_kv - (int64_t)(a.n_chunks - 1) * chunk_len + kAtKv - 1) / kAtKv - 1;
            g = last - (last - p) % parts;
            t = place_tile(s, (int)(g / tpc), (int)(g % tpc));
        }
        for (; t.valid; t = next_tile(s, t), g += parts) {
            if (t.chunk != g / tpc) return "order";
            if (t.t0 < 0 || t.t0 >= n_kv || t.cend > n_kv || t.t0 >= t.cend) return "range";
            if (t.t0 != t.chunk * chunk_len + g % tpc * kAtKv) return "position";
        }
        if (g % tpc == 0 && g / tpc < a.n_chunks) return "end";
    }
    return "ok";
}

// bounds of squared norms: not below the norm, at most 2^-21 above it, and ordered as bit patterns
static const char *norm_bounds() {
    uint32_t prev = 0;
    double v = 0.0;
    for (int i = 0; i < 4000; ++i) {
        const float b = norm_bound(split_half_norm(v));
        const uint32_t u = norm_order(b);
        if (u & 0x80000000u) return "sign";
        if ((double)b < v || (double)b > v * (1.0 + 0x1p-21)) return "bound";
        if (u < prev) return "order";
        prev = u;
        v = v == 0.0 ? 0x1p-100 : v * 1.0353;              // to about 2^100
    }
    return "ok";
}

// the reach is not below (||x|| + d)^2, from the smallest normal numbers to where the sum overflows; the
// device's square root flushes subnormals
static const char *norm_reaches() {
    auto flushing = [](float v) { return v < 0x1p-126f ? 0.0f : sqrtf(v); };
    for (int i = -126; i < 127; ++i)
        for (int j = -126; j < 127; ++j) {
            const float xn = ldexpf(1.37f, i), d2 = ldexpf(1.61f, j);
            const double want = pow(sqrt((double)xn) + sqrt((double)d2), 2.0);
            const double got = norm_reach(xn, d2, flushing);
            if (got < want) return "below";
            if ((double)xn * d2 > 3.4e38) continue;          // the product overflows: the reach is infinite, the table's own norms limit the band
            if (got > want * (1.0 + 0x1p-8) + 0x1p-58) return "above";
        }
    return "ok";
}

// sums just below a power of two (the largest relative errors of s r), above one, and in between, over every count
static const char *quotients() {
    uint64_t state = 1;
    for (int n = 1; n <= 8192; ++n) {
        const double r = 1.0 / n;
        for (int i = 0; i < 400; ++i) {
            state = state * 6364136223846793005ull + 1442695040888963407ull;
            const uint64_t some = state >> 12, top = (1ull << 52) - 1;
            const uint64_t m = i < 100 ? top - i : i < 150 ? i - 100 : i < 250 ? top - (some >> (i % 40)) : some;
            const double s = ldexp((double)((1ull << 52) | (m & top)), i % 2 ? -133 : 40);
            if (quotient(s, n, r) != s / n || quotient(-s, n, r) != -s / n) return "not the rounded quotient";
            const double whole = (double)(m & 0xffffffffu) * n;      // exact ones
            if (quotient(whole, n, r) != whole / n) return "not the exact quotient";
        }
    }
    return "ok";
}

int main() {
    std::printf("quotients %s\n", quotients());
    std::printf("norm_reaches %s\n", norm_reaches());
    std::printf("norm_bounds %s\n", norm_bounds());
    std::printf("tiles_small %s\n", tiles_of(1000, 130, 3, false));
    std::printf("tiles_one_chunk %s\n", tiles_of(8191, (int64_t)1 << 36, 16, false));
    const int64_t top = 0x7fffffff;
    std::printf("tiles_top %s\n", tiles_of(top, 4680, 256, true));
    std::printf("tiles_top_one_chunk %s\n", tiles_of(top, (int64_t)1 << 36, 256, true));
    std::printf("tiles_top_undivided %s\n", tiles_of(top, (int64_t)1 << 36, 1, true));
    return 0;
}
