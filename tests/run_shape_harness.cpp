// Host harness for the cut of a call's work (paper_2607_06731_amd/csrc/
// run_shape.h), built by tests/test_run_shape.py with the host compiler.
//
// TEST INFRASTRUCTURE.  Cuts random calls as configure_eval and k_order do and
// walks their items as k_run does: every (program, tile) is run exactly once,
// every piece fits the staged memory with the outputs that a split class keeps
// there, pieces end on whole windows, lists hold two items, and the running sums
// behind the staged memory are aligned for 64-bit values.
//
// Usage: run_shape_harness SEED CALLS.  Prints the calls and items looked at;
// exit status 1 with a line on stderr at the first failure.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#define __host__
#define __device__
#include "run_shape.h"

#define CHECK(cond)                                                                                                 \
    do {                                                                                                            \
        if (!(cond)) {                                                                                              \
            std::fprintf(stderr, "%s: fit %d vars %d cases %lld class %d programs %d tile_lds %d tile_max %d\n",    \
                         #cond, fit, n_vars, (long long)n_cases, c, count, tile_lds, tile_max);                     \
            return 1;                                                                                               \
        }                                                                                                           \
    } while (0)

int main(int argc, char** argv)
{
    if (argc != 3) return 2;
    std::mt19937_64 rng(std::strtoull(argv[1], nullptr, 10));
    const int calls = std::atoi(argv[2]);
    std::uniform_real_distribution<double> u01(0.0, 1.0);
    auto log_int = [&](double lo, double hi) { return (int64_t)std::exp(std::log(lo) + u01(rng) * (std::log(hi) - std::log(lo))); };
    long long items_seen = 0;
    for (int call = 0; call < calls; ++call) {
        const int fit = (int)(rng() % 4);            // MSE, correlation, reward, outputs
        const int32_t n_vars = (int32_t)(rng() % 3 ? rng() % 21 : rng() % 159);
        const bool wide = n_vars >= kWideVars;
        const int64_t n_cases = log_int(1, 3e6);
        const int32_t lds_choice[5] = {4096, 24 * 1024, 40 * 1024, 65536, (int32_t)(4096 + rng() % 61440)};
        const int32_t tile_lds = fit == 3 ? 24 * 1024 : lds_choice[rng() % 5];
        const int32_t count = (int32_t)log_int(1, 3e4);
        const int32_t max_choice[4] = {32, 1, 2, 8};
        const int32_t tile_max = fit == 3 ? predict_tiles(count) : max_choice[rng() % 4];
        const int32_t rows = staged_rows(fit == 3, n_vars), lds_floats = run_lds_floats(rows, tile_lds);
        const int32_t chunk = wide ? kRunWaves : (fit == 1 ? 32 : kChunkMax);
        const int32_t g_max = std::min<int32_t>(rng() % 3 ? 64 : (int32_t)(1 + rng() % 128), chunk);
        const int32_t list = wide ? 2 * kRunWaves : kListed;
        for (int c = 0; c < kClasses; ++c) {
            CHECK(lds_floats % 4 == 0);
            CHECK(rows == n_vars + (fit != 3));          // outputs have no targets
            CHECK((int64_t)rows * 256 <= lds_floats);
            const TileShape t = tile_shape(n_cases, class_k(c, n_vars), n_vars, tile_lds, tile_max);
            CHECK(t.sub == sub_cases(c) && t.n_tiles >= 1 && t.n_tiles <= tile_max);
            const ClassCut cut = class_cut(c, count, t.passes, t.n_tiles, n_cases, rows, g_max, 4 * 3 * 256, lds_floats,
                                           !wide && rng() % 2, fit == 3);
            CHECK(cut.G >= 1 && cut.G <= g_max);
            CHECK(cut.split || (int64_t)t.passes * t.sub > staged_cases(lds_floats, rows) || cut.G <= kRunOn ||
                  cut.G * std::min<int64_t>((int64_t)t.passes * t.sub, (n_cases + 255) / 256 * 256) <= kRunOnCases);
            const int32_t m = item_tiles(t.passes, t.n_tiles, c, rows, lds_floats, cut.m_cap);
            const int32_t runs = item_groups(t.n_tiles, m), groups = (count + cut.G - 1) / cut.G;
            CHECK(cut.items == (uint32_t)groups * (uint32_t)runs);
            const int64_t tile = (int64_t)t.passes * t.sub, cap = staged_cases(lds_floats, rows);
            const bool whole = tile <= cap;
            CHECK(!whole || cut.G + cut.G <= list);
            std::vector<int> seen((size_t)t.n_tiles, 0);
            for (int32_t tg = 0; tg < runs; ++tg) {
                const int32_t first_tile = tg * m, tiles = std::min(m, t.n_tiles - first_tile);
                CHECK(tiles >= 1 && (whole || tiles == 1));
                for (int32_t k = 0; k < tiles; ++k) ++seen[(size_t)(first_tile + k)];
                const int64_t first = tile * first_tile, last = std::min(first + tile * tiles, n_cases);
                CHECK(first < last);
                const int32_t window = t.window * t.sub;
                const int64_t step = whole ? last - first : piece_cases(cap, window);
                CHECK(whole || step % window == 0);
                for (int64_t f0 = first; f0 < last; f0 += step) {
                    const int64_t cases = std::min(step, last - f0), stride = (cases + 255) & ~(int64_t)255;
                    CHECK(rows * stride <= lds_floats);
                    if (cut.split && fit != 3) CHECK((rows + std::min(cut.G, count)) * stride <= lds_floats);
                    ++items_seen;
                    if (f0 - first > 8 * step && f0 + 8 * step < last) f0 += (last - f0) / step / 2 * step;   // (the middle alike)
                }
            }
            for (int v : seen) CHECK(v == 1);
            CHECK(!cut.split || (whole && m == 1 && cut.G <= kSplitMax));
        }
    }
    std::printf("%d %lld\n", calls, items_seen);
    return 0;
}
