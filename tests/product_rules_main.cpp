// Host rules that pick tiles, K ranges and the share of the vocabulary per launch, over sweeps of
// shapes: whatever they pick covers the product exactly, keeps to the kernels' limits and to the
// memory a plan may take.
#include <cstdio>
#include <cstdlib>

#include "../paper_2410_10989_amd/csrc/scheduler.h"

#define CHECK(cond, ...)                                        \
    do {                                                        \
        if (!(cond)) {                                          \
            std::printf("FAILED %s: ", #cond);                  \
            std::printf(__VA_ARGS__);                           \
            std::printf("\n");                                  \
            std::exit(1);                                       \
        }                                                       \
    } while (0)

int main() {
    using namespace flce;
    const int64_t Vs[] = {1, 63, 256, 257, 300, 1000, 4096, 7011, 8192, 12289, 32000, 50257, 128256, 152064, 262151, 1 << 20};
    const int64_t others[] = {1, 8, 64, 127, 128, 129, 256, 300, 512, 1000, 1024, 2047, 2304, 4096, 8192, 16384, 150001};
    const int64_t Ks[] = {1, 8, 63, 64, 65, 200, 512, 1000, 1024, 2304, 4096, 50257, 128256};
    long n = 0, shared = 0, small = 0;
    for (int tuned = 0; tuned < 2; ++tuned)
        for (int64_t V : Vs)
            for (int64_t o : others)
                for (int64_t K : Ks)
                    for (int tail = 0; tail < 2; ++tail) {
                        const VocabCut c = vocab_cut(tuned != 0, V, o, K, tail != 0);
                        ++n;
                        CHECK(c.tile == 256 || c.tile == 128 || (!tuned && c.tile == 64), "tile %d", c.tile);
                        CHECK(c.main >= 1 && c.main <= V, "main %lld of %lld", (long long)c.main, (long long)V);
                        if (c.tile < 256) ++small;
                        if (c.main == V) continue;
                        ++shared;
                        // whole 256-tiles that fit whole rounds of the CUs, and a rest on smaller tiles
                        CHECK(c.tile == 256 && c.main % 256 == 0, "shared launch: main %lld tile %d", (long long)c.main, c.tile);
                        CHECK(c.rest_tile == 128 || (!tuned && c.rest_tile == 64), "rest tile %d", c.rest_tile);
                        const int64_t per = (o + 255) / 256, t = c.main / 256 * per, all = tiles_of(V, o, 256);
                        CHECK(t <= all / 256 * 256 && t > all / 256 * 256 - per, "%lld tiles do not fill the rounds", (long long)t);
                    }
    CHECK(shared > 0 && small > 0, "a branch of the rule is never taken");
    long cut = 0, streaming = 0;
    for (int tuned = 0; tuned < 2; ++tuned)
        for (int64_t rows : others)
            for (int64_t H : others)
                for (int64_t V : Vs)
                    for (size_t budget : {(size_t)1, (size_t)1 << 20, (size_t)1 << 30, (size_t)1 << 33})
                    for (bool bounded : {false, true}) {
                        if (H > 16384) continue;
                        const ProductCut c = dx_cut(tuned != 0, rows, H, V, budget, bounded);
                        const int tile = tuned ? 256 : 128;
                        CHECK(!bounded || c.ranges <= choose_ksplit(tiles_of(rows, H, tile), tuned ? (V + 63) / 64 : V / 4,
                                                                    std::min(16, max_dx_ranges(budget, round_up(rows, tile), H))),
                              "a bounded cut takes %d ranges", c.ranges);
                        CHECK(c.tile == 256 || c.tile == 128 || (!tuned && c.tile == 64), "dX tile %d", c.tile);
                        CHECK(c.ranges >= 1 && c.ranges <= 64, "dX ranges %d", c.ranges);
                        // large tiles in more than 16 ranges: operands that stream from HBM, one round of long ranges
                        if (tuned && c.tile == 256 && c.ranges > 16) {
                            ++streaming;
                            CHECK(!bounded && dx_streams(rows, H, V), "streaming cut");
                            CHECK(V / c.ranges >= 1024 && tiles_of(rows, H, 256) * c.ranges <= 256, "streaming cut into %d", c.ranges);
                        }
                        if (c.ranges == 1) continue;
                        ++cut;
                        CHECK((size_t)c.ranges * (size_t)rows * (size_t)H * 4 <= budget / 2, "partial results past half the budget");
                        CHECK(V / c.ranges >= 256 || (tuned && c.tile == 256 && (V + 63) / 64 / c.ranges >= 64), "short range");
                        // the kernels' ranges of K steps (64, 32 or 16 elements) tile the steps and none is empty
                        const int64_t bk = tuned ? 64 : c.tile == 64 ? 32 : 16, steps = (V + bk - 1) / bk;
                        int64_t at = 0;
                        for (int r = 0; r < c.ranges; ++r) {
                            const int64_t b = steps * r / c.ranges, e = steps * (r + 1) / c.ranges;
                            CHECK(b == at && e > b, "ranges do not tile the K steps");
                            at = e;
                        }
                        CHECK(at == steps, "K steps lost");
                    }
    CHECK(cut > 0 && streaming > 0, "no dX product is cut");
    // a few outputs of either size: what the dX tests rely on to reach both tile sizes, and the device's own
    // choice of ranges for fewer live rows (256-tiles only)
    const size_t gib = (size_t)1 << 30;
    CHECK(dx_cut(true, 1024, 512, 8192, gib, false).tile == 128, "small outputs take small tiles");
    CHECK(dx_cut(true, 600, 256, 16384, gib, false).tile == 128, "small outputs take small tiles");
    CHECK(dx_cut(true, 2047, 1000, 50257, gib, false).tile == 256, "long products keep the large tiles");
    const struct { int64_t rows, H, V; int tile, ranges; } streams[] = {
        {257, 512, 180001, 256, 64}, {700, 512, 128256, 256, 42}, {1024, 512, 128256, 256, 32}, {2048, 512, 128256, 256, 16},
        {24, 3584, 40003, 128, 18}, {1024, 512, 8192, 128, 8},   // (the last one's operands stay in the cache)
    };
    for (const auto& c : streams) {
        const ProductCut got = dx_cut(true, c.rows, c.H, c.V, gib, false);
        CHECK(got.tile == c.tile && got.ranges == c.ranges, "%lld x %lld x %lld: %d ranges of %d-tiles", (long long)c.rows,
              (long long)c.H, (long long)c.V, got.ranges, got.tile);
        for (const size_t part : {(size_t)0, (size_t)3 << 20, (size_t)20 << 20}) {   // in less room
            const ProductCut less = dx_cut(true, c.rows, c.H, c.V, gib, false, part);
            CHECK(less.ranges == 1 || (size_t)less.ranges * c.rows * c.H * 4 <= part, "%d ranges in %zu bytes", less.ranges, part);
        }
        // one round: the live rows do not change the ranges
        const Plan p = make_plan(c.rows, c.H, c.V, 1, gib, false, true, gib);
        CHECK(p.dx_dyn == (p.dx_tile == 256 && tiles_of(c.rows, c.H, 256) * p.dx_ranges > 256), "ranges chosen on the device");
    }
    const ProductCut dyn = dx_cut(true, 4100, 2048, 29596, gib, false);
    auto live = [&](int64_t rows) { return choose_ksplit(tiles_of(rows, 2048, 256), (29596 + 63) / 64, dyn.ranges); };
    CHECK(dyn.tile == 256 && dyn.ranges == 7 && live(2460) == 3 && live(1148) == 6, "tile %d, ranges %d, live %d and %d",
          dyn.tile, dyn.ranges, live(2460), live(1148));
    // Workspace: the least plan fits the sizes that callers may have set aside for the plan of large tiles
    // (with the index maps of the compaction only for fp32 and H % 64 == 0), the bounded one too but for the maps.
    long plans = 0;
    for (int dtype = 0; dtype < 2; ++dtype)
        for (int64_t BT : {1, 4, 100, 600, 1000, 2047, 8192, 33000})
            for (int64_t H : {1, 7, 8, 64, 100, 256, 968, 1000, 4096})
                for (int64_t V : {1, 300, 1000, 4096, 16384, 16916, 50257})
                    for (int chunk_rows : {0, 256}) {
                        const size_t es = elem_size(dtype);
                        const size_t budget = chunk_rows ? chunk_rows * (size_t)round_up(V, 64) * es : (size_t)1 << 30;
                        auto plan = [&](Room r) { return make_plan(BT, H, V, dtype, budget, false, true, budget, r); };
                        const Plan full = plan(Room::full), bounded = plan(Room::bounded), least = plan(Room::least);
                        const bool tuned = dtype != 0 && H % 8 == 0;
                        const int64_t C = full.C, rows = full.nchunks > 1 ? C : BT, tile = tuned ? 256 : 128;
                        const int ranges = choose_ksplit(tiles_of(rows, H, tile), tuned ? (V + 63) / 64 : V / 4,
                                                         std::min(16, max_dx_ranges(budget, round_up(rows, tile), H)));
                        auto r256 = [](size_t b) { return (b + 255) / 256 * 256; };
                        const size_t aside = 256 + r256(4 * C) + r256((size_t)C * full.ldz * es) +
                                             r256(full.fp32_dw_acc ? (size_t)V * H * 4 : 0) +
                                             r256(ranges > 1 ? (size_t)ranges * C * H * 4 : 0) + 2 * r256((size_t)C * H * es) + 256 +
                                             r256(full.tail_bytes);
                        const size_t maps = full.compact ? r256(4 * C) + r256(8 * C) : 0;
                        const bool without = dtype != 0 && H % 64 != 0;
                        ++plans;
                        CHECK(least.total <= aside + (without ? 0 : maps), "dtype %d %lld x %lld x %lld: least %zu, set aside %zu", dtype,
                              (long long)BT, (long long)H, (long long)V, least.total, aside);
                        CHECK(bounded.total <= aside + maps, "bounded %zu, set aside %zu", bounded.total, aside + maps);
                        CHECK(least.C == full.C && bounded.C == full.C && least.nchunks == full.nchunks, "the room changes the chunks");
                    }
    CHECK(plans > 0, "no plan");
    // One launch for both gradients or two: shapes measured on either side of each line of the rule, bf16 unless
    // it says otherwise (the times stand beside grads_in_one).
    struct { int dtype; int64_t BT, H, V; bool want_dw, places, one; } const grads[] = {
        {1, 18, 960, 384, true, true, true}, {0, 3639, 16, 489, true, true, true}, {0, 4474, 128, 101, true, true, false},
        {0, 6723, 80, 91, true, true, false}, {0, 5018, 64, 622, true, true, false},
        // dX alone
        {1, 56, 1024, 400, false, true, true}, {1, 64, 1024, 400, false, true, false}, {1, 400, 64, 800, false, true, false},
        {1, 1901, 1024, 433, false, true, true}, {1, 1901, 144, 433, false, true, false},
        {1, 44, 368, 110, false, true, true}, {1, 77, 1016, 161, false, true, false}, {1, 221, 720, 101, false, true, false},
        {1, 221, 720, 101, false, false, true}, {1, 8010, 32, 125, false, true, true}, {0, 5025, 120, 284, false, true, true},
        {1, 1024, 512, 8192, false, true, false},
        // dX in K ranges
        {1, 1024, 512, 8192, true, true, true}, {1, 497, 2304, 4240, true, true, true}, {1, 377, 832, 56112, true, true, true},
        {1, 459, 64, 42658, true, true, false}, {1, 617, 64, 44793, true, true, false}, {1, 2008, 64, 37387, true, true, false},
        {1, 400, 384, 14000, true, true, false}, {1, 200, 384, 42000, true, true, false}, {1, 620, 256, 42000, true, true, false},
        {1, 280, 512, 14000, true, true, false}, {1, 900, 512, 9000, true, true, true}, {1, 900, 1152, 9000, true, true, true},
        {1, 2000, 64, 70000, true, true, true}, {1, 400, 64, 100000, true, true, false}, {1, 3820, 64, 39221, true, true, true},
        {1, 86, 824, 19859, true, true, false}, {1, 102, 192, 37246, true, true, true}, {1, 101, 3328, 9664, true, true, true},
        {1, 16, 320, 52308, true, true, false}, {1, 20, 832, 23116, true, false, false}, {1, 2, 1728, 5253, true, true, true},
        {1, 16, 48, 34492, true, true, false}, {1, 5, 64, 15903, true, true, true}, {1, 24, 64, 154137, true, true, true},
        {1, 24, 1024, 31078, true, false, false}, {0, 256, 512, 4096, true, true, true}, {0, 54, 384, 11328, true, true, false},
    };
    for (const auto& g : grads) {
        const bool bf16 = g.dtype != 0;
        const size_t budget = std::max<size_t>((size_t)1 << 30, (size_t)4096 * round_up(g.V, 64) * elem_size(g.dtype));
        const Plan p = make_plan(g.BT, g.H, g.V, g.dtype, budget, false, true, budget);
        const bool tuned = bf16 && p.fast_dw_last;
        const VocabCut cut = vocab_cut(tuned, g.V, g.H, g.BT, p.tail_bytes > 0);
        CHECK(grads_in_one(p, cut, bf16, g.want_dw, tuned, g.places, g.BT, g.H, g.V) == g.one, "%lld x %lld x %lld dtype %d",
              (long long)g.BT, (long long)g.H, (long long)g.V, g.dtype);
    }
    // the rotated K loop visits every step once
    for (int nk = 1; nk <= 70; ++nk)
        for (int rot = 0; rot < nk; ++rot) {
            unsigned char seen[70] = {0};
            for (int kt = 0; kt < nk; ++kt) {
                const int k = rotated_step(kt, rot, nk);
                CHECK(k >= 0 && k < nk && !seen[k], "step %d of %d", k, nk);
                seen[k] = 1;
            }
        }
    std::printf("product rules: %ld shares (%ld of them of two launches), %ld cut dX products\n", n, shared, cut);
    return 0;
}
