// Host-side chunk scheduler and workspace layout.  Pure integer arithmetic, no
// HIP calls, so it can be exercised on a machine without a GPU.
//
// The method bounds memory by projecting only a chunk of C rows at a time
// (paper section 3.2, FLCE paragraph).  Here C is set by a byte budget for the
// chunk's logits instead of the paper's power-of-two rule: on this chip each
// chunk re-reads W twice and read-modify-writes the fp32 dW accumulator, so C
// has to stay in the thousands for the products to remain compute bound.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#if defined(__HIPCC__)
#define FLCE_HD __host__ __device__
#else
#define FLCE_HD
#endif

namespace flce {

constexpr size_t DYN_WORDS = 4;        // device words of the compaction (see compact.h)
constexpr int64_t CHUNK_ALIGN = 256;   // chunk rows are a multiple of the GEMM macro tile

// A launch of one workgroup per 256 x 256 tile runs in rounds of as many tiles as the chip
// has CUs (one tile per CU at a time: a tile takes the whole LDS), dealt to the 8 XCDs in
// equal spans.  When the last round holds only r <= 16 tiles per XCD, half or more of the
// CUs would idle through it, so each of those tiles is cut into s = 32 / r K ranges instead
// (at most 8, each at least 16 K steps long): the round takes 1 / s of a tile's time plus a
// small reduction of fp32 partial blocks.  s = 1: the launch is left as it is.  `total` =
// tiles of the launch, ksteps = K steps (of 64) per tile; begin = position inside an XCD's
// span of its first tail tile.
constexpr int TAIL_XCDS = 8, TAIL_CUS_PER_XCD = 32;
constexpr size_t TAIL_BLOCK_BYTES = (size_t)256 * 256 * sizeof(float);
struct TailPlan {
    int begin, r, s;
};
inline TailPlan tail_plan(int64_t total, int64_t ksteps) {
    TailPlan t{0, 0, 1};
    const int64_t per_xcd = (total + TAIL_XCDS - 1) / TAIL_XCDS;
    const int r = (int)(per_xcd % TAIL_CUS_PER_XCD);
    if (per_xcd < TAIL_CUS_PER_XCD || r == 0 || r > TAIL_CUS_PER_XCD / 2) return t;
    int s = TAIL_CUS_PER_XCD / r;
    if (s > 8) s = 8;
    while (s > 1 && ksteps / s < 16) --s;
    if (s <= 1) return t;
    t.begin = (int)(per_xcd - r);
    t.r = r;
    t.s = s;
    return t;
}
// How a launch's tiles, numbered 0 .. total-1 in its tile order, are dealt to the 8 XCDs
// (workgroup id % 8 is the XCD, id / 8 the position in_xcd in that XCD's list of
// per_xcd = ceil(total / 8) = 32 F + r tiles): the 8 F full rounds of 32 consecutive numbers
// go round-robin (round j to XCD j % 8, so that at any time the XCDs work on 256 consecutive
// tiles), the numbers from 256 F on, at most r per XCD, are dealt in 8 runs of r: these are the
// tiles tail_plan cuts.  Numbers >= total (the last XCDs' lists can be short) mean "no tile".
FLCE_HD inline int xcd_tile_number(int xcd, int in_xcd, int per_xcd) {
    const int full = per_xcd / TAIL_CUS_PER_XCD * TAIL_CUS_PER_XCD;   // 32 F
    if (in_xcd < full)
        return ((in_xcd / TAIL_CUS_PER_XCD) * TAIL_XCDS + xcd) * TAIL_CUS_PER_XCD + in_xcd % TAIL_CUS_PER_XCD;
    return full * TAIL_XCDS + xcd * (per_xcd - full) + (in_xcd - full);
}
// K step that a K loop of `steps` steps takes as its kt-th when it starts at step rot < steps and wraps around.
FLCE_HD inline int rotated_step(int kt, int rot, int steps) {
    kt += rot;
    return kt - (kt >= steps ? steps : 0);
}
// bytes of partial blocks such a launch needs (0 when it is not cut)
inline size_t tail_partial_bytes(int64_t total, int64_t ksteps) {
    const TailPlan t = tail_plan(total, ksteps);
    return t.s > 1 ? (size_t)TAIL_XCDS * t.r * t.s * TAIL_BLOCK_BYTES : 0;
}

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
inline size_t elem_size(int dtype) { return dtype == 0 ? 4 : 2; }

struct Plan {
    int64_t C = 0;         // rows per chunk (last chunk may hold fewer)
    int64_t nchunks = 0;
    int64_t ldz = 0;       // row stride of the logits chunk, elements
    bool fp32_dw_acc = false;   // dW is accumulated in an fp32 scratch across chunks
    // which products run on the tuned bf16 kernel; the others run on the guarded one
    bool fast_logits = false, fast_dx = false, fast_dw_full = false, fast_dw_last = false;
    int dx_ranges = 1;     // K ranges of the dX product (K = V), > 1 when C x H has few tiles
    int dx_tile = 256;     // its tile size
    bool dx_dyn = false;   // several rounds of large tiles: fewer live rows may want fewer ranges
    // chunks are compacted, i.e. rows with an ignored target are left out of the products (see
    // compact.h)
    bool compact = false;
    // byte offsets into the workspace
    size_t off_hdr = 0, off_row_loss = 0, off_z = 0, off_dwacc = 0, off_dxpart = 0, off_xg = 0, off_dxg = 0,
           off_idx = 0, off_tv = 0, off_dyn = 0, off_tail = 0, total = 0;
    size_t tail_bytes = 0;     // room at off_tail
    size_t dxpart_bytes = 0;   // room at off_dxpart
};

// How many K ranges to cut a product with `tiles` output tiles and `ksteps` K steps
// into, so that tiles * ranges fills whole rounds of the chip's 256 CUs (one tile per
// CU at a time).  288 tiles, for example, run as two rounds at 56 % occupancy; cut
// into 8 ranges they are 9 full rounds.  Prefers few ranges (each costs an fp32
// partial result: a larger count must fill the rounds better by more than 2 % of the
// chip, and more than 8 are only taken while they fill a first round) and keeps ranges
// at least 64 K steps long; with many rounds the tail does not
// matter and the answer is 1.  Integer arithmetic only: the host and the device (which
// knows the live row count of a compacted chunk) must agree on the answer.
FLCE_HD inline int choose_ksplit(int64_t tiles, int64_t ksteps, int max_ranges) {
    constexpr int64_t CUS = 256, MIN_STEPS = 64;
    int best = 1;
    int64_t best_work = 0, best_rounded = 1;   // occupancy of the best choice = best_work / best_rounded
    for (int s = 1; s <= 16 && s <= max_ranges && ksteps / s >= MIN_STEPS; ++s) {
        const int64_t work = tiles * s;
        if (s > 8 && work > CUS) break;   // more than 8 ranges only to fill a first round
        const int64_t rounded = ((work + CUS - 1) / CUS) * CUS;
        // work / rounded > best_work / best_rounded + 1/50
        if (rounded > 0 && 50 * work * best_rounded > (50 * best_work + best_rounded) * rounded) {
            best_work = work;
            best_rounded = rounded;
            best = s;
        }
    }
    return best;
}

// The fp32 partial results of a cut dX product (ranges x rows x H) may take half as much
// memory as the logits chunk, not more.
inline int max_dx_ranges(size_t budget_bytes, int64_t rows, int64_t H) {
    const size_t one = (size_t)rows * (size_t)H * sizeof(float);
    const size_t n = one ? budget_bytes / 2 / one : 1;
    return (int)std::max<size_t>(1, std::min<size_t>(n, 64));
}

// ---- tile sizes and K ranges, by the time (ns) a launch takes ----
// Tiles run in rounds of 256 CUs.
//
// Tuned bf16 kernel, K steps of 64: a 256 x 256 tile takes 1.55 us per step plus 4 us, a 128 x 128
// tile 0.53 us per step in long loops (0.39 in short ones; a step's 16 MFMAs per wavefront alone take 0.3 on
// random data, its loads 0.24, its LDS reads 0.17, and they overlap in part) plus 0.65 us.  Measured (M x N x K,
// 256-tiles / 128-tiles, us):
//   1024 x 8192 x 512 (logits)  18.8 / 12.8      4096 x 32000 x 4096 (logits)  809 / 1104
//   2048 x 4096 x 1024 (logits) 31.9 / 21.6      2048 x 8192 x 1024 (logits)  34.9 / 37.6
//   8192 x 512 x 1024 (dW)      24.4 / 12.1      50257 x 1000 x 2047 (dW)      202 / 217
//   1024 x 512 x 8192 (dX)      67.1 (2 ranges) / 20.3, 14.8, 18.8 (4, 8, 16 ranges)
// so the small tiles serve outputs that do not fill a first round or two of large ones.
//
// Guarded kernel, fp32 (six times the matrix instructions), K in units of 16: a 256-tile takes 2.3
// us per unit plus 12 us (its 256 KB of output leave all CUs at once), 128-tiles 0.66 us (0.81 alone
// on a CU) plus 3, 64-tiles 0.21 us (0.31 alone, 0.46 for two) plus 1.  Measured (256 / 128 / 64, us):
//   4096 x 32000 x 4096  4640 / 5480 / -        2048 x 1024 x 50257  885 (8 ranges) / 1086 (4) / -
//   2048 x 8192 x 1024    163 / 180 / -         2048 x 4096 x 1024   124 / 93 / -
//   1024 x 4096 x 1024      - / 62 / 62         256 x 4096 x 512     - / - / 18.5
inline int64_t rounds_of_256(int64_t n) { return (n + 255) / 256; }
inline int64_t tiles_of(int64_t m, int64_t n, int64_t tile) { return ((m + tile - 1) / tile) * ((n + tile - 1) / tile); }
inline int64_t product_ns(bool tuned, int tile, int64_t tiles, int64_t k) {
    const int64_t n = rounds_of_256(tiles), steps = (k + 63) / 64, units = (k + 15) / 16;
    if (tuned) return tile == 256 ? n * (1550 * steps + 4000) : n * (530 * steps + 650);
    if (tile == 256) return n * (2300 * units + 12000) + 3000;
    if (tile == 128) return (n == 1 ? 810 : 660 * n) * units + 3000 * n + 6000;
    return (n == 1 ? 310 : n == 2 ? 460 : 210 * n) * units + 1000 * n + 6000;
}
// Cutting K costs a second launch and the fp32 partial results, written and read at about 8 TB/s.
inline int64_t cut_ns(int64_t tiles, int64_t tile, int64_t ranges) {
    return ranges > 1 ? 4000 + tiles * tile * tile * ranges / 1000 : 0;
}

// A dX product whose operands (G and W: (rows + H) V bf16) do not stay in the 256 MB memory-side cache is
// bound by how many loads the CUs have in flight: a step of a 128-tile takes 0.78 us alone on a CU (0.83
// at 24 rows, 0.79 at 512, 0.75 at 2048) and 0.62 to 0.75 beside another, of a 256-tile 1.7.  So one round of
// large tiles in up to 64 ranges, or two small tiles per CU, serve such products.  Measured (M x N x K, 128-tiles
// alone / two per CU / 256-tiles, ranges in parentheses, us):
//   24 x 4096 x 128256    208 (8) / 183 (16) / 181 (16)       200 x 832 x 128256    82 (18) / 66 (36) / 64 (64)
//   512 x 512 x 128256    100 (16) / 87 (32) / 74 (64)        1024 x 512 x 128256  197 (8) / 164 (16) / 117 (32)
//   2048 x 512 x 128256   377 (4) / 301 (8) / 219 (16)        512 x 2048 x 128256  376 (4) / 315 (8) / 217 (16)
// and where they do stay: 1024 x 512 x 32000 39.9 (8) / 37.6 (16) / 38.5 (32), 2048 x 2048 x 8192 73.5 (1) / 65 (2)
// / 61 (4).
constexpr int64_t DX_STREAM_BYTES = (int64_t)256 << 20;
inline bool dx_streams(int64_t rows, int64_t H, int64_t V) { return (rows + H) * V * 2 > DX_STREAM_BYTES; }
inline int64_t dx_streaming_ns(int tile, int64_t tiles, int64_t k) {
    const int64_t n = rounds_of_256(tiles), steps = (k + 63) / 64;
    return tile == 256 ? n * (1700 * steps + 4000) : n == 1 ? 780 * steps + 650 : n * (700 * steps + 650);
}

// The dX product of a chunk (rows x H output, K = V): tile size and K ranges.  The tuned kernel's
// large tiles keep at least 64 K steps per range (choose_ksplit; 16 where a streaming product fills one
// round), the others 512 elements (64-tiles 256).
struct ProductCut {
    int tile, ranges;
};
//
// bounded: the partial results may take no more memory than those of the large tiles cut to fill
// whole rounds (choose_ksplit, at most 16 ranges), which for many small products is none at all.
// part_bytes: room for the partial results.
inline ProductCut dx_cut(bool tuned, int64_t rows, int64_t H, int64_t V, size_t budget_bytes, bool bounded,
                         size_t part_bytes = SIZE_MAX) {
    int max_ranges = max_dx_ranges(budget_bytes, round_up(rows, 256), H);
    max_ranges = (int)std::min<size_t>((size_t)max_ranges, std::max<size_t>(1, part_bytes / ((size_t)rows * H * sizeof(float))));
    if (bounded) {
        const int tile = tuned ? 256 : 128;
        max_ranges = std::min(max_ranges, choose_ksplit(tiles_of(rows, H, tile), tuned ? (V + 63) / 64 : V / 4,
                                                        std::min(16, max_dx_ranges(budget_bytes, round_up(rows, tile), H))));
    }
    ProductCut best{0, 1};
    int64_t best_ns = 0;
    const bool streams = tuned && dx_streams(rows, H, V);
    auto consider = [&](int tile, int ranges) {
        const int64_t t = tiles_of(rows, H, tile), k = (V + ranges - 1) / ranges;
        const int64_t ns = (streams ? dx_streaming_ns(tile, t * ranges, k) : product_ns(tuned, tile, t * ranges, k)) +
                           cut_ns(t, tile, ranges);
        if (!best.tile || ns < best_ns) {
            best = {tile, ranges};
            best_ns = ns;
        }
    };
    if (tuned) consider(256, choose_ksplit(tiles_of(rows, H, 256), (V + 63) / 64, max_ranges));
    for (int r = 1; r <= max_ranges && (r == 1 || V / r >= 256); ++r) {
        if (!tuned) {
            if (r == 1 || V / r >= 512) consider(256, r);
            consider(64, r);
        }
        if (r == 1 || V / r >= 512) consider(128, r);
        if (streams && V / r >= 1024 && tiles_of(rows, H, 256) * r <= 256) consider(256, r);
    }
    return best;
}

// The logits and dW products have V along one output dimension, which can be shared out: columns (or
// rows) 0 .. main - 1 on 256 x 256 tiles that fill whole rounds of the CUs, the rest on smaller
// tiles in a second launch, instead of one more, mostly empty round of large ones.  tail: the last
// round of large tiles may be cut along K instead (tail_plan).  main = V: one launch.
struct VocabCut {
    int64_t main;
    int tile, rest_tile;
};
inline VocabCut vocab_cut(bool tuned, int64_t V, int64_t other, int64_t K, bool tail) {
    VocabCut best{V, 256, 0};
    const int64_t t256 = tiles_of(V, other, 256), steps = (K + 63) / 64;
    int64_t best_ns = product_ns(tuned, 256, t256, K);
    if (tail && tuned) {
        const TailPlan p = tail_plan(t256, steps);
        if (p.s > 1) best_ns += product_ns(true, 256, 1, K) / p.s + 5000 - product_ns(true, 256, 1, K);
    }
    const int64_t per = (other + 255) / 256, main = t256 / 256 * 256 / per * 256;   // whole rounds
    for (int small = 128; small >= (tuned ? 128 : 64); small /= 2) {
        const int64_t ns = product_ns(tuned, small, tiles_of(V, other, small), K);
        if (ns < best_ns) {
            best = {V, small, 0};
            best_ns = ns;
        }
        if (main <= 0 || main >= V) continue;
        const int64_t both = product_ns(tuned, 256, main / 256 * per, K) + 4000 +
                             product_ns(tuned, small, tiles_of(V - main, other, small), K);
        if (both < best_ns - best_ns / 32) {   // (3 %: the rows that turn out to have a target may be fewer)
            best = {main, 256, small};
            best_ns = both;
        }
    }
    return best;
}

// Whether the gradients of a batch that is one chunk are one launch (GradArgs).  The two products share the
// chip and, without K ranges, the launch that puts dX's rows in place goes as well; with K ranges a launch
// that adds them up follows, which otherwise runs beside dW's tiles, so that only the better fill is gained.
// places: the launch puts dX's rows in place (not behind an RMSNorm).
// Whole calls, us, two launches / one (workgroups of dX + dW), bf16 unless it says fp32,
// or how many times as fast one launch is:
// - dX uncut: 18 x 960 x 384 25.8 / 21.5, 1765 x 3584 x 2635 148 / 133, fp32 1871 x 1240 x 2653 277 / 261.
// - fp32 launches of at most 256 64-tiles have a variant with more loads in flight, which dW's long K loops want:
//   3639 x 16 x 489 (57 + 8) 114.7 / 110.3, 4474 x 128 x 101 (140 + 4) 125.7 / 128.9, 6723 x 80 x 91 175 / 184.
// - dX alone waits for its own stores to read them back: 19 x 1408 x 216 27.7 / 26.4, 44 x 368 x 110 19.8 / 19.1,
//   56 x 1024 x 400 23.9 / 23.4, 64 x 1024 x 400 23.7 / 24.4, 221 x 720 x 101 21.5 / 24.3, 360 x 16 x 98 19.6 / 18.3,
//   400 x 64 x 400 20.9 / 20.9, 400 x 64 x 800 22.0 / 22.5, 400 x 144 x 100 20.0 / 21.3,
//   1901 x 1024 x 433 32.7 / 31.1, 2600 x 1024 x 433 39.8 / 40.5, 1901 x 144 x 433 26.3 / 27.4, 958 x 2600 x 1702
//   58.4 / 60.3; fp32 5025 x 120 x 284 49.8 / 47.2.
// - dX in K ranges, from 128 rows on.  While all workgroups run at the same time: 532 x 64 x 2353 (20 + 19) 29.0 /
//   24.6, 1024 x 512 x 8192 (256 + 256) 57.2 / 53.6, 2000 x 640 x 5000 (240 + 200) 1.24 times as fast.  A few more
//   start a second round behind a dX that is planned for one tile per CU: 459 x 64 x 42658 (244 + 334) 65.8 / 70.6,
//   400 x 384 x 14000 (240 + 330) 0.88 times, 280 x 512 x 14000 (240 + 440) 0.92, 620 x 256 x 42000 (250 + 658) 0.965,
//   200 x 384 x 42000 (252 + 987) 0.95.  Wide or long enough, that round fills as well: 900 x 1152 x 9000 (216 +
//   639) 1.14, 900 x 512 x 9000 (256 + 284) 1.09, 2000 x 64 x 70000 (256 + 547) 1.11, 280 x 1152 x 60000 (243 +
//   4221) 1.08.
// - a dW of one or two K steps is bound by its writes, which hold up a dX that covers most CUs: 86 x 824 x 19859
//   (245 + 1092) 47.2 / 51.6, 16 x 320 x 52308 (189 + 1227) 45.1 / 50.4, 43 x 320 x 31475 (165 + 738) 38.3 / 41.6,
//   20 x 832 x 23116 behind an RMSNorm (231 + 1267) 54.1 / 56.2; but 2 x 1728 x 5253 (140 + 588) 39.9 / 37.7, 9 x
//   3264 x 11273 (234 + 2314) 72.1 / 69.7, 102 x 192 x 37246 (118 + 582) 40.3 / 37.2.  In one column of tiles: 16 x
//   48 x 34492 (60 + 270) 27.5 / 28.4, 21 x 64 x 56186 (63 + 439) 33.8 / 34.8, but 5 x 64 x 15903 (28 + 125) 24.1 /
//   23.4, 24 x 64 x 154137 (64 + 1205) 70.9 / 64.8.
// - fp32 with K ranges: 256 x 512 x 4096 (512 + 512 64-tiles) 53.1 / 51.6, 604 x 2112 x 14422 (128-tiles) 721 / 701,
//   54 x 384 x 11328 (252 + 1062 64-tiles) 45.1 / 47.6.
inline bool grads_in_one(const Plan& p, const VocabCut& dw, bool bf16, bool want_dw, bool dw_fast, bool places, int64_t rows,
                         int64_t H, int64_t V) {
    if (p.nchunks != 1 || p.dx_tile == 256 || p.fast_dx != bf16 || H % 4 != 0) return false;
    if (want_dw && (dw_fast != bf16 || dw.main != V || dw.tile != p.dx_tile)) return false;
    const int64_t of_dx = tiles_of(rows, H, p.dx_tile) * p.dx_ranges;
    const int64_t all = of_dx + (want_dw ? tiles_of(V, H, p.dx_tile) : 0);
    if (!want_dw) {
        const bool gains = rows <= 56 || (V <= 512 && (H <= 128 || (rows > 1300 && H % 128 == 0 && all <= 128)));
        return p.dx_ranges == 1 && all <= 256 && (!bf16 || !places || gains);
    }
    if (p.dx_tile == 64 && all <= 256 && rows > 4096) return false;
    if (p.dx_ranges == 1) return all <= 2048;
    if (!bf16) return all <= (p.dx_tile == 64 ? 1024 : 4096);
    if (rows >= 128) {
        if (all <= 512 || (of_dx < 200 && H < 512)) return all <= 8192;
        if (H >= 512) return all <= 8192 && (all > 700 || rows >= 800);
        return all <= 8192 && rows > (all <= 950 ? 1800 : H < 128 ? 700 : 200) && (all > 660 || H > 128);
    }
    return all <= (rows <= 64 ? 2048 : 8192) && !(H <= 1024 && of_dx >= 160 && all > 600) &&
           !(rows <= 64 && H <= 128 && all > 256 && all < 600);
}

// Limits of the tuned kernel's 32-bit offsets inside one tile (see gemm_bf16_nt.h).
inline bool fits_row_form(int64_t ld, int64_t) { return 256 * ld * 2 + 128 < ((int64_t)1 << 30); }
inline bool fits_col_form(int64_t ld, int64_t) { return 64 * ld * 2 + 512 < ((int64_t)1 << 30); }

// How much workspace a plan may take, the fastest plan first:
//   full     up to 64 K ranges of dX on small tiles (dx_cut); what the automatic chunk rule takes
//   bounded  partial results as under dx_cut's bound: what an explicit logits budget takes, whose
//            caller limits memory, and calls whose buffer is too small for `full`
//   least    bounded, and without the index maps of the row compaction (12 bytes per row) where the
//            problem is a bf16 one with H % 64 != 0, for buffers that were sized without them
enum class Room { full, bounded, least };

// Byte offsets of the workspace for a plan whose chunking (C, nchunks, rows of the last
// chunk) is decided; `dxpart_floor` is a lower bound for the K-range partials.
inline void lay_out(Plan& p, int64_t H, int64_t V, int dtype, int64_t rows_last, size_t budget_bytes,
                    bool allow_compact, size_t dxpart_floor, Room room, size_t part_bytes = SIZE_MAX) {
    const size_t es = elem_size(dtype);
    p.fp32_dw_acc = (dtype != 0) && p.nchunks > 1;
    p.fast_logits = p.fast_dx = p.fast_dw_full = p.fast_dw_last = false;
    if (dtype != 0) {
        const bool out_ok = 256 * H * 4 < ((int64_t)1 << 31);
        p.fast_logits = (H % 8 == 0) && fits_row_form(H, H) && 256 * p.ldz * 2 < ((int64_t)1 << 31);
        // K of the dX product is V: the dlogits rows are padded with zeros to ldz, W is read
        // K-major; K of the dW product is the chunk's row count, both operands K-major: any
        // V and any row count do
        p.fast_dx = (H % 8 == 0) && fits_row_form(p.ldz, V) && fits_col_form(H, V) && out_ok;
        auto dw_ok = [&](int64_t rows) {
            return (H % 8 == 0) && fits_col_form(p.ldz, rows) && fits_col_form(H, rows) && out_ok;
        };
        p.fast_dw_full = (p.nchunks > 1) ? dw_ok(p.C) : dw_ok(rows_last);
        p.fast_dw_last = dw_ok(rows_last);
    }
    {
        const int64_t rows = p.nchunks > 1 ? p.C : rows_last;
        const ProductCut cut = dx_cut(p.fast_dx, rows, H, V, budget_bytes, room != Room::full, part_bytes / p.C * rows);
        p.dx_tile = cut.tile;
        p.dx_ranges = cut.ranges;
        p.dx_dyn = p.fast_dx && cut.tile == 256 && tiles_of(rows, H, 256) * cut.ranges > 256;
    }
    // (the copies move 16-byte vectors; bf16 rows of other lengths do not run on the tuned kernel)
    p.compact = allow_compact && !(room == Room::least && dtype != 0 && H % 64 != 0) &&
                (dtype == 0 ? H % 4 == 0 : p.fast_logits && p.fast_dx && p.fast_dw_full && p.fast_dw_last);

    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += (bytes + 255) / 256 * 256;
        return at;
    };
    p.off_hdr = take(256);
    // per-row values in one piece: losses, the compaction's targets and batch rows, its device words
    const size_t maps = p.compact ? (size_t)p.C : 0;
    p.off_row_loss = take((size_t)round_up(p.C, 2) * sizeof(float) + maps * (sizeof(int64_t) + sizeof(int32_t)) +
                          DYN_WORDS * sizeof(int32_t));
    p.off_tv = p.off_row_loss + (size_t)round_up(p.C, 2) * sizeof(float);
    p.off_idx = p.off_tv + maps * sizeof(int64_t);
    p.off_dyn = p.off_idx + maps * sizeof(int32_t);
    p.off_z = take((size_t)p.C * p.ldz * es);
    p.off_dwacc = take(p.fp32_dw_acc ? (size_t)V * H * sizeof(float) : 0);
    const size_t dxpart = p.dx_ranges > 1 ? (size_t)p.dx_ranges * p.C * H * sizeof(float) : 0;
    p.dxpart_bytes = std::max(dxpart, dxpart_floor);
    p.off_dxpart = take(p.dxpart_bytes);
    // a chunk of gathered input rows and of their gradient (also the normalised rows and
    // their gradient when an RMSNorm runs in front)
    p.off_xg = take((size_t)p.C * H * es);
    p.off_dxg = take((size_t)p.C * H * es);
    // fp32 partial blocks of the dW product's last, partly filled round of tiles when it is cut
    // along K (tail_plan; a shorter last chunk has fewer K steps and never needs more)
    const int64_t dw_tiles = ((V + 255) / 256) * ((H + 255) / 256);
    p.tail_bytes = (p.fast_dw_full && p.fast_dw_last) ? tail_partial_bytes(dw_tiles, (p.C + 63) / 64) : 0;
    p.off_tail = take(p.tail_bytes);
    p.total = off;
}

// budget_bytes bounds one chunk of logits.  A batch whose WHOLE logits fit in
// single_bytes (>= budget_bytes) runs as one chunk whatever the budget says: the
// automatic rule passes the chunk budget plus the size of the fp32 dW partial sums,
// which only several chunks need, so that one chunk is taken whenever it needs no more
// memory than the chunked plan would (and it is always faster: no second pass over W,
// no fp32 round trip of dW).  worst_case_bt: the plan with the largest workspace any BT
// can lead to (BT is ignored).
inline Plan make_plan(int64_t BT, int64_t H, int64_t V, int dtype, size_t budget_bytes,
                      bool worst_case_bt = false, bool allow_compact = true, size_t single_bytes = 0,
                      Room room = Room::full, size_t part_bytes = SIZE_MAX) {
    Plan p;
    const size_t es = elem_size(dtype);
    p.ldz = round_up(V, 64);
    const size_t row_bytes = (size_t)p.ldz * es;
    int64_t cmax = (int64_t)(budget_bytes / row_bytes);
    cmax = cmax / CHUNK_ALIGN * CHUNK_ALIGN;
    if (cmax < CHUNK_ALIGN) cmax = CHUNK_ALIGN;
    const int64_t single_max = std::max<int64_t>(cmax, (int64_t)(single_bytes / row_bytes));   // rows
    if (worst_case_bt) {
        // the bound has to hold for every chunk size the scheduler can pick: the number of
        // K ranges of the dX product depends on the row count through its tile count
        auto dxpart_over = [&](bool tuned, int64_t upto) {
            size_t m = 0;
            if (V < 512) return m;   // never cut
            for (int64_t c = 64; c <= upto && max_dx_ranges(budget_bytes, round_up(c, 256), H) > 1; c += 64) {
                const int ks = dx_cut(tuned, c, H, V, budget_bytes, room != Room::full).ranges;
                if (ks > 1) m = std::max(m, (size_t)ks * c * H * sizeof(float));
            }
            return m;
        };
        // several chunks, the last one ragged (the most expensive case) ...
        p.C = cmax;
        p.nchunks = 2;
        lay_out(p, H, V, dtype, 1, budget_bytes, allow_compact, 0, room);
        lay_out(p, H, V, dtype, 1, budget_bytes, allow_compact, dxpart_over(p.fast_dx, cmax), room);
        // ... or the largest batch that still runs as one chunk
        Plan q;
        q.ldz = p.ldz;
        q.C = single_max;
        q.nchunks = 1;
        lay_out(q, H, V, dtype, single_max, budget_bytes, allow_compact, 0, room);
        lay_out(q, H, V, dtype, single_max, budget_bytes, allow_compact, dxpart_over(q.fast_dx, single_max), room);
        return q.total > p.total ? q : p;
    }
    int64_t rows_last;
    if (BT <= single_max) {
        p.C = BT;
        p.nchunks = 1;
        rows_last = BT;
    } else {
        p.nchunks = (BT + cmax - 1) / cmax;
        p.C = round_up((BT + p.nchunks - 1) / p.nchunks, CHUNK_ALIGN);   // even out the chunks
        p.nchunks = (BT + p.C - 1) / p.C;
        rows_last = BT - (p.nchunks - 1) * p.C;
    }
    lay_out(p, H, V, dtype, rows_last, budget_bytes, allow_compact, 0, room, part_bytes);
    return p;
}

// Paper's rule: chunk = 2^ceil(log2(ceil(BT / ceil(V / H)))).
inline int64_t paper_chunk_rows(int64_t BT, int64_t H, int64_t V) {
    const int64_t inc = (V + H - 1) / H;
    const int64_t c = (BT + inc - 1) / inc;
    int64_t p2 = 1;
    while (p2 < c) p2 <<= 1;
    return p2;
}

}  // namespace flce
