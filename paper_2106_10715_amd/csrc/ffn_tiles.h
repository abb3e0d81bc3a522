// How the rows of an expert are cut into tiles by the bf16 expert FFN kernels (host code; no GPU header is needed to compile it).
#pragma once
#include <math.h>

#include "moe355.h"

namespace moe {

// Most rows of one expert segment covered by one block of the large FFN kernels.
constexpr int kTileM = 320;
// Rows of a tile when the up-projection gathers its rows itself: a thread then holds one source offset per
// 32-row block, which the registers allow up to seven blocks (eight accumulator blocks leave no room).
constexpr int kGatherTileM = 224;
// Rows of a tile of the kernels for few rows: with more on one expert, its tiles run side by side.
constexpr int kFewTileM = 64;
constexpr int kMinTileM = 64;           // lowest row tile a launch is ever cut into
static_assert(kFewTileM >= kMinTileM, "the work list has room for the tiles");

// Whether a layer's experts run on the kernels for few rows (ffn_few.h; the same bits either way).  The large kernel needs work
// items (an expert's tile x 256 columns in the down-projection) for the compute units; the fewer it has, the more rows per
// expert the other one may be given.
// Large kernel / few rows, layer us, d 4096 f 10240: 32 experts 40 rows in all 904 / 871, 64 rows 1029 / 1032, 128 rows
// 1195 / 1196, 256 rows 1197 / 1216; 64 experts 128 rows 1979 / 1962; 16 experts 64 rows 636 / 634, 128 rows 640 / 641,
// 192 rows 621 / 633; 8 experts 64 rows 334 / 320, 128 rows 337 / 334, 192 rows 341 / 364; 4 experts 128 rows 242 / 238,
// 192 rows 243 / 295.  Smaller layers: d 1024 f 2048 8 experts 256 rows 54 / 47, 512 rows 63 / 78; d 512 f 1024 33 experts
// 1056 rows 55 / 54, 1500 rows 54 / 58; d 768 f 3072 33 experts 256 rows 119 / 113, 500 rows 121 / 120, 1056 rows 133 / 145;
// d 2048 f 4096 16 experts 128 rows 155 / 143, 400 rows 162 / 181.  All rows on one of the experts (the FFN alone): 64 rows of
// 32 experts 180 / 110, 128 rows of 16 185 / 150, 128 rows of 64 212 / 149; d 1024 f 2048 256 rows of 8 64 / 27; d 512 f 1024
// 1056 rows of 33 38 / 31.
inline bool few_rows(const moe_cfg& c, int n_cu) {
    const long rows = static_cast<long>(c.T) * c.k, items = static_cast<long>(c.E) * ((c.d / 64 + 3) / 4);
    return rows <= (3 * items < n_cu ? 32L : items <= n_cu ? 8L : 2L) * c.E;
}

// How a launch of the large kernels over e_count experts with max_rows rows in all is cut.
struct FfnTiles {
    int up, down;       // most rows of a tile of the two projections (a work list each, unless equal)
    bool narrow;        // units of 32 columns in the down-projection instead of 64
};

// Blocks of 16 rows of the experts of a launch, as far as they are known before the loads are: an eighth of the experts each and the largest one, if the loads are
// less, or more, uneven than those of a random gate, whose columns differ in length by 1 / sqrt(2 d).
constexpr int kShares = 9;
struct ExpertBlocks {
    int blocks[2][kShares], most = 1;
    double experts[kShares];
    ExpertBlocks(double mean, int e_count, int d) {
        const double log_e = log(static_cast<double>(e_count)), skew = 0.9 * mean * log_e;
        const double spread = e_count > 1 ? sqrt(mean + skew * skew / d) : 0;          // (the rows of a single expert are known)
        // of the normal distribution, at the middle of every share and of the last of e_count
        const double at[kShares] = {-1.534, -0.887, -0.489, -0.157, 0.157, 0.489, 0.887, 1.534, 1.48 * sqrt(log_e) - 0.6};
        for (int i = 0; i < kShares; ++i) {
            experts[i] = i < 8 ? (e_count - 1) / 8.0 : 1;
            for (int s = 0; s < 2; ++s) {
                const double rows = mean + (s == 0 ? 0.6 : 1.4) * spread * at[i];
                blocks[s][i] = rows < 1 ? 1 : static_cast<int>((static_cast<long>(rows) + 15) / 16);
                if (blocks[s][i] > most) most = blocks[s][i];
            }
        }
    }
};

// A product's work items are its row tiles by its `columns` groups of four column units.  This is the time of all of them on n_cu compute units, in that of a
// block of 16 rows: an item takes its blocks and per_item of the reduction (above 18, with two steps of loads ahead instead of three, half a block more, and 19 as
// much as 20, which are staged alike: 65536 tokens on 32 experts of 10240, tiles of 272, 288, 304 and 320 rows 12.39, 12.30, 12.53 and 12.49 ms, but 50000
// 9.91, 9.90, 9.78 and 9.64), and the whole lies half-way between every round as long as its longest item and all items spread evenly (a round that is not full
// is faster, and short items make up for long ones).
inline double per_item(int reduction, bool narrow) { return 4 + 960.0 / reduction + (narrow ? 4 : 0); }      // (narrow units: bound by their weights)
inline double ffn_cost(const ExpertBlocks& of, int columns, double item, int tile_rows, int n_cu) {
    const int most = tile_rows / 16;
    double total = 0;
    for (int s = 0; s < 2; ++s) {
        double of_height[kTileM / 16 + 1] = {};
        auto add = [&](int b, double n) { of_height[b < 4 ? 4 : b] += n; };             // (the steps of lower tiles take as long)
        for (int i = 0; i < kShares; ++i) {
            const int n = of.blocks[s][i];
            if (n <= most) {
                add(n, of.experts[i]);
                continue;
            }
            const int tiles = (n + most - 1) / most, each = n / tiles, more = n - each * tiles;
            add(each, (tiles - more) * of.experts[i]);
            if (more > 0) add(each + 1, more * of.experts[i]);
        }
        double items = 0;
        int begun = 0;
        for (int b = most; b >= 4; --b) {
            if (of_height[b] == 0) continue;
            const double here = of_height[b] * columns;
            items += here;
            const int rounds = items > 0.5 ? static_cast<int>((items - 0.5) / n_cu) + 1 : 0;        // (a fraction of an item begins none)
            total += (rounds - begun + here / n_cu) * (item + b + (b == 19 ? 1 : b == 20 ? 0.5 : 0));
            begun = rounds;
        }
    }
    return total;
}

// The height of a product's tiles: `before` (256 rows, 224 where the up-projection gathers, lower ones for a down-projection of few items; see ffn_tiles), unless a
// multiple of 32 rows is better by 4 % of a round and 1 % of the whole (2 % beyond 16 rounds).  What matters is how the items divide into rounds of the compute units, how often the weights
// are read and how long the steps of low tiles are: a tile of 17 or 18 blocks costs less than two of 9, and small layers need low tiles to have an item for
// every unit.  Time against that with `before`, layers of one gate each, every height of each product timed, d 64 to 4096, f 192 to 10240, 4 to 64 experts, up to
// 32768 tokens: 0.959 in the mean of 3083 with random gates, 137 of them more than 2 % slower and 52 more than 5 % (the loads are not known; the best height of each would take 0.940),
// 0.976, 111 and 36 of 2286 with Zipf loads, exponents of 0.4 to 1.2.  (Low tiles wherever items leave units idle, else 320 rows up to two tiles and even ones of 288 beyond: 0.979, 312 and 134,
// 0.991, 235 and 101.)  Layer us by limit, d 4096, f 10240 (tokens / experts):
//            2048/8  2300/8  4096/8  4500/8  6000/8  4300/16  8192/32  9000/32  16384/32  20000/64  28000/32  65536/32
//   160         552     591     978    1004    1385     1096     2133     2197      3665      5116      6056     13055
//   224         549     593     977    1037    1201     1089     2143     2194      3558      4644      5541     12561
//   256         540     590     952    1035    1270     1156     2086     2268      3441      4643      5347     12486
//   288         521     604     850    1006    1272      953     1932     2085      3440      4668      5361     12155
//   320         519     568     844     920    1272      949     1862     1975      3339      4440      5540     12145
inline int ffn_tile_rows(const ExpertBlocks& of, double rounds, int columns, double item, int before, int most, int n_cu) {
    int best = before;
    double least = ffn_cost(of, columns, item, before, n_cu) * (rounds > 16 ? 0.98 : rounds > 4 ? 0.99 : rounds > 1 ? 1 - 0.04 / rounds : 0.96);
    for (int rows = most / 32 * 32; rows >= kMinTileM; rows -= 32) {
        if (rows - 32 >= 16 * of.most) continue;           // (the next one has the same tiles)
        const double cost = ffn_cost(of, columns, item, rows, n_cu);
        if (cost < least) {
            least = cost;
            best = rows;
        }
    }
    // With items for less than 0.8 of the units an expert of more rows than expected would leave the others idle: as low as leaves the expected tiles whole (466 tokens on 12 experts, d 1024,
    // f 320, loads by a Zipf law with an exponent of 1.2, the largest 196 rows: tiles of 224 rows 48 us, of 64 40).
    const int whole = (of.most + 1) / 2 * 32;
    if (rounds <= 0.8 && whole < best) best = whole < kMinTileM ? kMinTileM : whole;
    return best;
}

inline FfnTiles ffn_tiles(const moe_cfg& c, bool gather, int n_cu, int e_count, long max_rows) {
    if (few_rows(c, n_cu)) return {kFewTileM, kFewTileM, false};
    const long mean_rows = max_rows / e_count;
    const double mean = static_cast<double>(max_rows) / e_count, tiles = e_count * (mean > 256 ? mean / 256 : 1);
    const ExpertBlocks of(mean, e_count, c.d);
    FfnTiles t;
    // (nothing may go over what the kernel has code for: the one that gathers has less)
    const int up_columns = (c.f / 32 + 3) / 4, wide = (c.d / 64 + 3) / 4;
    const double up_rounds = tiles * up_columns / n_cu;
    // In long launches on experts of many rows it also matters that neighbours in the list belong to one expert (groups of four share its weights): where all of 32
    // experts have four tiles 28000 tokens take 5391-5406 us, where some have three up to 5678. As many rows, then, as give nearly all experts the same number
    // of tiles of at most 288 (65536 tokens, eight tiles of up to 272 rows against seven and eight of 288 12.00 / 12.06 ms, of four gates).
    long before = gather ? kGatherTileM : 256, even = 0;
    if (!gather && mean > 2 * kTileM && up_rounds > 16) {
        const double most = mean + 2.5 * sqrt(mean);
        before = even = static_cast<long>(most / (static_cast<long>(most / 288) + 1) + 16) / 16 * 16;
    }
    t.up = ffn_tile_rows(of, up_rounds, up_columns, per_item(c.d, false), static_cast<int>(before), gather ? kGatherTileM : kTileM, n_cu);
    // Narrow units while the experts are likely to have a single tile each, mean rows up to 224, and their items are
    // bound by the weight stream: on 256-row tiles, and once experts spill into second tiles, the narrow unit's
    // second LDS read per MFMA costs more than the idle compute units do; measured on 8 experts: 128 rows per
    // expert 0.148 ms narrow against 0.177 ms wide, 256 rows 0.274 against 0.239.
    const long tiles_hint = (max_rows + t.up - 1) / t.up > e_count ? (max_rows + t.up - 1) / t.up : e_count;
    t.narrow = tiles_hint * wide < 2 * 256 && mean_rows <= 224;
    // Wide units: with few experts of a tile or so each there are fewer items than compute units (8 experts of about 256 rows: 8 to 16 tiles x 16 column
    // groups for 256 compute units, and a tile takes as long as its 160 reduction steps whether others run or not).  The
    // tiles are then cut lower, so that every expert gives as many tiles as fill the chip (with a quarter of headroom for
    // experts above the mean); measured on that layer: 0.235 -> 0.184 ms.
    if (mean_rows > 224 && static_cast<long>(e_count) * wide < n_cu) {
        const long per_expert = (n_cu + static_cast<long>(e_count) * wide - 1) / (static_cast<long>(e_count) * wide);
        const long fill = ((mean_rows * 5 / 4 + per_expert - 1) / per_expert + 31) / 32 * 32;
        before = fill < kMinTileM ? kMinTileM : fill < before ? fill : before;
    }
    const int columns = t.narrow ? (c.d / 32 + 3) / 4 : wide;
    const double item = per_item(c.f, t.narrow);
    t.down = ffn_tile_rows(of, tiles * columns / n_cu, columns, item, static_cast<int>(before), kTileM, n_cu);
    // (nor a list of its own for 2 %: it costs 0.3 to 1.5 us, and the even tiles of long launches are the better ones for both products)
    if (t.up == even && tiles * columns / n_cu > 8) t.down = t.up;
    else if (t.down != t.up && ffn_cost(of, columns, item, t.up, n_cu) <= 1.02 * ffn_cost(of, columns, item, t.down, n_cu)) t.down = t.up;
    return t;
}

}  // namespace moe
