// How the rows of an expert are cut into tiles by the bf16 expert FFN kernels (host code; no GPU header is needed to compile it).
#pragma once
#include <math.h>

#include "moe355.h"

namespace moe {

// Most rows of one expert segment covered by one block of the large FFN kernels.
constexpr int kTileM = 320;
constexpr int kEvenTileM = 288;         // most rows of one where the experts have more than two
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

// Highest row tile of the up-projection.  A tile of 17 or 18 blocks of 16 rows costs less than two of 9, which read the weights twice and need 1.5
// times the bytes per product, and experts that all have as many tiles keep the rounds of the compute units even; so what matters is where the limit lies
// against the mean and its spread.  Layer us by limit (d 4096, f 10240; tokens / experts):
//            2048/8  2300/8  4096/8  4500/8  6000/8  4300/16  8192/32  9000/32  16384/32  20000/64  28000/32  65536/32
//   160         552     591     978    1004    1385     1096     2133     2197      3665      5116      6056     13055
//   224         549     593     977    1037    1201     1089     2143     2194      3558      4644      5541     12561
//   256         540     590     952    1035    1270     1156     2086     2268      3441      4643      5347     12486
//   288         521     604     850    1006    1272      953     1932     2085      3440      4668      5361     12155
//   320         519     568     844     920    1272      949     1862     1975      3339      4440      5540     12145
// Hence 320 up to two such tiles per expert, and beyond as many rows as give nearly all experts the same number of tiles of at most 288 rows: tiles of 19
// and 20 blocks, with two steps of loads ahead instead of three, gain nothing where the matrix pipes are the bound.
// With fewer items than compute units the tiles are cut as low as leaves no more items than those (1100 tokens on 4 experts, d 1024, f 4096 320 /
// 160 rows 101.9 / 93.5 us; 4000 on 8, d 512, f 1024 66 / 59; whole experts / cut, 400 on 4, d 512, f 1024 36.2 / 26.4, 820 on 4, d 1024, f 1024 64.5 / 50.4, 700 on
// 4, d 768, f 3072 72.2 / 59.4, 1500 on 12, d 320, f 640 39.1 / 33.6, 300 on 4, d 1024, f 2048 53.9 / 47.9, but 1200 on 16, d 1024, f 512 49.8 / 53.0); and where the experts have several tiles, one more each if the items then take their rounds
// in less time, by their blocks and 4 for what an item costs beside them (3000 tokens on 4 experts, d 2048, f 6144 285 -> 257; 6000 on 8 as above).
inline int ffn_tile_rows(const moe_cfg& c, bool gather, int n_cu, int e_count, long max_rows) {
    if (few_rows(c, n_cu)) return kFewTileM;
    const long mean_rows = max_rows / (e_count > 0 ? e_count : 1), columns = static_cast<long>(e_count) * ((c.f / 32 + 3) / 4);
    const double most = mean_rows + 2.5 * sqrt(static_cast<double>(mean_rows));       // rows of nearly all experts, if the loads are even
    auto rows_for = [&](long n) { return (static_cast<long>(most / n) + 16) / 16 * 16; };
    // (the kernel that gathers has code for tiles up to its own limit: nothing below may go over it)
    const long even = gather ? kGatherTileM : kEvenTileM;
    long limit = gather ? kGatherTileM : kTileM, tiles = (mean_rows + limit - 1) / limit;
    if (tiles > 2) {
        tiles = static_cast<long>(most / even) + 1;
        limit = rows_for(tiles);
    }
    if (columns * tiles < n_cu) {
        long n = n_cu / columns;
        // (tiles of fewer than 48 rows, whose steps take as long as theirs, only where the down-projection needs them as well)
        const bool low = 8L * e_count * ((c.d / 32 + 3) / 4) <= 3L * n_cu;
        while (n > 1 && (rows_for(n) < kMinTileM || (!low && mean_rows < 48 * n))) --n;
        const long rows = rows_for(n) < kMinTileM ? kMinTileM : rows_for(n);
        return static_cast<int>(rows < limit ? rows : limit);
    }
    auto cost = [&](long n) { return (columns * n + n_cu - 1) / n_cu * (4 + ((mean_rows + n - 1) / n + 15) / 16); };
    if (tiles > 1 && cost(tiles + 1) <= cost(tiles)) limit = rows_for(tiles + 1) < limit ? rows_for(tiles + 1) : limit;
    return static_cast<int>(limit);
}

// Height of the down-projection's row tiles.  Its work items are (row tile x 256 output columns): with few experts of
// a tile or so each there are fewer items than compute units (8 experts of about 256 rows: 8 to 16 tiles x 16 column
// groups for 256 compute units, and a tile takes as long as its 160 reduction steps whether others run or not).  The
// tiles are then cut lower, so that every expert gives as many tiles as fill the chip (with a quarter of headroom for
// experts above the mean); measured on that layer: 0.235 -> 0.184 ms.  Lower tiles for the up-projection, which has
// five times the column groups, only cost (0.327 -> 0.354 ms), so the two kernels have a tile list each.
inline int ffn_down_tile_rows(const moe_cfg& c, int e_count, long max_rows, int tile_m_up, int n_cu) {
    const long mean_rows = max_rows / (e_count > 0 ? e_count : 1);
    const int col_groups = (c.d / 64 + 3) / 4;
    if (mean_rows <= 224 || static_cast<long>(e_count) * col_groups >= n_cu) return tile_m_up;
    const long per_expert = (n_cu + static_cast<long>(e_count) * col_groups - 1) / (static_cast<long>(e_count) * col_groups);
    long tm = ((mean_rows * 5 / 4 + per_expert - 1) / per_expert + 31) / 32 * 32;
    tm = tm < kMinTileM ? kMinTileM : tm;
    return tm < tile_m_up ? static_cast<int>(tm) : tile_m_up;
}

}  // namespace moe
