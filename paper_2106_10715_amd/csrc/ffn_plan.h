// Work list of one launch of the expert FFN kernels: which (expert, rows) every row tile covers, in the
// order the tiles are handed out.  An expert's rows are split evenly over its tiles (in multiples of 16 rows), not into full
// tiles and a small remainder.  Also clears the work counters of the two kernels that follow.
// The two kernels of a launch have a list each when their row tiles differ in height (else both read the first):
//   plan[0..7], plan[8..15] : next work item of each of the 8 queues, up and down kernel
//   plan[16], plan[17]      : number of tiles of the up and of the down kernel's list
//   plan[32 + 4 s ..]       : up kernel's tile s = (expert, first row, rows, row tiles of this expert)
//   plan[32 + 4 max_tiles + 4 s ..] : the same for the down kernel
#pragma once
#include "common.h"

namespace moe {

constexpr int kPlanHeader = 32;
constexpr int kPlanScratch = 7;           // arrays of 256 numbers in LDS, the first at a 16-byte boundary

// Where the sum of an output column over the reduction dimension starts (step key % steps of 64; it wraps around).  It depends
// on the expert and on the column's chunk only (1024 columns of the up-projection, 2048 of the down-projection), never on the
// launch or on the kernel that computes the column, so that every kernel gives the same bits.
__device__ inline unsigned sweep_key(int e, unsigned chunk) { return static_cast<unsigned>(e) * 37u + chunk; }

// By one block of at least 256 threads (all of them must call; the first 256 work): offsets[e_first ..
// e_first + e_count] -> list `list` (0: up kernel, 1: down kernel) of the plan, in tiles of at most tile_m rows.
// `scratch` is LDS of the caller.  e_count <= 256.  The call for list 0 also clears the work counters.
__device__ inline void ffn_plan_block(const int32_t* offsets, int e_first, int e_count, int tile_m, int32_t* plan,
                                      int total_rows, int max_tiles, int (&scratch)[kPlanScratch][256], int list) {
    int (&n)[256] = scratch[0], (&first)[256] = scratch[1], (&order)[256] = scratch[2], (&tl)[256] = scratch[3];
    const int t = threadIdx.x;
    const bool worker = t < 256;
    int cnt = 0, lo = 0;
    if (worker && t < e_count) {
        // whatever the offsets hold, no tile may reach outside the total_rows rows or the work list
        lo = min(max(offsets[e_first + t], 0), total_rows);
        cnt = min(max(offsets[e_first + t + 1], lo), total_rows) - lo;
    }
    // The highest tiles first among those of either kind below, so that the last items are the short ones; among equals the expert with more
    // rows, then by index.
    // (By rows alone, with tiles of up to 256 rows: 2048 tokens on 8 experts, whose tiles were 16 blocks high up to 256 rows and 8 or 9 above, ended with the 16;
    // 65536 tokens on 32 experts 12424 -> 12334 us.)
    constexpr int kRowBits = 26;               // rows < 2^31 / 64
    static_assert(kTileM / 16 < 1 << (31 - kRowBits), "a height and the rows below it fit the key");
    int key = 0;
    if (cnt > 0) {
        const int tiles = (cnt + tile_m - 1) / tile_m;
        key = ((cnt + 15) / 16 + tiles - 1) / tiles << kRowBits | cnt;
    }
    if (worker) {
        n[t] = key;
        first[t] = lo;
        order[t] = t;
        tl[t] = 0;
    }
    __syncthreads();
    if (worker && t < e_count) {
        int rank = 0;                   // a permutation of 0..e_count-1 (keys past the last are 0 and count for nobody)
#pragma unroll 1
        for (int u = 0; u < e_count; u += 4) {
            const int4 v = *reinterpret_cast<const int4*>(&n[u]);
            rank += (v.x > key || (v.x == key && u < t)) + (v.y > key || (v.y == key && u + 1 < t)) + (v.z > key || (v.z == key && u + 2 < t)) +
                    (v.w > key || (v.w == key && u + 3 < t));
        }
        order[rank] = t;
    }
    __syncthreads();
    const int mine = worker ? order[t] : 0, my_n = worker && t < e_count ? n[mine] & ((1 << kRowBits) - 1) : 0;
    const int my_tiles = (my_n + tile_m - 1) / tile_m;
    if (worker) tl[t] = my_tiles;
    int4* tiles = reinterpret_cast<int4*>(plan + kPlanHeader + 4 * list * max_tiles);
    // tile mt of an expert with n_e rows and n_tiles tiles, its blocks of 16 rows spread evenly (the first tiles have one more where they do not
    // divide), at place `at` of the list.  No product is larger than the number of blocks.
    auto put = [&](int e, int n_e, int n_tiles, int mt, int at) {
        const int blocks = (n_e + 15) / 16, each = blocks / n_tiles, more = blocks - each * n_tiles;
        const int lo = (mt * each + min(mt, more)) * 16, hi = min(lo + (each + (mt < more ? 1 : 0)) * 16, n_e);
        if (at < max_tiles) tiles[at] = make_int4(e_first + e, first[e] + lo, hi - lo, n_tiles);
    };
    // Experts with several tiles, bound by the matrix pipes, and those with one, bound by reading their weights, take turns over the whole list,
    // so that neither resource idles while the other is the bound: groups of four tiles of the first kind (neighbours in the list share weights in
    // one L2) among groups of four of the rest, evenly.  Whole layers, sorted -> merged: 16384 tokens x 2 skewed over 64 experts 7067 -> 6992 us,
    // 16000 x 1 on 64 4086 -> 3867, 8192 x 1 on 32 2123 -> 2074, 2048 on 8 567 -> 565, 65536 on 32 equal.  Small layers of few rows per expert, where
    // hardly any has several tiles, only pay for the longer code (1025 x 2 on 33, d 320 47.2 -> 48.5 us): hence the limits.
    // The list is bound by the latency of its steps and by the fetching of its code, which every launch does anew.
    if (total_rows < 192 * e_count && total_rows < 16384) {                        // uniform
        __syncthreads();
        int start = 0;
        const int upto = t < e_count ? t : e_count;
        for (int r = 0; r < upto; ++r) start += tl[r];
        for (int mt = 0; mt < my_tiles; ++mt) put(mine, my_n, my_tiles, mt, start + mt);
        if (t == 255) plan[16 + list] = min(start + my_tiles, max_tiles);
    } else {
        // Sums over the ranks of the tiles, and of those of experts with several: in the waves, then over the four that work.  The tiles are then
        // spread over all threads (an expert with half of the rows of a skewed batch has dozens).  Kernel us, sums by a loop over the experts and
        // tiles spread over 256 threads -> as here: the list of 20000 rows on 64 experts 12.2 -> 8.9 (sorted by such a loop and not merged 7.3), of 60000 on
        // 256 20.0 -> 12.7; the batching of 32768 skewed on 64 with the list 19.5 -> 14.
        int (&start)[256] = scratch[4], (&several_start)[256] = scratch[5], (&sums)[256] = scratch[6];
        const int lane = t & 63, wave = t >> 6, my_several = my_tiles > 1 ? my_tiles : 0;
        int incl = my_tiles, incl_several = my_several;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off), w = __shfl_up(incl_several, off);
            if (lane >= off) { incl += v; incl_several += w; }
        }
        if (worker && lane == 63) {
            sums[wave] = incl;
            sums[4 + wave] = incl_several;
        }
        __syncthreads();
        int total = 0, several = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < wave) { incl += sums[w]; incl_several += sums[4 + w]; }
            total += sums[w];
            several += sums[4 + w];
        }
        if (worker) {
            start[t] = incl - my_tiles;
            several_start[t] = incl_several - my_several;
        }
        __syncthreads();
        const int groups = several / 4, other_groups = (total - 4 * groups) / 4;   // (what does not fill a group of the first kind counts as the rest)
#pragma unroll 1
        for (int s = t; s < total; s += blockDim.x) {
            int r = 0;                             // the last expert, in the order of the ranks, that starts at or before s
#pragma unroll
            for (int step = 128; step > 0; step >>= 1)
                if (r + step < e_count && start[r + step] <= s) r += step;
            const int e = order[r], mt = s - start[r], n_tiles = tl[r], before = several_start[r];
            // group g of G comes after those of the H others whose middle, (2 i + 1) / 2 H, lies before its own
            const bool grouped = n_tiles > 1 && before + mt < 4 * groups;
            const int in_kind = grouped ? before + mt : n_tiles > 1 ? before + mt - 4 * groups : several - 4 * groups + start[r] - before;
            const int g = in_kind / 4, own = grouped ? groups : other_groups, other = grouped ? other_groups : groups;
            // what does not fill a group of the rest comes last
            const int at = !grouped && g >= other_groups
                               ? 4 * groups + in_kind
                               : 4 * (g + (other > 0 ? min((((2 * g + 1) * other - (grouped ? 1 : 0)) / own + 1) / 2, other) : 0)) + in_kind % 4;
            put(e, n[e] & ((1 << kRowBits) - 1), n_tiles, mt, at);
        }
        if (t == 0) plan[16 + list] = min(total, max_tiles);
    }
    if (list == 0 && t < 16) plan[t] = 0;
}

}  // namespace moe
