// Expert FFN kernels for batches of few rows per expert: every product is then a read of the experts' weights and nothing
// else, and with few experts hit, or small ones, the tiles of the large kernel are too few to have enough of that read in
// flight.  Here a wave owns 16 columns (32 in the down-projection of more than 16 rows) for up to 64 rows of an expert, in blocks of
// one or two waves that know nothing of each other: some ten times the waves of the large kernel, no barrier, no LDS, weights and
// activations straight into operand registers several steps ahead.  A column's sum is one chain over the reduction dimension that
// starts where the large kernel starts it: both kernels give the same bits, so a row's result depends neither on the batch it came in nor on which of the
// two ran, and the choice between them is a question of time alone.
// Layer of 32 experts, d 4096, f 10240, large kernel -> here: 1 token 186 -> 61 us, 4 tokens 257 -> 167, 16 tokens 540 -> 508,
// 40 tokens 906 -> 856.  (A block of four waves that split the steps of a chain between them takes 61, 165, 494 and 863 us,
// but its four partial sums round differently.)
#pragma once
#include "common.h"
#include "ffn_plan.h"

#include <type_traits>

namespace moe {

// Steps of 64 reduction elements in flight, as the registers of 2 to 4 waves per SIMD allow.  SMALL (16 rows in all), steps of the
// down-projection and waves: 8 and 3 / 7 and 4 / 6 and 4 measure 59.6 / 60.8 / 62.7 us for one token, 523 / 508 / 509 for 16.
// DEEP, a down-projection with a wave per compute unit at most, which then has the unit's loads in flight to itself (one token: 14 KiB of the 44 that a unit
// can have): 7 / 14 / 24 steps take 56.0 / 54.4 / 55.3 us for one token on 32 experts, 57.4 / 54.0 / 54.2 on 8; two tokens, whose units
// have two waves, 91.7 / 92.9 / 94.0, and 32 steps in all (4 tokens on 8 experts, d 512, f 2048) 16.0 / 16.5 / 17.5.
constexpr int few_depth(bool up, bool small, bool deep, int RB) { return deep ? 14 : small ? (up ? 4 : 7) : RB == 1 ? 8 : RB == 2 ? 6 : 3; }
constexpr int few_waves_per_simd(bool small, bool deep) { return small && !deep ? 4 : 2; }
constexpr int few_columns(bool up, bool small) { return up || small ? 16 : 32; }

// The rows of a tile: row_begin, row_begin + 1, ... of the batched order; or, where the kernel reads idx itself, in the order of the
// assignments, lane r holding the r-th.
template <bool DIRECT>
struct FewRows {
    int e, row_begin, rows, assignment;
    __device__ int row(int r) const { return DIRECT ? __builtin_amdgcn_ds_bpermute(4 * r, assignment) : row_begin + r; }
};

// GATED: H = act(A W_gate) * (A W_in), 16 columns of d_ff per block; else 16 or 32 columns of W_out.  Rows row_begin ..
// row_begin + rows of the batched order, rows <= 16 RB, all of expert e.  Act: act(z) of the gate.  A: GATED, the token array
// (row r of the batched order is row gather[r] / gather_k) or the batched rows (gather NULL); else H in its chunked order,
// [chunk of 64 columns][row][64].
template <bool GATED, bool SMALL, bool DEEP, int RB, bool DIRECT, class Act>
__device__ inline void ffn_few_rows(const uint16_t* A, const FewRows<DIRECT>& tile, int e_first, const char* W,
                                    size_t expert_stride_bytes, size_t block_offset_bytes, uint16_t* __restrict__ C, int K, int N,
                                    const int32_t* __restrict__ row_map, const int32_t* __restrict__ gather, int gather_k,
                                    int h_rows, Act act) {
    typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 b16x4 __attribute__((ext_vector_type(4)));
    typedef float fx4 __attribute__((ext_vector_type(4)));
    typedef uint32_t ux4 __attribute__((ext_vector_type(4)));
    constexpr int kColumns = few_columns(GATED, SMALL);
    constexpr int NJ = GATED ? 2 : kColumns / 16;   // weight operands of a k-step of 32: gate and in, or 16 columns each
    constexpr int kDepth = few_depth(GATED, SMALL, DEEP, RB);
    const int lane = threadIdx.x & 63, c15 = lane & 15, g = lane >> 4;
    const int e = tile.e, rows = tile.rows;
    // The units that share the 8 KiB window of a step in the packed weights (two, or four of 16 columns of W_out) go to blocks
    // of one XCD that start together: 64 experts, 64 tokens x 2: 2.29 -> 2.25 ms.
    constexpr int kShare = GATED || kColumns == 32 ? 1 : 2, kGroup = 8 << kShare;
    // Blocks of two waves hold two neighbours.
    const int bx = blockIdx.x, inside_group = bx % kGroup;
    const int unit = blockDim.x > 64 ? 2 * bx + __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6))
                   : bx < static_cast<int>(gridDim.x) / kGroup * kGroup
                         ? bx - inside_group + ((inside_group & 7) << kShare) + (inside_group >> 3) : bx;
    const int col0 = unit * kColumns;

    // this wave's weight stream: 16 columns x 32 rows per operand, taken from the packed 16-row x 32-column fragments
    // (lane 16 g + c: fragment row step g / 2, slot 32 (g % 2) + c)
    const int pair = GATED ? col0 >> 5 : col0 >> 6;
    const int inside = (GATED ? 0 : ((col0 >> 5) & 1) * 1024) + ((col0 >> 4) & 1) * 256;
    const char* wb = W + static_cast<size_t>(e - e_first) * expert_stride_bytes + block_offset_bytes +
                     static_cast<size_t>(pair) * (K / 16) * 2048 + inside;
    const uint32_t w_lane = ((g >> 1) << 11) + ((g & 1) << 9) + (c15 << 4);
    const size_t a_step = GATED ? 128 : static_cast<size_t>(h_rows) * 128;
    const int steps = K / 64;
    const int phase = static_cast<int>(sweep_key(e, static_cast<unsigned>(col0) >> (GATED ? 10 : 11)) % static_cast<unsigned>(steps));
    auto at = [&](int i) { return phase + i < steps ? phase + i : phase + i - steps; };       // i < steps

    fx4 acc[RB][NJ];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[rb][j] = fx4{0.f, 0.f, 0.f, 0.f};
    // this lane's activation rows: byte offsets from A
    uint32_t a_lane[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = tile.row(min(rb * 16 + c15, rows - 1));         // past the end: the last row again, not stored
        const int src = !GATED ? row : DIRECT ? row / gather_k : gather != nullptr ? gather[row] / gather_k : row;
        a_lane[rb] = static_cast<uint32_t>(src) * (GATED ? static_cast<uint32_t>(K) * 2u : 128u) + 16u * g;
    }
    ux4 wr[kDepth][2][NJ], ar[kDepth][2][RB];
    // Every step issues the same loads in the same order, the first ones and those past the last step (where all lanes read one
    // line) as well, so that the compiler knows how many are outstanding at every wait.  The mask is opaque because the compiler
    // would make it a branch around the loads, and W and A are not __restrict__ because the fence would not hold their loads then:
    // it would move them down to their use.
    auto load = [&](int q, int s) __attribute__((always_inline)) {
        const bool past = s >= steps;
        const size_t step = past ? 0 : at(s);
        uint32_t keep = past ? 0u : ~0u;
        asm("" : "+v"(keep));
        const char* wp = wb + step * 8192;
        const char* ap = reinterpret_cast<const char*>(A) + step * a_step;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                wr[q][k2][j] = __builtin_nontemporal_load(reinterpret_cast<const ux4*>(wp + 4096 * k2 + (GATED ? j * 1024 : j * 256) + (w_lane & keep)));
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) ar[q][k2][rb] = *reinterpret_cast<const ux4*>(ap + 64 * k2 + (a_lane[rb] & keep));
        asm volatile("" : : : "memory");
    };
#pragma unroll
    for (int q = 0; q < kDepth; ++q) load(q, q);
    for (int s0 = 0; s0 < steps; s0 += kDepth) {
#pragma unroll
        for (int q = 0; q < kDepth; ++q) {
            if (s0 + q < steps) {                    // uniform
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b16x8, wr[q][k2][j]),
                                                                                 __builtin_bit_cast(b16x8, ar[q][k2][rb]), acc[rb][j], 0, 0, 0);
            }
            load(q, s0 + q + kDepth);
        }
    }
    // the weights are the first operand: lane 16 g + c holds row c of its row block and columns 4 g .. 4 g + 3 of every 16
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = tile.row(rb * 16 + c15);                        // (all lanes: it may be a lane exchange)
        if (rb * 16 + c15 < rows) {
            const size_t out_row = GATED || row_map == nullptr ? row : row_map[row];
#pragma unroll
            for (int j = 0; j < kColumns / 16; ++j) {
                b16x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    o[i] = static_cast<__bf16>(GATED ? act(acc[rb][0][i]) * acc[rb][NJ - 1][i] : acc[rb][j][i]);
                const int c = col0 + 16 * j + 4 * g;
                const size_t to = GATED ? (static_cast<size_t>(c >> 6) * h_rows + row) * 64 + (c & 63) : out_row * N + c;
                *reinterpret_cast<b16x4*>(C + to) = o;
            }
        }
    }
}

// A wave: one column unit (from blockIdx.x) of one row tile (blockIdx.y, an entry of the work list, at most kFewTileM rows).
// DIRECT: there is no work list and no batched order, but idx; tile blockIdx.y is the expert whose first assignment is the blockIdx.y-th such, and all A
// assignments are looked through here (one read and a few lane votes, against a launch and three dependent reads: 1 token
// 59.7 -> 55.2 us, 30 tokens x 2 on 8 experts, d 1024, f 2048 37.6 -> 33.3; fp32, 64 tokens, d 256, f 512, 4 experts 23.3 -> 19.7).
template <bool GATED, bool SMALL, bool DEEP, bool DIRECT, class Act>
__device__ inline void ffn_few_block(const uint16_t* A, const int32_t* __restrict__ plan, int e_first, const char* W,
                                     size_t expert_stride_bytes, size_t block_offset_bytes, uint16_t* __restrict__ C, int K, int N,
                                     const int32_t* __restrict__ row_map, const int32_t* __restrict__ gather, int gather_k,
                                     int h_rows, const int32_t* __restrict__ idx, int n_idx, int E, Act act) {
    const int tile = blockIdx.y;
    FewRows<DIRECT> at;
    if constexpr (DIRECT) {
        const int lane = threadIdx.x & 63;
        int expert;
        const unsigned long long peers = direct_peers(idx, n_idx, E, lane, expert), below = (1ull << lane) - 1ull;
        const bool first = peers != 0ull && (peers & below) == 0ull;
        const unsigned long long firsts = __ballot(first);
        if (tile >= __popcll(firsts)) return;       // uniform: fewer experts have rows than the grid provides for
        const int leader = __ffsll(static_cast<long long>(__ballot(first && __popcll(firsts & below) == tile))) - 1;
        const unsigned lo = __builtin_amdgcn_readlane(static_cast<int>(peers), leader), hi = __builtin_amdgcn_readlane(static_cast<int>(peers >> 32), leader);
        const unsigned long long members = static_cast<unsigned long long>(hi) << 32 | lo;
        at.e = __builtin_amdgcn_readlane(expert, leader);
        at.rows = __popcll(members);
        at.row_begin = 0;
        // every lane sends its number to its place: the members in order, the others behind them
        const int place = (members >> lane) & 1ull ? __popcll(members & below) : at.rows + __popcll(~members & below);
        at.assignment = __builtin_amdgcn_ds_permute(4 * place, lane);
    } else {
        const int n_tiles = plan[16];
        const int4 t = reinterpret_cast<const int4*>(plan + kPlanHeader)[tile];      // (the list has room for every tile of the grid)
        if (tile >= n_tiles) return;                // uniform, as above
        // the same for all lanes: kept in scalar registers
        at.e = __builtin_amdgcn_readfirstlane(t.x);
        at.row_begin = __builtin_amdgcn_readfirstlane(t.y);
        at.rows = __builtin_amdgcn_readfirstlane(t.z);
        at.assignment = 0;
    }
    const int rows = at.rows;
    auto run = [&](auto rb) __attribute__((always_inline)) {
        ffn_few_rows<GATED, SMALL, DEEP, decltype(rb)::value, DIRECT>(A, at, e_first, W, expert_stride_bytes, block_offset_bytes, C, K, N,
                                                        row_map, gather, gather_k, h_rows, act);
    };
    if constexpr (SMALL) {
        run(std::integral_constant<int, 1>{});
    } else {
        if (rows <= 16) run(std::integral_constant<int, 1>{});
        else if (rows <= 32) run(std::integral_constant<int, 2>{});
        else run(std::integral_constant<int, 4>{});
    }
}

}  // namespace moe
