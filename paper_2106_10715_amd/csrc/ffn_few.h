// Expert FFN kernels for batches of few rows per expert: every product is then a read of the experts' weights and nothing
// else, and with few experts hit, or small ones, the tiles of the large kernel are too few, and each too long a chain, to have
// enough of that read in flight.  Here a block holds one unit of 16 or 32 output columns for all rows of an expert, its waves
// take the steps of the reduction dimension in turn, and the partial tiles are added in wave order through the LDS;
// activations come straight from the L2 into operand registers, so a wave's loop has no barrier and no LDS access.  Steps in
// turn, not a slice per wave: a block then reads one contiguous window (16 tokens 531 -> 516 us).  Four waves or eight, and
// one, two or three steps in flight, measure the same.  Layer of 32 experts, d 4096, f 10240, large kernel -> here: 1 token
// 167 -> 61 us, 4 tokens 267 -> 174, 16 tokens 556 -> 517, 40 tokens 900 -> 849.
#pragma once
#include "common.h"
#include "ffn_plan.h"

#include <type_traits>

namespace moe {

constexpr int kFewWaves = 4;

// GATED: H = act(A W_gate) * (A W_in), 32 columns of d_ff per block; else 16 CB columns of W_out.  Rows row_begin ..
// row_begin + rows of the batched order, rows <= 16 RB, all of expert e.  Act: act(z) of the gate.  A: GATED, the token array
// (row r of the batched order is row gather[r] / gather_k) or the batched rows (gather NULL); else H in its chunked order,
// [chunk of 64 columns][row][64].
template <bool GATED, int RB, int CB, class Act>
__device__ inline void ffn_few_rows(float* lds, const uint16_t* __restrict__ A, int e, int row_begin, int rows, int e_first,
                                    const char* __restrict__ W, size_t expert_stride_bytes, size_t block_offset_bytes,
                                    uint16_t* __restrict__ C, int K, int N, const int32_t* __restrict__ row_map,
                                    const int32_t* __restrict__ gather, int gather_k, int h_rows, Act act) {
    typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
    typedef float fx4 __attribute__((ext_vector_type(4)));
    typedef uint32_t ux4 __attribute__((ext_vector_type(4)));
    constexpr int NJ = GATED ? 4 : CB;              // weight operands of a k-step of 32: (gate, in) x halves, or halves
    constexpr int kDepth = RB == 4 ? (GATED ? 1 : 2) : GATED ? 2 : 4;         // steps of 64 in flight
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int c15 = lane & 15, g = lane >> 4;
    const int unit = blockIdx.x;

    // this wave's weight stream: 16 columns x 32 rows per operand, taken from the packed 16-row x 32-column fragments
    // (lane 16 g + c: fragment row step g / 2, slot 32 (g % 2) + c)
    const int pair = GATED ? unit : (CB == 2 ? unit >> 1 : unit >> 2);
    const int inside = GATED ? 0 : CB == 2 ? (unit & 1) * 1024 : ((unit >> 1) & 1) * 1024 + (unit & 1) * 256;
    const char* wb = W + static_cast<size_t>(e - e_first) * expert_stride_bytes + block_offset_bytes +
                     static_cast<size_t>(pair) * (K / 16) * 2048 + inside;
    const uint32_t w_lane = ((g >> 1) << 11) + ((g & 1) << 9) + (c15 << 4);
    const size_t a_step = GATED ? 128 : static_cast<size_t>(h_rows) * 128;
    const int steps = K / 64, mine = (steps - wave + kFewWaves - 1) / kFewWaves;       // step i of the wave: wave + kFewWaves i

    fx4 acc[RB][NJ];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[rb][j] = fx4{0.f, 0.f, 0.f, 0.f};
    ux4 wr[kDepth][2][NJ], ar[kDepth][2][RB];
    // Every step issues the same loads, also past the wave's last step (there all lanes read one line), so that the number
    // of loads outstanding is known at every wait.
    auto load_w = [&](int q, int s) __attribute__((always_inline)) {
        const bool past = s >= mine;
        const char* wp = wb + (past ? size_t(0) : static_cast<size_t>(wave + s * kFewWaves) * 8192);
        const uint32_t wl = past ? 0u : w_lane;
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                wr[q][k2][j] = __builtin_nontemporal_load(reinterpret_cast<const ux4*>(wp + 4096 * k2 + (GATED ? (j >> 1) * 1024 + (j & 1) * 256 : j * 256) + wl));
        asm volatile("" : : : "memory");             // the loads stay here: the compiler would move them down to their use
    };
    // the first weights are requested before the activation rows are looked up
#pragma unroll
    for (int q = 0; q < kDepth; ++q) load_w(q, q);
    // this lane's activation rows: byte offsets from A
    uint32_t a_lane[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = row_begin + min(rb * 16 + c15, rows - 1);       // past the end: the last row again, not stored
        const int src = GATED && gather != nullptr ? gather[row] / gather_k : row;
        a_lane[rb] = static_cast<uint32_t>(src) * (GATED ? static_cast<uint32_t>(K) * 2u : 128u) + 16u * g;
    }
    auto load_a = [&](int q, int s) __attribute__((always_inline)) {
        const bool past = s >= mine;
        const char* ap = reinterpret_cast<const char*>(A) + (past ? size_t(0) : static_cast<size_t>(wave + s * kFewWaves) * a_step);
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) ar[q][k2][rb] = *reinterpret_cast<const ux4*>(ap + 64 * k2 + (past ? 0u : a_lane[rb]));
        asm volatile("" : : : "memory");
    };
#pragma unroll
    for (int q = 0; q < kDepth; ++q) load_a(q, q);
    for (int s0 = 0; s0 < mine; s0 += kDepth) {
#pragma unroll
        for (int q = 0; q < kDepth; ++q) {
            if (s0 + q < mine) {                     // uniform for the wave
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b16x8, wr[q][k2][j]),
                                                                                 __builtin_bit_cast(b16x8, ar[q][k2][rb]), acc[rb][j], 0, 0, 0);
            }
            load_a(q, s0 + q + kDepth);
            load_w(q, s0 + q + kDepth);
        }
    }
    // partial tiles through the LDS, one 16-row block at a time: [wave][operand][row][16 columns + 4]
    constexpr int kRow = 20, kTile = 16 * kRow;
    constexpr int kCols = GATED ? 32 : 16 * CB;      // output columns of the block
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (rb * 16 >= rows) break;                  // uniform
        if (rb > 0) __syncthreads();
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            *reinterpret_cast<fx4*>(lds + (wave * NJ + j) * kTile + c15 * kRow + 4 * g) = acc[rb][j];
        __syncthreads();
        constexpr int kPerPass = kFewWaves * 64 / kCols;                 // rows all threads cover at once
        const int col = threadIdx.x % kCols;
        for (int r = threadIdx.x / kCols; r < 16; r += kPerPass) {
            if (rb * 16 + r >= rows) break;
            const float* p = lds + (col >> 4) * kTile + r * kRow + (col & 15);
            float v = p[0], u = GATED ? p[2 * kTile] : 0.f;
#pragma unroll
            for (int w = 1; w < kFewWaves; ++w) {
                v += p[w * NJ * kTile];
                if (GATED) u += p[(w * NJ + 2) * kTile];
            }
            if (GATED) v = act(v) * u;
            const int row = row_begin + rb * 16 + r, c = unit * kCols + col;
            const size_t at = GATED ? (static_cast<size_t>(c >> 6) * h_rows + row) * 64 + (c & 63)
                                    : static_cast<size_t>(row_map != nullptr ? row_map[row] : row) * N + c;
            C[at] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
        }
    }
}

// A block: one column unit (blockIdx.x) of one expert with rows (blockIdx.y, an entry of the work list).
template <bool GATED, int CB, class Act>
__device__ inline void ffn_few_block(float* lds, const uint16_t* __restrict__ A, const int32_t* __restrict__ plan, int e_first,
                                     const char* __restrict__ W, size_t expert_stride_bytes, size_t block_offset_bytes,
                                     uint16_t* __restrict__ C, int K, int N, const int32_t* __restrict__ row_map,
                                     const int32_t* __restrict__ gather, int gather_k, int h_rows, Act act) {
    const int tile = blockIdx.y;
    const int n_tiles = plan[16];
    const int4 t = reinterpret_cast<const int4*>(plan + kPlanHeader)[tile];      // (the list has room for every tile of the grid)
    if (tile >= n_tiles) return;                    // uniform: fewer experts have rows than the grid provides for
    auto rows_of = [&](auto rb, int first, int rows) __attribute__((always_inline)) {
        ffn_few_rows<GATED, decltype(rb)::value, CB>(lds, A, t.x, t.y + first, rows, e_first, W, expert_stride_bytes, block_offset_bytes,
                                                     C, K, N, row_map, gather, gather_k, h_rows, act);
    };
    if (t.z <= 16) {
        rows_of(std::integral_constant<int, 1>{}, 0, t.z);
    } else if (t.z <= 32) {
        rows_of(std::integral_constant<int, 2>{}, 0, t.z);
    } else {
        for (int first = 0; first < t.z; first += 64) {
            if (first > 0) __syncthreads();
            rows_of(std::integral_constant<int, 4>{}, first, min(64, t.z - first));
        }
    }
}

}  // namespace moe
