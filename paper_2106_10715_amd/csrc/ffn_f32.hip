// fp32 expert feed-forward networks (the same grouped products as ffn.hip, on row-major fp32 weights):
//
//     H  = act(Xp W_gate[e]) * (Xp W_in[e])        "up",   epilogue fused
//     Yp = H W_out[e]                               "down"
//
// on the bf16 matrix instruction, with every fp32 value as the sum of three bf16 values that together hold all its 24 bits.
#include "common.h"

#include <math.h>

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline float act_f32(float z, int act) {
    if (act == 0) return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
    const float u = 0.79788456080286536f * (z + 0.044715f * z * z * z);
    return 0.5f * z * (1.0f + tanhf(u));
}

// Which (expert, row tile) a block works on: tile slot `slot` counted over the experts
// [e_first, e_first + e_count) in order, at most tile_m rows per tile.  Returns false when the slot is past
// the last tile (uniform for the block).  Must be called by all threads of the block.
__device__ inline bool find_tile(const int32_t* __restrict__ offsets, int e_first, int e_count, int tile_m, int slot,
                                 int total_rows, int& e_out, int& row_begin, int& rows) {
    // segment of expert e, clamped so that whatever the offsets hold no tile reaches outside the rows there are
    auto seg_lo = [&](int e) { return min(max(offsets[e], 0), total_rows); };
    auto seg_hi = [&](int e) { return min(max(offsets[e + 1], seg_lo(e)), total_rows); };
    __shared__ int sh_e, sh_mt;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int tl[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = lane * 4 + q;
            const int cnt = e < e_count ? seg_hi(e_first + e) - seg_lo(e_first + e) : 0;
            tl[q] = (cnt + tile_m - 1) / tile_m;
            sum += tl[q];
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        const int target = slot;
        int run = incl - sum;
        if (target >= run && target < incl) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (target >= run && target < run + tl[q]) { sh_e = lane * 4 + q; sh_mt = target - run; }
                run += tl[q];
            }
        }
        const int total = __shfl(incl, 63);
        if (lane == 0 && target >= total) sh_e = -1;
    }
    __syncthreads();
    if (sh_e < 0) return false;
    e_out = e_first + sh_e;
    // the expert's rows are split evenly over its tiles (in multiples of 16 rows), not into full tiles
    // and a small remainder: equal tiles finish together and none is nearly empty
    const int lo = seg_lo(e_out), hi = seg_hi(e_out), n = hi - lo;
    const int tiles = (n + tile_m - 1) / tile_m;
    const int per_tile = min(tile_m, ((n + tiles - 1) / tiles + 15) & ~15);
    row_begin = lo + sh_mt * per_tile;
    rows = min(per_tile, hi - row_begin);
    return true;
}

// The same for at most kDirectRows assignments that nothing has batched: the experts in the order of their
// first assignments, row r of the tile is assignment sh_row[r].
__device__ inline bool find_tile_direct(const int32_t* __restrict__ idx, int A, int E, int tile_m, int slot, int (&sh_row)[kDirectRows], int& e_out, int& rows) {
    __shared__ int sh_e, sh_n;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int expert;
        const unsigned long long peers = direct_peers(idx, A, E, lane, expert), below = (1ull << lane) - 1ull;
        const int n = __popcll(peers), tiles = (n + tile_m - 1) / tile_m;
        const bool first = peers != 0ull && (peers & below) == 0ull;
        // tiles of the experts before this lane's; an expert has at most kDirectRows / 16
        int start = 0;
#pragma unroll
        for (int i = 0; i < kDirectRows / 16; ++i) start += __popcll(__ballot(first && tiles > i) & below);
        const unsigned long long found = __ballot(first && slot >= start && slot < start + tiles);
        if (found == 0ull) {
            if (lane == 0) sh_e = -1;
        } else {
            const int leader = __ffsll(static_cast<long long>(found)) - 1;
            const int per_tile = min(tile_m, ((n + tiles - 1) / max(tiles, 1) + 15) & ~15), lo = (slot - __shfl(start, leader)) * per_tile;
            if (lane == leader) { sh_e = expert; sh_n = min(per_tile, n - lo); }
            const int at = __popcll(peers & below) - lo;
            if (((peers >> leader) & 1ull) && at >= 0 && at < per_tile) sh_row[at] = lane;
        }
    }
    __syncthreads();
    if (sh_e < 0) return false;
    e_out = sh_e;
    rows = sh_n;
    return true;
}

// Eight values, times 2^16, as three bf16 operands: the upper 16 bits of the value, of what they leave, and of what is left then (8 + 8 + 8
// significant bits, nothing is rounded).  Without the factor the last bits of values below 2^-110 would lie below the smallest bf16 (2^-133; the
// instruction takes those below its normal range as they are); values of 2^112 and more become infinite by it.
constexpr float kUp = 65536.0f, kDown = 1.0f / (kUp * kUp);                  // of an operand, of a product
struct Split { u32x4 v[3]; };
__device__ __attribute__((always_inline)) inline Split split8(const float (&x)[8]) {
    Split s;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        uint32_t bits[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float v = x[2 * p + h] * kUp;
            const float rest = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
            const float last = rest - __uint_as_float(__float_as_uint(rest) & 0xffff0000u);
            bits[h][0] = __float_as_uint(v);
            bits[h][1] = __float_as_uint(rest);
            bits[h][2] = __float_as_uint(last);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) s.v[q][p] = __builtin_amdgcn_perm(bits[1][q], bits[0][q], 0x07060302u);      // the upper halves
    }
    return s;
}
__device__ __attribute__((always_inline)) inline f32x4 mfma(const u32x4& w, const u32x4& a, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
}

constexpr int kRows = 64;                                // most rows of a tile
constexpr int kPartRow = 68;                             // floats per row of a partial tile in LDS: up to 64 and 4 of padding
// Columns of a lane, of each matrix: a block has 16 times as many.
constexpr int lane_columns(bool gated, bool narrow) { return (gated ? 2 : 4) >> (narrow ? 1 : 0); }

// What bounds it: the vector instructions that split the operands and add the sums (58 % of the cycles at 1024 rows of 8 experts, d 1024, f 4096, the matrix
// instructions 35 %); the latency of a block's few steps in short launches.  Eight of the nine products of the parts are formed, so that a product has all its bits: the one
// left out, of the two last parts, is below 2^-30 of the whole (second part < 2^-7 of the value, third < 2^-15).  The instruction cuts off where it adds, so the product of the first parts, which for one
// product is exact, is added to the sum of the seven small ones outside of it, and both to the running sum, in fp32: two roundings per 32 elements.
// Relative error against 64 bits, sums of normally distributed products, here / by chains of fp32 multiply-adds in four quarters: 4096 products 1.2e-7 / 5.7e-7
// (positive ones 0.6e-7 / 2.5e-7), 64 products 4.7e-8 / 8.4e-8, 16 5.3e-8 / 5.8e-8, one 2.6e-8 (half of the last bit at most) / the same; 1024 equal
// products (1/3 squared) 0.8e-7 / 27e-7.  Six products (without second x third) and one addition take 10 % less time, but leave out up to 2^-21 of a
// product, always of its sign (one product 6.9e-8).
// A block is one tile of up to 64 rows by 64 weight columns (GATED: 32 of each matrix), or half as many; its four waves take a quarter of the
// reduction dimension each and share nothing until their partial tiles are added in wave order at the end, so there is no barrier
// in the loop, no LDS, and every row's sum has the same order in every tile and batch.  Weights and activations go straight into registers in operand order: a lane's
// eight reduction elements are 4 g .. 4 g + 3 and 16 + 4 g .. of 32 (g = lane / 16), its two or four columns are neighbours.
// A value that comes out infinite or NaN is computed again in fp64, by one thread per four columns: the parts of an infinity are no numbers, and
// the operands' factor may have made it one.  So the result is infinite only where the sum is.  It is slow: 512 tokens x 2 of the layer below take 0.5 ms with one NaN
// among them and 2 ms if all are (0.3 ms without).
// Against tiles of 64 x 64 and 32 x 32 through LDS with the fp32 instruction, layers in us: 512 tokens x 2, d 1024, f 4096, 8 experts 354 -> 297, 4096 x 2 1947 ->
// 1671, 8192 x 1, d 512, f 2048 555 -> 477, 16 x 1 on 8 142 -> 106, 1000 x 1, f 1024, 5 experts 119 -> 94, 100 x 1, d 512, f 2048, 4 experts
// 45.4 -> 38.8, 64 x 1, d 256, f 512, 4 experts 23.2 -> 19.2; 142 x 2, d 192, f 576, 4 experts 26.4 -> 28.7 and others of that size lose 1-2 us to the
// start of a block. Blocks that take several column groups one after the other: 5-15 % slower.
template <bool GATED, bool NARROW, int RB>
__device__ inline void ffn_f32_tile(const float* A, const int32_t* gather, int gather_k, bool direct, const int (&sh_row)[kDirectRows], int row_begin,
                                    int rows, const float* W0, const float* W1, float* C, int K, int N, int n0, int act, const int32_t* row_map,
                                    float (&part)[4][kRows * kPartRow]) {
    constexpr int kDepth = RB >= 3 ? 1 : RB == 2 ? 2 : 3;                   // steps requested ahead, as the registers allow
    constexpr int NC = lane_columns(GATED, NARROW), NM = GATED ? 2 : 1, NJ = NM * NC;     // a lane's columns, matrices, operands
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c15 = lane & 15, g = lane >> 4;
    const int steps = K / 32, s_lo = wave * steps / 4, s_hi = (wave + 1) * steps / 4;
    auto in_row = [&](int r) {                                              // where row r of the tile is read
        const int at = row_begin + min(r, rows - 1);                        // past the end: the last row again, not stored
        const int row = direct ? sh_row[at] : at;
        return GATED && direct ? row / gather_k : gather != nullptr ? gather[row] / gather_k : row;
    };
    typedef float wcols __attribute__((ext_vector_type(NC)));
    const float* a_src[RB];                                                 // next to be requested
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) a_src[rb] = A + static_cast<size_t>(in_row(16 * rb + c15)) * K + 4 * g + 32 * min(s_lo, steps - 1);
    const uint32_t w_lane = static_cast<uint32_t>(4 * g * N + NC * c15) * 4u;
    f32x4 acc[RB][NJ];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[rb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float aw[kDepth][RB][8], ww[kDepth][8][NJ];
    // (steps past the wave's last one are read from that one and not used; a fence after every batch of loads, and pointers that are
    // not __restrict__: the compiler would move the loads down to their use.  The same for all lanes up to the lane's 32-bit offset.)
    auto load_w = [&](int q, int s) __attribute__((always_inline)) {
        const size_t at = (static_cast<size_t>(32 * max(min(s, s_hi - 1), 0)) * N + n0) * 4;
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const char* from = reinterpret_cast<const char*>(m == 0 ? W0 : W1) + (at + static_cast<size_t>(j < 4 ? j : 12 + j) * N * 4);
                const wcols u = *reinterpret_cast<const wcols*>(from + w_lane);
#pragma unroll
                for (int i = 0; i < NC; ++i) ww[q][j][m * NC + i] = u[i];
            }
    };
    auto load_a = [&](int q, int rb, int s) __attribute__((always_inline)) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(a_src[rb]), v = *reinterpret_cast<const f32x4*>(a_src[rb] + 16);
        if (s + 1 < s_hi) a_src[rb] += 32;                                  // uniform
#pragma unroll
        for (int i = 0; i < 4; ++i) { aw[q][rb][i] = u[i]; aw[q][rb][4 + i] = v[i]; }
    };
#pragma unroll
    for (int q = 0; q < kDepth; ++q) {
        load_w(q, s_lo + q);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) load_a(q, rb, s_lo + q);
        asm volatile("" : : : "memory");
    }
    for (int s0 = s_lo; s0 < s_hi; s0 += kDepth) {
#pragma unroll
        for (int q = 0; q < kDepth; ++q) {
            const int s = s0 + q;
            if (s >= s_hi) break;                                           // uniform
            // The next loads go out as soon as their registers are free, and the operands of a row block are split under the products
            // of the one before: nothing is moved across the barriers of the scheduler.
            Split w[NJ], a;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const float x[8] = {ww[q][0][j], ww[q][1][j], ww[q][2][j], ww[q][3][j], ww[q][4][j], ww[q][5][j], ww[q][6][j], ww[q][7][j]};
                w[j] = split8(x);
            }
            a = split8(aw[q][0]);
            __builtin_amdgcn_sched_barrier(0);
            load_w(q, s + kDepth);
            load_a(q, 0, s + kDepth);
            asm volatile("" : : : "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                Split next;
                if (rb + 1 < RB) next = split8(aw[q][rb + 1 < RB ? rb + 1 : rb]);
                f32x4 z[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[2], a.v[1], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[1], a.v[2], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[2], a.v[0], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[0], a.v[2], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[1], a.v[1], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[1], a.v[0], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[j] = mfma(w[j].v[0], a.v[1], z[j]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[rb][j] += z[j] + mfma(w[j].v[0], a.v[0], f32x4{0.f, 0.f, 0.f, 0.f});
                if (rb + 1 < RB) {
#pragma unroll
                    for (int i = 0; i < 8 * NJ; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA,
                        __builtin_amdgcn_sched_group_barrier(0x002, 7 / NJ, 0);  // some of the splitting
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    load_a(q, rb + 1, s + kDepth);
                    asm volatile("" : : : "memory");
                    a = next;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // the weights are the first operand: lane 16 g + c holds row c of its block and, in acc[..][m NC + j][i], column NC (4 g + i) + j of matrix m.
    // Partial tile: a row's columns of the first matrix, then those of the second.
    float* mine = part[wave];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            float* to = mine + (16 * rb + c15) * kPartRow + 16 * NC * m + NC * 4 * g;
#pragma unroll
            for (int v = 0; v < NC; ++v) {
                f32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = acc[rb][m * NC + (4 * v + i) % NC][(4 * v + i) / NC];
                *reinterpret_cast<f32x4*>(to + 4 * v) = o;
            }
        }
    __syncthreads();
    constexpr int kVec = 16 * NC / 4;                                       // 16-byte pieces of an output row
    for (int id = tid; id < RB * 16 * kVec; id += 256) {
        const int r = id / kVec, col = 4 * (id % kVec);
        f32x4 sum[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            sum[m] = *reinterpret_cast<const f32x4*>(part[0] + r * kPartRow + 16 * NC * m + col);
#pragma unroll
            for (int v = 1; v < 4; ++v) sum[m] += *reinterpret_cast<const f32x4*>(part[v] + r * kPartRow + 16 * NC * m + col);
        }
        if (r >= rows) continue;
        bool finite = true;
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                finite = finite && fabsf(sum[m][i]) <= 3.402823466e38f;
                sum[m][i] *= kDown;                                         // (an infinity or a NaN stays one)
            }
        if (!finite) {
            constexpr int kAhead = 16 / NM;
            const float* a = A + static_cast<size_t>(in_row(r)) * K;
            double total[NM][4];
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) total[m][i] = 0.0;
            for (int k0 = 0; k0 < K; k0 += kAhead) {
                f32x4 av[kAhead / 4], wv[NM][kAhead];
#pragma unroll
                for (int q = 0; q < kAhead / 4; ++q) av[q] = *reinterpret_cast<const f32x4*>(a + k0 + 4 * q);
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int q = 0; q < kAhead; ++q) wv[m][q] = *reinterpret_cast<const f32x4*>((m == 0 ? W0 : W1) + static_cast<size_t>(k0 + q) * N + n0 + col);
                asm volatile("" : : : "memory");
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int i = 0; i < 4; ++i) total[m][i] = fma(static_cast<double>(av[q / 4][q % 4]), static_cast<double>(wv[m][q][i]), total[m][i]);
            }
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!(fabsf(sum[m][i]) <= 3.402823466e38f)) sum[m][i] = static_cast<float>(total[m][i]);
        }
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = GATED ? act_f32(sum[0][i], act) * sum[NM - 1][i] : sum[0][i];
        const int at = row_begin + r, row = direct ? sh_row[at] : at;
        *reinterpret_cast<f32x4*>(C + static_cast<size_t>(row_map != nullptr ? row_map[row] : row) * N + n0 + col) = o;
    }
}

// GATED: C = act(A B0) * (A B1), else C = A B0.  gather (may be NULL): row r of the batched order is row gather[r] / gather_k
// of A; row_map (may be NULL): row r is written to row row_map[r] of C.  idx (may be NULL): nothing has batched the assignments.
template <bool GATED, bool NARROW>
__global__ __launch_bounds__(256, 2) void ffn_f32_kernel(const float* A, const int32_t* __restrict__ offsets, int e_first, int e_count, const float* W,
                                                         size_t expert_stride_elems, size_t off_b0, size_t off_b1, float* C, int K, int N, int act,
                                                         int total_rows, const int32_t* __restrict__ gather, int gather_k,
                                                         const int32_t* __restrict__ row_map, const int32_t* __restrict__ idx, int E, int tile_rows) {
    __shared__ __align__(16) float part[4][kRows * kPartRow];
    __shared__ int sh_row[kDirectRows];
    int e, row_begin = 0, rows;
    const bool direct = idx != nullptr;
    if (direct) {
        if (!find_tile_direct(idx, total_rows, E, tile_rows, blockIdx.y, sh_row, e, rows)) return;
    } else {
        if (!find_tile(offsets, e_first, e_count, tile_rows, blockIdx.y, total_rows, e, row_begin, rows)) return;
    }
    const int n0 = blockIdx.x * 16 * lane_columns(GATED, NARROW);
    const float* Wb = W + static_cast<size_t>(e - e_first) * expert_stride_elems;
    const int blocks = __builtin_amdgcn_readfirstlane((rows + 15) >> 4);
#define MOE_F32_TILE(RB)                                                                                                              \
    case RB:                                                                                                                          \
        ffn_f32_tile<GATED, NARROW, RB>(A, gather, gather_k, direct, sh_row, row_begin, rows, Wb + off_b0, Wb + off_b1, C, K, N, n0, act, row_map, part); \
        break;
    switch (blocks) { MOE_F32_TILE(1) MOE_F32_TILE(2) MOE_F32_TILE(3) MOE_F32_TILE(4) }
#undef MOE_F32_TILE
}

}  // namespace

int launch_expert_ffn_f32(const moe_cfg& c, const float* Xp, const int32_t* offsets, int e_first, int e_count, const float* W,
                          size_t expert_stride_elems, long max_rows, float* H, float* Yp, hipStream_t s, hipEvent_t between,
                          const int32_t* row_map, const int32_t* gather, const int32_t* idx) {
    const size_t df = static_cast<size_t>(c.d) * c.f;
    if (max_rows / kRows + e_count > 65535) return fail(MOE_ERR_UNSUPPORTED, "too many row tiles for one launch (%ld)", max_rows / kRows + e_count);
    int dev = 0;
    const DeviceInfo* info = nullptr;
    if (int rc = device_info(&dev, &info)) return rc;
    // Blocks of half the columns when there are too few for the compute units.  us, wide / half, by the wide blocks likely: up-projection 64 (191 x 2, d 512,
    // f 256, 8 experts) 35.8 / 32.3, 90 (239 x 1, d 576, f 576, 5) 40.7 / 37.8, 110 (22 x 1, d 576, f 704, 5) 30.5 / 31.5, 160 (22 x 2, d 1024, f 1024, 5) 43.0 / 49.1,
    // 240 (31 x 1, d 640, f 960, 8) 36.6 / 40.5; down-projection 96 (300 x 1, d 768, f 1600, 8) 68.6 / 61.0, 128 (200 x 1, d 1024, f 2048, 8) 79.7 / 70.8, 160
    // (700 x 1, d 1024, f 1024, 8) 76.8 / 78.4, 240 (968 x 1, d 1024, f 384, 8) 60.1 / 63.0.
    const long likely = max_rows / kRows > e_count ? max_rows / kRows : e_count < max_rows ? e_count : max_rows;
    const bool up_narrow = 5 * likely * (c.f / 32) < 2L * info->compute_units, down_narrow = 5 * likely * (c.d / 64) < 3L * info->compute_units;
    // Tiles of 32 or 16 rows where those give no more blocks than run at once, for experts of two standard deviations above the mean (tiles
    // of the mean would often leave a few rows over): a wave then has less to do in each
    // step of a chain that nothing else hides.  us, 64 / 32 / 16 rows in the down-projection: 117 x 1, d 256, f 3136, 4 experts 50.9 / 47.0 / 43.0, 242 x 2,
    // d 192, f 2752, 4 66.8 / 59.0 / 55.7, 201 x 2, d 576, f 2240, 4 72.9 / 68.4 / 71.9, 239 x 1, d 576, f 576, 5 37.7 / 37.3 / 39.5, 216 x 2, d 640, f 960, 8
    // 53.8 / 57.3 / 61.3.  The up-projection, whose reductions are shorter, has less to gain: 185 x 1, d 704, f 320, 4 32.7 / 32.6 / 33.5, 31 x 2, d 512, f 704, 4
    // 25.5 / 25.1 / 28.6.
    const long hit = e_count < max_rows ? e_count : max_rows;
    const double mean = static_cast<double>(max_rows) / hit;
    const long most = static_cast<long>(mean + 2.0 * sqrt(mean));
    auto tile_rows = [&](long columns, long limit) {
        int rows = kRows;
        while (rows > 16 && hit * ((most + rows / 2 - 1) / (rows / 2)) * columns <= limit) rows /= 2;
        return rows;
    };
    const int up_rows = tile_rows(c.f / 16, info->compute_units * 3L / 4), down_rows = tile_rows(c.d / 32, info->compute_units * 9L / 8);
    const dim3 block(256);
    auto up = [&](auto kernel, int columns) {
        hipLaunchKernelGGL(kernel, dim3(c.f / columns, static_cast<unsigned>(max_rows / up_rows + e_count)), block, 0, s, Xp, offsets, e_first, e_count, W,
                           expert_stride_elems, size_t(0), df, H, c.d, c.f, c.act, c.T * c.k, gather, c.k, static_cast<const int32_t*>(nullptr), idx, c.E,
                           up_rows);
    };
    if (up_narrow) up(ffn_f32_kernel<true, true>, 16);
    else up(ffn_f32_kernel<true, false>, 32);
    MOE_LAUNCH_CHECK("ffn_f32_kernel<up>");
    if (between != nullptr) MOE_HIP_CHECK(hipEventRecord(between, s));
    auto down = [&](auto kernel, int columns) {
        hipLaunchKernelGGL(kernel, dim3(c.d / columns, static_cast<unsigned>(max_rows / down_rows + e_count)), block, 0, s, H, offsets, e_first, e_count, W,
                           expert_stride_elems, 2 * df, 2 * df, Yp, c.f, c.d, c.act, c.T * c.k, static_cast<const int32_t*>(nullptr), 1, row_map, idx, c.E,
                           down_rows);
    };
    if (down_narrow) down(ffn_f32_kernel<false, true>, 32);
    else down(ffn_f32_kernel<false, false>, 64);
    MOE_LAUNCH_CHECK("ffn_f32_kernel<down>");
    return MOE_OK;
}

}  // namespace moe
