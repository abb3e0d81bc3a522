// fp32 expert feed-forward networks (the same grouped products as ffn.hip, on row-major fp32 weights):
//
//     H  = act(Xp W_gate[e]) * (Xp W_in[e])        "up",   epilogue fused
//     Yp = H W_out[e]                               "down"
//
// on the fp32 matrix instruction 32x32x2, whose products and sums are fp32 fused multiply-adds.
#include "common.h"

namespace moe {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

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
    // the expert's rows are split evenly over its tiles (in multiples of 32 rows), not into full tiles
    // and a small remainder: equal tiles finish together and none is nearly empty
    const int lo = seg_lo(e_out), hi = seg_hi(e_out), n = hi - lo;
    const int tiles = (n + tile_m - 1) / tile_m;
    const int per_tile = min(tile_m, ((n + tiles - 1) / tiles + 31) & ~31);
    row_begin = lo + sh_mt * per_tile;
    rows = min(per_tile, hi - row_begin);
    return true;
}

// The same for at most kDirectRows assignments that nothing has batched: the experts in the order of their first assignments, row r of an expert
// is assignment sh_row[row_begin + r].
__device__ inline bool find_tile_direct(const int32_t* __restrict__ idx, int A, int E, int tile_m, int slot, int (&sh_row)[kDirectRows], int& e_out,
                                        int& row_begin, int& rows) {
    __shared__ int sh_e, sh_mt, sh_n;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int expert;
        const unsigned long long peers = direct_peers(idx, A, E, lane, expert), below = (1ull << lane) - 1ull;
        const bool first = peers != 0ull && (peers & below) == 0ull;
        const int tiles = (__popcll(peers) + tile_m - 1) / tile_m;         // one or two
        const unsigned long long two = __ballot(first && tiles == 2);
        const int start = __popcll(__ballot(first) & below) + __popcll(two & below);
        const unsigned long long found = __ballot(first && start <= slot && slot < start + tiles);
        if (found == 0ull) {
            if (lane == 0) sh_e = -1;
        } else {
            const int leader = __ffsll(static_cast<long long>(found)) - 1;
            if (lane == leader) { sh_e = expert; sh_mt = slot - start; sh_n = __popcll(peers); }
            if (peers != 0ull && (peers >> leader) & 1ull) sh_row[__popcll(peers & below)] = lane;
        }
    }
    __syncthreads();
    if (sh_e < 0) return false;
    e_out = sh_e;
    const int tiles = (sh_n + tile_m - 1) / tile_m, per_tile = min(tile_m, ((sh_n + tiles - 1) / tiles + 31) & ~31);
    row_begin = sh_mt * per_tile;
    rows = min(per_tile, sh_n - row_begin);
    return true;
}

// What bounds it: the matrix instruction (157 TFLOP/s) once there are enough blocks, the latency of the steps of one block
// in short launches.  The kernel it replaces (vector multiply-adds, scalar loads, no load in flight across steps) ran at
// 18 TFLOP/s.  Whole layer before -> after, with the rows read and written through the permutation: 64 tokens, d 256, f 512,
// 4 experts 144 -> 23 us; 512 tokens x 2, d 1024, f 4096, 8 experts 1386 -> 340 to
// 365 us by the rows per expert.
// Two shapes of a block (four waves, each with 32 x 32 output tiles, twice that when GATED):
//   wide   64 rows x 64 columns, a wave per quarter, 32 reduction elements per step
//   split  32 rows x 32 columns, all four waves on the same tile, each with a quarter of the reduction dimension, 16
//          elements per step; the four partial tiles are added in wave order at the end
// The wide shape adds up the same four quarters one after the other, so that both give the same bits and a row's result does
// not depend on the batch it came in (d 1024, f 4096, 8 experts, k 2, one sum over the whole dimension -> four quarters: 512
// tokens 334 -> 340 us, 2048 tokens 1037 -> 1046).
// Both stage the activations ([row][k]) and the weights ([k][column]) of a step through LDS, double buffered, one barrier
// per step; the global loads of a step are issued kAhead steps earlier into registers.  Row strides in LDS are chosen so
// that the 16-byte activation reads and the 4-byte weight reads of a wave touch every bank once.
template <bool SPLIT>
struct Shape {
    static constexpr int BM = SPLIT ? 32 : 64, BN = SPLIT ? 32 : 64, KC = SPLIT ? 64 : 32;
    static constexpr int kAhead = SPLIT ? 3 : 2;
    static constexpr int kWaveK = SPLIT ? KC / 4 : KC;          // reduction elements of a step one wave multiplies
    static constexpr int kStride = kWaveK;                      // elements from one step to the next
    static constexpr int kARow = KC + 4, kBRow = BN + 8;        // floats per LDS row
};

// GATED: C = act(A B0) * (A B1), else C = A B0.  gather (may be NULL): row r of the batched order is row gather[r] / gather_k
// of A; row_map (may be NULL): row r is written to row row_map[r] of C.
template <bool GATED, bool SPLIT>
__global__ __launch_bounds__(256, 2) void ffn_f32_kernel(const float* __restrict__ A, const int32_t* __restrict__ offsets,
                                                         int e_first, int e_count, const float* __restrict__ W,
                                                         size_t expert_stride_elems, size_t off_b0, size_t off_b1,
                                                         float* __restrict__ C, int K, int N, int act, int total_rows,
                                                         const int32_t* __restrict__ gather, int gather_k,
                                                         const int32_t* __restrict__ row_map, const int32_t* __restrict__ idx, int E) {
    using S = Shape<SPLIT>;
    constexpr int NB = GATED ? 2 : 1;
    constexpr int kAFloats = S::BM * S::kARow, kBFloats = S::KC * S::kBRow, kBuf = kAFloats + NB * kBFloats;
    __shared__ __align__(16) float lds[2][kBuf];
    int e, row_begin, rows;
    __shared__ int sh_row[kDirectRows];
    const bool direct = idx != nullptr;
    if (direct) {
        if (!find_tile_direct(idx, total_rows, E, S::BM, blockIdx.y, sh_row, e, row_begin, rows)) return;
    } else {
        if (!find_tile(offsets, e_first, e_count, S::BM, blockIdx.y, total_rows, e, row_begin, rows)) return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n0 = blockIdx.x * S::BN;
    const float* Wb[NB];
    Wb[0] = W + static_cast<size_t>(e - e_first) * expert_stride_elems + off_b0 + n0;
    if (GATED) Wb[NB - 1] = W + static_cast<size_t>(e - e_first) * expert_stride_elems + off_b1 + n0;

    // this thread's two 16-byte pieces of the activation tile and of every weight tile
    constexpr int kAVec = S::KC / 4, kBVec = S::BN / 4;          // pieces per row
    const float* a_src[2];
    int a_dst[2], b_dst[2];
    size_t b_src[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int id = tid + i * 256;
        const int r = id / kAVec, at = row_begin + min(r, rows - 1);       // rows past the end repeat the last one, not stored
        const int row = direct ? sh_row[at] : at;
        const size_t src = GATED && direct ? static_cast<size_t>(row / gather_k) : gather != nullptr ? static_cast<size_t>(gather[row] / gather_k) : static_cast<size_t>(row);
        // (SPLIT: element 16 w + n of a step is element n of the step in quarter w)
        a_src[i] = A + src * K + (SPLIT ? id % kAVec / 4 * (K / 4) + 4 * (id % 4) : 4 * (id % kAVec));
        a_dst[i] = r * S::kARow + 4 * (id % kAVec);
        b_src[i] = static_cast<size_t>(SPLIT ? id / kBVec / 16 * (K / 4) + id / kBVec % 16 : id / kBVec) * N + 4 * (id % kBVec);
        b_dst[i] = kAFloats + (id / kBVec) * S::kBRow + 4 * (id % kBVec);
    }
    f32x4 ra[S::kAhead][2], rb[S::kAhead][NB][2];
    const int steps = K / S::KC;
    auto fetch = [&](int q, int step) {
        const int c = min(step, steps - 1);                               // past the end: the last step again, unused
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ra[q][i] = *reinterpret_cast<const f32x4*>(a_src[i] + c * S::kStride);
#pragma unroll
            for (int b = 0; b < NB; ++b)
                rb[q][b][i] = *reinterpret_cast<const f32x4*>(Wb[b] + static_cast<size_t>(c) * S::kStride * N + b_src[i]);
        }
    };
    // the wave's place in the tile: rows and columns, or (SPLIT) its part of the reduction elements of a step
    const int wrow = SPLIT ? 0 : 32 * (wave >> 1), wcol = SPLIT ? 0 : 32 * (wave & 1), wk = SPLIT ? wave * S::kWaveK : 0;
    const int h = lane >> 5, c31 = lane & 31;
    f32x16 acc[NB], total[NB];                   // the quarter at hand; the quarters before it (not SPLIT)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = total[b][v] = 0.f;
    int quarter_end = K / 4;
#pragma unroll
    for (int q = 0; q < S::kAhead; ++q) fetch(q, q);
    for (int s0 = 0; s0 < steps; s0 += S::kAhead) {
#pragma unroll
        for (int q = 0; q < S::kAhead; ++q) {
            const int s = s0 + q;
            if (s >= steps) break;                                        // uniform
            float* buf = lds[s & 1];         // its last readers passed the barrier of the step before
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                *reinterpret_cast<f32x4*>(buf + a_dst[i]) = ra[q][i];
#pragma unroll
                for (int b = 0; b < NB; ++b) *reinterpret_cast<f32x4*>(buf + b_dst[i] + b * kBFloats) = rb[q][b][i];
            }
            fetch(q, s + S::kAhead);
            __syncthreads();
            const float* pa = buf + (wrow + c31) * S::kARow + wk + 4 * h;
            const float* pb = buf + kAFloats + (wk + 4 * h) * S::kBRow + wcol + c31;
            // eight reduction elements at a time: lanes 0..31 hold the first four, lanes 32..63 the others; those of the next eight are
            // read before the products of these
            constexpr int kG = S::kWaveK / 8;
            f32x4 av[kG];
            float bv[kG][NB][4];
            auto read = [&](int g) __attribute__((always_inline)) {
                av[g] = *reinterpret_cast<const f32x4*>(pa + 8 * g);
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) bv[g][b][i] = pb[b * kBFloats + (8 * g + i) * S::kBRow];
            };
            read(0);
#pragma unroll
            for (int g = 0; g < kG; ++g) {
                if (g + 1 < kG) read(g + 1);
                if (!SPLIT && g % 2 == 0 && s * S::KC + 8 * g == quarter_end) {       // uniform (a quarter is a multiple of 16)
                    quarter_end += K / 4;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        total[b] += acc[b];
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[g][b][i], av[g][i], acc[b], 0, 0, 0);
            }
        }
    }
    // the weights are the first operand: lane l holds token row l % 32 and, in v = 4 g .. 4 g + 3, columns 8 g + 4 (l / 32) + 0..3
    auto value = [&](float gate, float in) { return GATED ? act_f32(gate, act) * in : gate; };
    auto out_at = [&](int r, int col) {
        const int row = direct ? sh_row[row_begin + r] : row_begin + r;
        return reinterpret_cast<f32x4*>(C + static_cast<size_t>(row_map != nullptr ? row_map[row] : row) * N + n0 + col);
    };
    if constexpr (!SPLIT) {
#pragma unroll
        for (int b = 0; b < NB; ++b) total[b] += acc[b];
        if (wrow + c31 < rows) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 o;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = value(total[0][4 * g + i], total[NB - 1][4 * g + i]);
                *out_at(wrow + c31, wcol + 8 * g + 4 * h) = o;
            }
        }
    } else {
        constexpr int kPRow = 36;                                         // floats per row of a partial tile
        static_assert(4 * NB * 32 * kPRow <= 2 * kBuf, "the partial tiles fit the staging buffers");
        float* part = &lds[0][0];
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f32x4*>(part + ((wave * NB + b) * 32 + c31) * kPRow + 8 * g + 4 * h) =
                    f32x4{acc[b][4 * g], acc[b][4 * g + 1], acc[b][4 * g + 2], acc[b][4 * g + 3]};
        __syncthreads();
        const int r = tid >> 3, col = 4 * (tid & 7);
        f32x4 sum[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            sum[b] = *reinterpret_cast<const f32x4*>(part + (b * 32 + r) * kPRow + col);
#pragma unroll
            for (int w = 1; w < 4; ++w) sum[b] += *reinterpret_cast<const f32x4*>(part + ((w * NB + b) * 32 + r) * kPRow + col);
        }
        if (r < rows) {
            f32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = value(sum[0][i], sum[NB - 1][i]);
            *out_at(r, col) = o;
        }
    }
}

}  // namespace

int launch_expert_ffn_f32(const moe_cfg& c, const float* Xp, const int32_t* offsets, int e_first, int e_count, const float* W,
                          size_t expert_stride_elems, long max_rows, float* H, float* Yp, hipStream_t s, hipEvent_t between,
                          const int32_t* row_map, const int32_t* gather, const int32_t* idx) {
    const size_t df = static_cast<size_t>(c.d) * c.f;
    int dev = 0;
    const DeviceInfo* info = nullptr;
    if (int rc = device_info(&dev, &info)) return rc;
    // Which shape: by the layer's own sizes, not the launch's, so that a launch over one expert sums like a launch over all.
    const long rows = static_cast<long>(c.T) * c.k;
    auto split_for = [&](int N) {
        const long tiles = rows / 64 > c.E ? rows / 64 : c.E;
        return tiles * (N / 64) < 2L * info->compute_units;
    };
    auto grid_for = [&](bool split, int N) {
        const int bm = split ? 32 : 64;
        return dim3(N / bm, static_cast<unsigned>(max_rows / bm + e_count));
    };
    if (max_rows / 64 + e_count > 65535) return fail(MOE_ERR_UNSUPPORTED, "too many row tiles for one launch (%ld)", max_rows / 64 + e_count);
    const bool up_split = split_for(c.f), down_split = split_for(c.d);
    const dim3 block(256);
    if (up_split)
        hipLaunchKernelGGL((ffn_f32_kernel<true, true>), grid_for(true, c.f), block, 0, s, Xp, offsets, e_first, e_count, W,
                           expert_stride_elems, size_t(0), df, H, c.d, c.f, c.act, c.T * c.k, gather, c.k,
                           static_cast<const int32_t*>(nullptr), idx, c.E);
    else
        hipLaunchKernelGGL((ffn_f32_kernel<true, false>), grid_for(false, c.f), block, 0, s, Xp, offsets, e_first, e_count, W,
                           expert_stride_elems, size_t(0), df, H, c.d, c.f, c.act, c.T * c.k, gather, c.k,
                           static_cast<const int32_t*>(nullptr), idx, c.E);
    MOE_LAUNCH_CHECK("ffn_f32_kernel<up>");
    if (between != nullptr) MOE_HIP_CHECK(hipEventRecord(between, s));
    if (down_split)
        hipLaunchKernelGGL((ffn_f32_kernel<false, true>), grid_for(true, c.d), block, 0, s, H, offsets, e_first, e_count, W,
                           expert_stride_elems, 2 * df, 2 * df, Yp, c.f, c.d, c.act, c.T * c.k,
                           static_cast<const int32_t*>(nullptr), 1, row_map, idx, c.E);
    else
        hipLaunchKernelGGL((ffn_f32_kernel<false, false>), grid_for(false, c.d), block, 0, s, H, offsets, e_first, e_count, W,
                           expert_stride_elems, 2 * df, 2 * df, Yp, c.f, c.d, c.act, c.T * c.k,
                           static_cast<const int32_t*>(nullptr), 1, row_map, idx, c.E);
    MOE_LAUNCH_CHECK("ffn_f32_kernel<down>");
    return MOE_OK;
}

}  // namespace moe
