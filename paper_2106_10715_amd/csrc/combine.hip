// Weighted un-permute (CPM-2 Section 2.1: the selected experts' outputs stand in for the FFN
// output of the token): y[t] = sum_j w[t, j] * Yp[inv[t*k + j]], fp32 sum in slot order, one
// rounding to the storage type.  One block per token, 16-byte vectors, coalesced on both sides.
#include "common.h"

namespace moe {
namespace {

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
__device__ inline uint32_t pack_bf16(float lo, float hi) {
    const uint16_t a = __builtin_bit_cast(uint16_t, static_cast<__bf16>(lo));
    const uint16_t b = __builtin_bit_cast(uint16_t, static_cast<__bf16>(hi));
    return a | (static_cast<uint32_t>(b) << 16);
}

// Bound by memory; a thread's pieces of all K rows are requested before the first is used, U positions of the row at a time.
// NT: non-temporal loads, where the rows and y are more than the last-level cache holds.
// DIRECT: there is no inv, row a of Yp is assignment a (known to the compiler: the K look-ups are else issued one after the other).
template <bool BF16, int K, int U, bool NT, bool DIRECT>
__global__ __launch_bounds__(256) void combine_kernel(const uint4* __restrict__ Yp, const int32_t* __restrict__ inv,
                                                      const float* __restrict__ w, uint4* __restrict__ y,
                                                      int vec_per_row, int n_rows) {
    typedef unsigned int u4v __attribute__((ext_vector_type(4)));
    const int t = blockIdx.x;
    const u4v* rows[K];
    float wt[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int row = DIRECT ? t * K + j : min(max(inv[static_cast<size_t>(t) * K + j], 0), n_rows - 1);   // never outside Yp
        rows[j] = reinterpret_cast<const u4v*>(Yp) + static_cast<size_t>(row) * vec_per_row;
        wt[j] = w[static_cast<size_t>(t) * K + j];
    }
    for (int v0 = threadIdx.x; v0 < vec_per_row; v0 += 256 * U) {
        u4v u[U][K];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int v = min(v0 + 256 * i, vec_per_row - 1);
#pragma unroll
            for (int j = 0; j < K; ++j) u[i][j] = NT ? __builtin_nontemporal_load(rows[j] + v) : rows[j][v];
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            float acc[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = 0.f;
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (BF16) {
                        acc[2 * c] = fmaf(wt[j], bf16_lo(u[i][j][c]), acc[2 * c]);
                        acc[2 * c + 1] = fmaf(wt[j], bf16_hi(u[i][j][c]), acc[2 * c + 1]);
                    } else {
                        acc[c] = fmaf(wt[j], __uint_as_float(u[i][j][c]), acc[c]);
                    }
                }
            uint4 o;
            if (BF16) {
                o.x = pack_bf16(acc[0], acc[1]); o.y = pack_bf16(acc[2], acc[3]);
                o.z = pack_bf16(acc[4], acc[5]); o.w = pack_bf16(acc[6], acc[7]);
            } else {
                o.x = __float_as_uint(acc[0]); o.y = __float_as_uint(acc[1]);
                o.z = __float_as_uint(acc[2]); o.w = __float_as_uint(acc[3]);
            }
            if (v0 + 256 * i < vec_per_row) y[static_cast<size_t>(t) * vec_per_row + v0 + 256 * i] = o;
        }
    }
}

// Two positions per thread for up to four rows, where rows are longer than one position of all threads (with fewer, half the
// requests are for nothing).  Non-temporal loads beyond 320 MB of rows and y together, us plain / non-temporal: 16384 tokens x 2,
// d 4096 (403 MB) 76.6 / 62.0, 9000 x 4 (369 MB) 71.3 / 62.6, 8000 x 8 (590 MB) 117 / 102; 8192 x 8, d 1024 fp32 (302 MB)
// 46.7 / 53.3, 16384 x 1, d 4096 (268 MB) 39.5 / 40.9, 4000 x 2 (98 MB) 15.5 / 16.9.
template <bool BF16, int K>
void launch_k(const moe_cfg& c, const uint4* Yp, const int32_t* inv, const float* w, uint4* y, int vec_per_row, hipStream_t s) {
    constexpr int kTwo = K <= 4 ? 2 : 1;
    const bool two = vec_per_row > 256, nt = static_cast<size_t>(c.T) * (c.k + 1) * vec_per_row * 16 > (size_t(320) << 20);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(c.T), dim3(256), 0, s, Yp, inv, w, y, vec_per_row, c.T * c.k); };
    if (inv == nullptr) two ? run(combine_kernel<BF16, K, kTwo, false, true>) : run(combine_kernel<BF16, K, 1, false, true>);      // at most kDirectRows rows
    else if (two && nt) run(combine_kernel<BF16, K, kTwo, true, false>);
    else if (two) run(combine_kernel<BF16, K, kTwo, false, false>);
    else if (nt) run(combine_kernel<BF16, K, 1, true, false>);
    else run(combine_kernel<BF16, K, 1, false, false>);
}

template <bool BF16>
void launch_for_k(const moe_cfg& c, const uint4* Yp, const int32_t* inv, const float* w, uint4* y, int vec_per_row, hipStream_t s) {
#define MOE_COMBINE(K) \
    case K: launch_k<BF16, K>(c, Yp, inv, w, y, vec_per_row, s); break;
    switch (c.k) {
        MOE_COMBINE(1) MOE_COMBINE(2) MOE_COMBINE(3) MOE_COMBINE(4) MOE_COMBINE(5) MOE_COMBINE(6) MOE_COMBINE(7) MOE_COMBINE(8)
    }
#undef MOE_COMBINE
}

}  // namespace

int launch_combine(const moe_cfg& c, const void* Yp, const int32_t* inv, const float* w, void* y, hipStream_t s) {
    if (c.T == 0) return MOE_OK;
    const int vec_per_row = static_cast<int>(c.d * elem_size(c) / 16);
    if (c.dtype == MOE_BF16)
        launch_for_k<true>(c, static_cast<const uint4*>(Yp), inv, w, static_cast<uint4*>(y), vec_per_row, s);
    else
        launch_for_k<false>(c, static_cast<const uint4*>(Yp), inv, w, static_cast<uint4*>(y), vec_per_row, s);
    MOE_LAUNCH_CHECK("combine_kernel");
    return MOE_OK;
}

}  // namespace moe
