// Batching of assignments by expert (CPM-2 Section 6.2: tokens are routed and batched to their
// experts before computation): a deterministic, stable counting sort of a = t*k + j by expert id,
// followed by the row copy Xp[row] = x[perm[row] / k].
//
//   1. chunk_hist_kernel : LDS histogram of each chunk of kPermChunk assignments
//   2. scan_kernel       : counts, offsets and, per chunk, the first row of every expert
//   3. scatter_kernel    : stable rank inside the chunk from wave ballots (no ordered atomics)
//      (up to 65536 assignments batch_kernel is all three)
//   4. gather_rows_kernel: 16-byte-vector row copy
#include "common.h"
#include "ffn_plan.h"

#include <mutex>

// Scratch of moe_permute_static, the variant of moe_permute for callers that can neither allocate nor pass a
// workspace: the per-chunk expert histograms / running bases of the chunked kernels, [chunks][E] int32, for
// up to kStaticChunks chunks of kPermChunk assignments and 256 experts.  Every device the library runs on
// holds its own copy of the array (256 KiB) until the process ends.  In host code the name is only a handle
// for hipGetSymbolAddress, never an address.
constexpr int kStaticChunks = 256;
constexpr int kStaticExperts = 256;
static __device__ __align__(256) int32_t scratch[kStaticChunks * kStaticExperts];

namespace moe {
namespace {

__device__ inline int clamp_expert(int e, int E) { return min(max(e, 0), E - 1); }

__global__ __launch_bounds__(256) void chunk_hist_kernel(const int32_t* __restrict__ idx, int A, int E,
                                                         int32_t* __restrict__ chunk_hist) {
    __shared__ int hist[256];
    hist[threadIdx.x] = 0;
    __syncthreads();
    const int a0 = blockIdx.x * kPermChunk;
    for (int i = threadIdx.x; i < kPermChunk; i += 256) {
        const int a = a0 + i;
        if (a < A) atomicAdd(&hist[clamp_expert(idx[a], E)], 1);   // integer counts: order cannot matter
    }
    __syncthreads();
    if (threadIdx.x < E) chunk_hist[static_cast<size_t>(blockIdx.x) * E + threadIdx.x] = hist[threadIdx.x];
}

// One block; thread e walks the chunks of expert e, turning histograms into running bases.  The chunk
// histograms are read kScanBatch at a time (independent loads: one memory latency per batch, not per chunk).
constexpr int kScanBatch = 16;

__global__ __launch_bounds__(256) void scan_kernel(int32_t* __restrict__ chunk_hist, int chunks, int E,
                                                   int32_t* __restrict__ counts, int32_t* __restrict__ offsets) {
    __shared__ int total[256];
    __shared__ int start[257];
    const int e = threadIdx.x;
    int run = 0;
    if (e < E) {
        for (int b0 = 0; b0 < chunks; b0 += kScanBatch) {
            int h[kScanBatch];
#pragma unroll
            for (int i = 0; i < kScanBatch; ++i)
                h[i] = b0 + i < chunks ? chunk_hist[static_cast<size_t>(b0 + i) * E + e] : 0;
#pragma unroll
            for (int i = 0; i < kScanBatch; ++i) run += h[i];
        }
    }
    total[e] = e < E ? run : 0;
    __syncthreads();
    if (e == 0) {
        int acc = 0;
        for (int i = 0; i < E; ++i) { start[i] = acc; acc += total[i]; }
        start[E] = acc;
    }
    __syncthreads();
    if (e < E) {
        counts[e] = total[e];
        offsets[e] = start[e];
        int base = start[e];                   // first row of expert e in the chunk at hand: its rows in earlier chunks come first
        for (int b0 = 0; b0 < chunks; b0 += kScanBatch) {
            int h[kScanBatch];
#pragma unroll
            for (int i = 0; i < kScanBatch; ++i)
                h[i] = b0 + i < chunks ? chunk_hist[static_cast<size_t>(b0 + i) * E + e] : 0;
#pragma unroll
            for (int i = 0; i < kScanBatch; ++i) {
                if (b0 + i < chunks) chunk_hist[static_cast<size_t>(b0 + i) * E + e] = base;
                base += h[i];
            }
        }
    }
    if (e == 0) offsets[E] = start[E];
}

__global__ __launch_bounds__(256) void scatter_kernel(const int32_t* __restrict__ idx, int A, int E,
                                                      const int32_t* __restrict__ chunk_base,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ inv) {
    __shared__ int run[256];          // next free row of each expert for this chunk
    __shared__ int wcnt[4][256];      // per wave, rows each expert takes in the current round
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    run[threadIdx.x] = threadIdx.x < E ? chunk_base[static_cast<size_t>(blockIdx.x) * E + threadIdx.x] : 0;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) wcnt[wv][threadIdx.x] = 0;
    __syncthreads();
    int bits = 0;
    while ((1 << bits) < E) ++bits;
    const int a0 = blockIdx.x * kPermChunk;
    for (int round = 0; round < kPermChunk / 256; ++round) {
        const int a = a0 + round * 256 + threadIdx.x;
        const bool valid = a < A;
        const int e = valid ? clamp_expert(idx[a], E) : 0;
        // lanes of this wave that hold the same expert
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (e >> b) & 1;
            const unsigned long long bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        if (valid && rank == 0) wcnt[wave][e] = __popcll(peers);
        __syncthreads();
        if (valid) {
            int row = run[e] + rank;
            for (int wv = 0; wv < wave; ++wv) row += wcnt[wv][e];
            perm[row] = a;
            inv[a] = row;
        }
        __syncthreads();
        {
            const int t = threadIdx.x;
            run[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
            wcnt[0][t] = 0; wcnt[1][t] = 0; wcnt[2][t] = 0; wcnt[3][t] = 0;
        }
        __syncthreads();
    }
}

// Up to kOneLaunchMaxA assignments: the same in one launch.  Every block reads all of idx and counts, beside the totals, what lies
// before its own kPermChunk assignments, so that no block needs anything of another.  The work list of the expert kernels that follow, when the caller wants it from here
// (saves a launch), is made by a block of its own, or by two when the down kernel does not read the up kernel's list.  Bound by the latency of its few steps (launch, the read of idx, counting, scan, stores):
// every assignment is counted by every block, which takes longer than the three kernels above only far beyond the limit.  us, against one block in
// rounds of 1024 (up to 16384) and the three kernels (beyond): 2050 assignments to 33 experts with the list 8.5 -> 5.0, 32768 to 64 experts without
// 14.7 -> 6.7; whole calls: 4096 tokens on 32 experts 1346 -> 1317, 60000 x 1, d 1024, f 64, 8 experts (a list by a kernel of its own before) 196.8 -> 194.7.
constexpr int kBatchWaves = kPermChunk / 64;           // one assignment of the block's own chunk per thread
// Histograms the counting is spread over (equal experts in a wave wait for each other, and so do different ones in one bank: hence the odd row).  A
// short batch has less to count than to clear and add up.  Kernel us, three kernels / four copies in one bank / as here: 65536 assignments to one expert
// 12.0 / 30.8 / 8.6, half of 65536 to one of 64 14.5 / 19.3 / 10.0, 65536 spread over 64 14.3 / 9.0 / 9.0, 32768 to one 10.3 / 17.3 / 7.6, spread over 64
// 12.3 / 6.5 / 6.7 (with 16 copies 7.0), 8193 over 32 - / 4.8 / 5.1 (5.5).
constexpr int kCopies = 16, kHistRow = 257;
__device__ inline int copies_for(int A) { return A <= 8192 ? 4 : A <= 32768 ? 8 : kCopies; }
constexpr int kOneLaunchMaxA = 64 * kPermChunk;

__global__ __launch_bounds__(kPermChunk) void batch_kernel(const int32_t* __restrict__ idx, int A, int E, int chunks,
                                                           int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                           int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                                           int32_t* __restrict__ plan, int plan_max_tiles, int plan_tile_rows,
                                                           int plan_tile_rows_down) {
    __shared__ int hist[2][kCopies][kHistRow];         // assignments before the block's chunk, and from there on
    __shared__ __align__(16) int wcnt[kBatchWaves][256];     // per wave, rows each expert takes
    __shared__ int run[256], start[257];               // first row of each expert, of the chunk's and of all
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool plans = static_cast<int>(blockIdx.x) >= chunks;
    const int a0 = plans ? 0 : blockIdx.x * kPermChunk, a = a0 + tid;
    const bool valid = !plans && a < A;
    const int mine = valid ? clamp_expert(idx[a], E) : 0;
    const int copies = copies_for(A);
    for (int i = tid; i < copies * kHistRow; i += kPermChunk) (&hist[0][0][0])[i] = (&hist[1][0][0])[i] = 0;
    for (int i = tid; i < kBatchWaves * 256; i += kPermChunk) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    // integer counts: order cannot matter
    auto count = [&](int at, int e) { atomicAdd(&hist[at >= a0 ? 1 : 0][lane & (copies - 1)][clamp_expert(e, E)], 1); };
    if ((reinterpret_cast<uintptr_t>(idx) & 15) == 0) {                    // uniform
        const int whole = A / 4;
        for (int q0 = tid; q0 < whole; q0 += 4 * kPermChunk) {
            int4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const int4*>(idx)[min(q0 + u * kPermChunk, whole - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int at = 4 * (q0 + u * kPermChunk);                  // (a chunk starts at a multiple of 4)
                if (q0 + u * kPermChunk < whole) { count(at, v[u].x); count(at, v[u].y); count(at, v[u].z); count(at, v[u].w); }
            }
        }
        if (tid < (A & 3)) count(4 * whole + tid, idx[4 * whole + tid]);
    } else {
        for (int at = tid; at < A; at += kPermChunk) count(at, idx[at]);
    }
    // the block's own chunk: lanes of this wave that hold the same expert
    int rank = 0;
    if (!plans) {                                                          // uniform
        int bits = 0;
        while ((1 << bits) < E) ++bits;
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            const bool bit = (mine >> b) & 1;
            const unsigned long long bal = __ballot(bit);
            peers &= bit ? bal : ~bal;
        }
        rank = __popcll(peers & ((1ull << lane) - 1ull));
        if (valid && rank == 0) wcnt[wave][mine] = __popcll(peers);
    }
    __syncthreads();
    if (wave == 0) {
        // exclusive scan of up to 256 counts by one wave: four experts per lane, then across the lanes
        int c[4] = {0, 0, 0, 0}, before[4] = {0, 0, 0, 0}, sum = 0;
        for (int q0 = 0; q0 < copies; q0 += 4)         // uniform
#pragma unroll
            for (int q = q0; q < q0 + 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) { before[j] += hist[0][q][4 * lane + j]; c[j] += hist[1][q][4 * lane + j]; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c[j] += before[j];
            sum += c[j];
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        int at = incl - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 4 * lane + j;
            if (blockIdx.x == 0 && e < E) { counts[e] = c[j]; offsets[e] = at; }
            start[e] = at;
            run[e] = at + before[j];
            at += c[j];
        }
        if (lane == 63) {                              // experts past E hold no assignment, so this is the total
            start[256] = incl;
            if (blockIdx.x == 0) offsets[E] = incl;
        }
    }
    __syncthreads();
    if (plans) {
        int (&scratch)[kPlanScratch][256] = reinterpret_cast<int (&)[kPlanScratch][256]>(wcnt);
        const int list = blockIdx.x - chunks;
        ffn_plan_block(start, 0, E, list == 0 ? plan_tile_rows : plan_tile_rows_down, plan, A, plan_max_tiles, scratch, list);
    } else if (valid) {
        int row = run[mine] + rank;
        for (int wv = 0; wv < wave; ++wv) row += wcnt[wv][mine];
        perm[row] = a;
        inv[a] = row;
    }
}

// One block per token: its row is read once and written to the batched rows of its k assignments (16-byte vectors, whole
// rows, coalesced on both sides).  Bound by memory; a thread requests U pieces, as many as rows are long, before it stores the
// first.  NT: x is read non-temporally, where it is more than the last-level cache holds; else the gate, or whoever wrote x, has
// left it there.  us non-temporal / plain, x in the cache if it fits: 8192 tokens x 1, d 1024 20.1 / 17.2; 16384 x 2, d 4096 85.1 /
// 70.7; 32000 x 1, d 4096 (262 MB) 103 / 87; 40000 x 1 (328 MB) 126 / 132, 65536 x 1 (537 MB) 201 / 212.
template <int U, bool NT>
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ x, const int32_t* __restrict__ inv,
                                                          int k, int vec_per_row, uint4* __restrict__ Xp) {
    // stored non-temporal: the rows are next read by the expert kernels, which want the L2 for themselves
    // (left there as dirty lines, the batch costs the up-projection 2.5 % at 128 tokens per expert)
    typedef unsigned int u4v __attribute__((ext_vector_type(4)));
    const size_t t = blockIdx.x;
    const u4v* src = reinterpret_cast<const u4v*>(x) + t * vec_per_row;
    u4v* dst = reinterpret_cast<u4v*>(Xp);
    for (int v0 = threadIdx.x; v0 < vec_per_row; v0 += 256 * U) {
        u4v piece[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const u4v* from = src + min(v0 + 256 * i, vec_per_row - 1);
            piece[i] = NT ? __builtin_nontemporal_load(from) : *from;
        }
        for (int j = 0; j < k; ++j) {
            const size_t row = inv[t * k + j];
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (v0 + 256 * i < vec_per_row) __builtin_nontemporal_store(piece[i], dst + row * vec_per_row + v0 + 256 * i);
        }
    }
}

}  // namespace

int launch_permute(const moe_cfg& c, const void* x, const int32_t* idx, int32_t* counts, int32_t* offsets,
                   int32_t* perm, int32_t* inv, void* Xp, int32_t* chunk_hist, hipStream_t s, int32_t* plan,
                   int plan_max_tiles, bool* planned, int plan_tile_rows, int plan_tile_rows_down) {
    if (planned != nullptr) *planned = false;
    const int A = c.T * c.k;
    const int chunks = (A + kPermChunk - 1) / kPermChunk;
    if (A <= kOneLaunchMaxA) {
        const bool with_plan = plan != nullptr && planned != nullptr && c.dtype == MOE_BF16 && A > 0;
        const int own = chunks > 0 ? chunks : 1;       // (no assignments: the counts are still written)
        hipLaunchKernelGGL(batch_kernel, dim3(own + (!with_plan ? 0 : plan_tile_rows_down != plan_tile_rows ? 2 : 1)), dim3(kPermChunk), 0, s, idx, A, c.E, own, counts, offsets, perm, inv,
                           with_plan ? plan : nullptr, plan_max_tiles, plan_tile_rows, plan_tile_rows_down);
        MOE_LAUNCH_CHECK("batch_kernel");
        if (with_plan) *planned = true;
    } else {
        if (chunk_hist == nullptr) return fail(MOE_ERR_WORKSPACE, "the batching of %d assignments needs scratch memory", A);
        hipLaunchKernelGGL(chunk_hist_kernel, dim3(chunks), dim3(256), 0, s, idx, A, c.E, chunk_hist);
        MOE_LAUNCH_CHECK("chunk_hist_kernel");
        hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(256), 0, s, chunk_hist, chunks, c.E, counts, offsets);
        MOE_LAUNCH_CHECK("scan_kernel");
        hipLaunchKernelGGL(scatter_kernel, dim3(chunks), dim3(256), 0, s, idx, A, c.E, chunk_hist, perm, inv);
        MOE_LAUNCH_CHECK("scatter_kernel");
    }
    if (chunks > 0) {
        if (Xp != nullptr) {
            const int vec_per_row = static_cast<int>(c.d * elem_size(c) / 16);
            auto run = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(c.T), dim3(256), 0, s, static_cast<const uint4*>(x), inv, c.k, vec_per_row, static_cast<uint4*>(Xp));
            };
            const bool nt = static_cast<size_t>(c.T) * vec_per_row * 16 > (size_t(288) << 20);
            if (vec_per_row <= 256) nt ? run(gather_rows_kernel<1, true>) : run(gather_rows_kernel<1, false>);
            else if (nt) run(gather_rows_kernel<4, true>);
            else vec_per_row <= 512 ? run(gather_rows_kernel<2, false>) : run(gather_rows_kernel<4, false>);
            MOE_LAUNCH_CHECK("gather_rows_kernel");
        }
    }
    return MOE_OK;
}

long permute_static_max_assignments() { return static_cast<long>(kStaticChunks) * kPermChunk; }

int launch_permute_static(const moe_cfg& c, const void* x, const int32_t* idx, int32_t* counts, int32_t* offsets,
                          int32_t* perm, int32_t* inv, void* Xp, hipStream_t s) {
    const long A = static_cast<long>(c.T) * c.k;
    const long chunks = (A + kPermChunk - 1) / kPermChunk;
    if (chunks > kStaticChunks || c.E > kStaticExperts)
        return fail(MOE_ERR_WORKSPACE, "moe_permute_static batches at most %ld assignments over at most %d experts "
                    "(got %ld and %d): its scratch is a fixed array; use moe_permute with a workspace",
                    permute_static_max_assignments(), kStaticExperts, A, c.E);
    // the array's address on the current device, looked up once per device
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static int32_t* on_device[kMaxDevices] = {};
    int dev = 0;
    MOE_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(MOE_ERR_UNSUPPORTED, "device %d: only devices 0..%d are supported", dev, kMaxDevices - 1);
    int32_t* ptr = nullptr;
    {
        std::lock_guard<std::mutex> guard(lock);
        if (on_device[dev] == nullptr) {
            void* p = nullptr;
            MOE_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
            if (p == nullptr) return fail(MOE_ERR_HIP, "hipGetSymbolAddress returned no address for the scratch array");
            on_device[dev] = static_cast<int32_t*>(p);
        }
        ptr = on_device[dev];
    }
    // Nothing has to be cleared: the histogram kernel writes all chunks x E entries the two kernels after it
    // read, whatever an earlier call left in the array.
    return launch_permute(c, x, idx, counts, offsets, perm, inv, Xp, ptr, s);
}

}  // namespace moe
