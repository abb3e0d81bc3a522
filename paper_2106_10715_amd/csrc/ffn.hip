// Expert feed-forward networks on the rows batched by expert (CPM-2 Section 2.1 / Table 1: each
// expert is a d_model -> d_ff -> d_model gated-GELU FFN; Section 6.2: an expert's work is
// proportional to its token count and its parameters form one equal-sized block):
//
//     H  = act(Xp W_gate[e]) * (Xp W_in[e])        "up"   grouped GEMM, epilogue fused
//     Yp = H W_out[e]                               "down" grouped GEMM
//
// bf16 path: 16x16x32 bf16 MFMA, fp32 accumulate.  One block = up to 320 rows of one expert x 4 waves;
// every wave owns its own output columns for all rows, so a weight fragment is needed by exactly
// one wave: weights go HBM -> registers directly in pre-packed fragment order (no LDS, fully
// coalesced 1 KiB reads), only the activation tile is shared through LDS (loaded
// straight into it, conflict-free 16-byte reads).  With few rows per expert the layer is bound by streaming the
// weights once from HBM, which is what this layout is built for.
// fp32 path: ffn_f32.hip.
#include "common.h"
#include "ffn_few.h"
#include "ffn_plan.h"

#include <type_traits>

// This file is compiled in five parts side by side (FFN_PART 0..4; a kernel holds the tile code for 12 or 18 heights in two
// load flavours and takes minutes): the four instantiations of ffn_mfma_kernel, and everything else.
#ifndef FFN_PART
#error "compile with -DFFN_PART=0..4"
#endif

namespace moe {

// One launch of ffn_mfma_kernel (arguments as there).
struct FfnLaunch {
    const void* A; int32_t* plan; int counter_base, e_first;
    const void* W; size_t expert_stride_bytes, block_offset_bytes;
    void* C; int K, N, act, y_chunks, y_shift, mt_shift;
    const int32_t *row_map, *gather;
    int gather_k, h_rows, list, max_tiles;
    unsigned grid;
};
void launch_ffn_up(const FfnLaunch& a, hipStream_t s);
void launch_ffn_up_gather(const FfnLaunch& a, hipStream_t s);
void launch_ffn_down(const FfnLaunch& a, hipStream_t s);
void launch_ffn_down_narrow(const FfnLaunch& a, hipStream_t s);

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline float act_fn(float z, int act) {
    if (act == 0) return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
    const float u = 0.79788456080286536f * (z + 0.044715f * z * z * z);
    return 0.5f * z * (1.0f + tanhf(u));
}

// Exact GELU for results that are rounded to bf16 right away, written on the lower tail of the normal
// distribution: with q(a) = 0.5 erfc(a / sqrt 2), GELU(z) = z Phi(z) = max(z, 0) - |z| q(|z|), which has no
// cancellation for negative z.  log2 q is smooth, so q = exp2(P(a)) with P a polynomial of degree 6,
// fitted on [0, 8] with the error weighted by a q(a) (so that the absolute error of GELU is level):
// |error| <= 1e-7 on GELU in fp32 arithmetic, four orders below the bf16 rounding of the result, in six
// fused multiply-adds and one hardware exponential instead of the several times longer library erff.
// Beyond 8, q < 1e-15 and the argument is clamped (by a comparison that lets a NaN through).
constexpr float kGeluTail[7] = {-0.999993085861206f,   -1.1512017250061035f,   -0.4587709605693817f, -0.05341210961341858f,
                                0.008080719038844109f, -0.0007692205253988504f, 3.309290696051903e-05f};
__device__ inline float act_fn_bf16(float z, int act) {
    if (act != 0) return act_fn(z, act);
    const float a = fabsf(z);
    const float ac = a > 8.0f ? 8.0f : a;
    float p = kGeluTail[6];
#pragma unroll
    for (int i = 5; i >= 0; --i) p = fmaf(p, ac, kGeluTail[i]);
    float relu;                                  // one instruction: fmaxf would first quiet a signalling NaN, and a NaN comes through ac anyway
    asm("v_max_f32 %0, 0, %1" : "=v"(relu) : "v"(z));
    return fmaf(-ac, __builtin_amdgcn_exp2f(p), relu);
}

#if FFN_PART == 0
// ------------------------------------------------------------------------------------------ packing

// One thread per 16-byte lane slot of a fragment: element 8 l + j of fragment (n, s) is
// W[16 s + 8 (l / 32) + j, col(n) + l % 32].
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint16_t* __restrict__ Win, const uint16_t* __restrict__ Wgate,
                                                        const uint16_t* __restrict__ Wout, uint4* __restrict__ packed,
                                                        int d, int f) {
    const long up_frags = static_cast<long>(f / 32) * (d / 16) * 2;
    const long down_frags = static_cast<long>(d / 64) * (f / 16) * 2;
    const long gid = static_cast<long>(blockIdx.x) * 256 + threadIdx.x;
    const long F = gid >> 6;
    const int l = static_cast<int>(gid & 63);
    if (F >= up_frags + down_frags) return;
    const uint16_t* src;
    int ld, row0, col;
    if (F < up_frags) {
        const long per_n = 2L * (d / 16);
        const int n = static_cast<int>(F / per_n);
        const int rem = static_cast<int>(F % per_n);
        src = (rem & 1) ? Win : Wgate;
        ld = f;
        row0 = 16 * (rem >> 1) + 8 * (l >> 5);
        col = 32 * n + (l & 31);
    } else {
        const long G = F - up_frags;
        const long per_p = 2L * (f / 16);
        const int p = static_cast<int>(G / per_p);
        const int rem = static_cast<int>(G % per_p);
        src = Wout;
        ld = d;
        row0 = 16 * (rem >> 1) + 8 * (l >> 5);
        col = 64 * p + 32 * (rem & 1) + (l & 31);
    }
    uint16_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = src[static_cast<size_t>(row0 + j) * ld + col];
    uint4 o;
    o.x = v[0] | (static_cast<uint32_t>(v[1]) << 16);
    o.y = v[2] | (static_cast<uint32_t>(v[3]) << 16);
    o.z = v[4] | (static_cast<uint32_t>(v[5]) << 16);
    o.w = v[6] | (static_cast<uint32_t>(v[7]) << 16);
    packed[F * 64 + l] = o;
}

__global__ __launch_bounds__(256) void copy_vec_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// The work list of a launch is written by ffn_plan_block (ffn_plan.h): here as a kernel of its own.
__global__ __launch_bounds__(256) void ffn_plan_kernel(const int32_t* __restrict__ offsets, int e_first, int e_count,
                                                       int tile_m_up, int tile_m_down, int32_t* __restrict__ plan, int total_rows,
                                                       int max_tiles) {
    __shared__ __align__(16) int scratch[kPlanScratch][256];
    // (a loop, not two calls: the code is fetched anew in every launch)
#pragma unroll 1
    for (int list = 0; list < (tile_m_down != tile_m_up ? 2 : 1); ++list) {      // one: the down kernel reads the up kernel's list
        if (list > 0) __syncthreads();
        ffn_plan_block(offsets, e_first, e_count, list == 0 ? tile_m_up : tile_m_down, plan, total_rows, max_tiles, scratch, list);
    }
}

// (DIRECT is known to the compiler: one kernel for both takes the batched calls 0.3 us longer, 37 tokens x 2, d 1152, f 320, 4 experts 6.7 + 4.1 -> 7.2 + 4.3)
template <bool GATED, bool SMALL, bool DIRECT, bool DEEP = false>
__global__ __launch_bounds__(SMALL ? 64 : 128, few_waves_per_simd(SMALL, DEEP)) void ffn_few_kernel(
    const uint16_t* A, const int32_t* __restrict__ plan, int e_first, const char* W, size_t expert_stride_bytes, size_t block_offset_bytes,
    uint16_t* __restrict__ C, int K, int N, int act, const int32_t* __restrict__ row_map, const int32_t* __restrict__ gather,
    int gather_k, int h_rows, const int32_t* __restrict__ idx, int E) {
    ffn_few_block<GATED, SMALL, DEEP, DIRECT>(A, plan, e_first, W, expert_stride_bytes, block_offset_bytes, C, K, N, row_map, gather, gather_k, h_rows, idx, h_rows, E,
                                [act](float z) { return act_fn_bf16(z, act); });
}

#else   // FFN_PART 1..4
// ------------------------------------------------------------------------------------------ bf16 MFMA
//
// Software pipeline of one block (4 waves, up to 320 rows of one expert, 64 reduction elements per
// step).  In step c every wave
//     issues its share of the activation tile of step c + D          (global -> LDS buffer (c + D) % R)
//     issues its weight fragments of step c + D                      (global -> registers, ring of R sets)
//     runs the MFMAs of step c (weights from the ring, activations from LDS buffer c % R, the LDS reads of a group
//         of MFMAs overlapping the group before it)
//     waits for its loads of step c + 1, barrier.
// The compiler would sink all those loads down to their first use and wait there, which serialises
// the pipeline, and it removes prefetches whose result is never read, which changes how many loads
// are in flight.  So every global load of the loop is issued from inline assembly (pinned in program
// order, never removed) and the one wait per step is written by hand: vector memory loads return in
// order, hence "at most N loads outstanding", N those issued after the loads of step c + 1, means that these have
// arrived.  The wait names the weight registers as read-write operands so that no use of them can be moved above it.
// Why the activations go straight into the LDS: it takes the staging writes and 64 registers out of the loop, and lets the activations be
// requested as early as the weights (loads return in order: one that is waited for soon after its issue makes every older one be waited for as
// well).  Measured against activations staged through registers one and a half steps ahead, whole layer: 65536 tokens on 32 experts
// 13.64 -> 12.82 ms, 16384 tokens x 2 skewed over 64 experts 7505 -> 7261 us, 2048 tokens on 8 experts 568 -> 564, 4096 on 32
// the same.  One step more or less of lead changes nothing: a compute unit has some 44 KiB of loads in flight at most, after which their issue blocks.

constexpr int kKC = 64;                 // reduction elements staged per pipeline step (2 MFMA k-steps)
constexpr int kKS = kKC / 32;           // MFMA k-steps per pipeline step
constexpr uint32_t kStepBytes = (kKC / 16) * 2048;   // bytes of a wave's weight stream one pipeline step spans
constexpr int kLdsRow = 8;              // uint4 per activation row in LDS: 128 B; piece p of row r lies at place p ^ (r % 8)
constexpr int kLdsBytes = 4 * 288 * kLdsRow * 16;   // four activation tiles of up to 288 rows, or three of up to 320, in blocks of 32

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int NF>
struct BFrags { u32x4 v[kKS][2 * NF]; };    // one pipeline step of one wave: 2 k-steps x NF column units x 2 halves of 16 columns

__device__ inline bf16x8 as_bf16x8(const u32x4& u) { return __builtin_bit_cast(bf16x8, u); }
__device__ inline bf16x8 as_bf16x8(const uint4& u) { return __builtin_bit_cast(bf16x8, u); }

// The weight loads: 16 bytes from (uniform base + per-lane byte offset + immediate), pinned in program order.  An expert with one row tile reads its weights once: marked non-temporal they do
// not push the activation tiles (which every column group of the expert re-reads) out of the L2, and the
// stream itself runs faster (a plain read stream of this shape reaches 6.2 TB/s, a non-temporal one 7.1).
// An expert with several row tiles re-reads its weights once per tile: there the plain load, which leaves them
// in the L2 for the tiles that follow, is the faster one (KEEP).
template <int IMM, bool KEEP>
__device__ inline void ld_pinned_stream(u32x4& dst, uint32_t voff, const void* sbase) {
    if constexpr (KEEP)
        asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(dst) : "v"(voff), "s"(sbase), "n"(IMM) : "memory");
    else
        asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3 nt" : "=v"(dst) : "v"(voff), "s"(sbase), "n"(IMM) : "memory");
}

// A packed fragment holds 16 reduction rows x 32 columns; the two fragments of one (column unit, 16 rows) are adjacent,
// [16-row step][2][64 slots] x 16 bytes (2 KiB per step); a wave with NF = 1 reads one of the two.  The 16x16x32
// instruction wants, in lane 16 g + c, column c and the reduction elements 8 g .. 8 g + 7 of 32: those lie in 16-row step
// g / 2, slot 32 (g % 2) + c (+ 16 for the upper half of the columns).  So a lane's offset inside the 4 KiB of a k-step is
// the constant below, and one load covers four runs of 256 bytes, whole cache lines, the other half of the columns the rest.
__device__ inline uint32_t weight_lane_offset(int lane) { return ((lane >> 5) << 11) + (((lane >> 4) & 1) << 9) + ((lane & 15) << 4); }
// Wait until at most N_YOUNGER loads are outstanding; the registers named become usable afterwards.
template <int N_YOUNGER, int NF>
__device__ inline void wait_loads(BFrags<NF>& b) {
    static_assert(N_YOUNGER <= 63, "the counter's range");
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N_YOUNGER) : "memory");
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int j = 0; j < 2 * NF; ++j) asm volatile("" : "+v"(b.v[ks][j]));
}
// An activation tile lies in LDS row-major, 128 bytes per row.  Thread t moves, for mb < MBS, the 16 bytes at place t % 8 of row
// 32 mb + t / 8: eight neighbouring lanes fetch one whole 128-byte line of a row, a wave fills 1 KiB, lane after lane, as the load into
// LDS wants it.  Place p of row r holds piece p ^ (r % 8), so that the fragment reads, one piece of 16 rows each, meet all banks.
// The load: 16 bytes per lane from (uniform base + per-lane byte offset) to LDS byte (base + OFFSET + 16 lane).
template <int OFFSET>
__device__ inline void ld_to_lds(uint32_t lds_base, uint32_t voff, const void* sbase) {
    // (one wait state between the write of m0 and its use)
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(voff), "s"(sbase), "n"(OFFSET) : "memory", "scc");
}

// The MFMAs of a pipeline step (RB blocks of 16 rows) are issued in units: unit u = (k-step u / H, row group u % H), H = 2, 4 or 5
// groups of at most 4 blocks.  The A fragments of unit u+1 are read from LDS while the MFMAs of unit u run; two
// register buffers of G fragments alternate.
// Fragment (rb, ks) of lane l = row rb*16 + l%16, 8 elements at k = 32 ks + 8 (l / 16).
// Why 16x16x32 and not 32x32x16, in whose operand order the weights are packed: experts with many rows are bound by the
// power the matrix pipes draw, and the narrow instruction spends less per multiplication, in the order used here, which keeps
// an activation fragment over the four weight fragments (a loop of nothing but MFMAs on normally distributed operands with the
// accumulators of this kernel: 2.07 PFLOP/s against 1.85; with other orders of the narrow one 1.46 and 1.02).  Measured,
// whole layer, 32x32x16 -> 16x16x32:
// 65536 tokens 13.96 -> 13.36 ms, 16384 tokens x 2 skewed over 64 experts 7.70 -> 7.47 ms, 2048 tokens on 8 experts
// 575 -> 560 us, 4096 tokens on 32 experts 1367 -> 1346 us, 512 tokens unchanged.
template <int RB>
struct Units {
    static constexpr int MBS = (RB + 1) / 2;                       // blocks of 32 rows the activations are staged in
    static constexpr int H = RB > 16 ? 5 : RB > 8 ? 4 : 2;
    static constexpr int G = (RB + H - 1) / H;
    static constexpr int U = kKS * H;
    static constexpr int R = RB > 18 ? 3 : 4;                      // activation tiles in LDS, weight sets in registers
    static constexpr int D = R - 1;                                // steps loads are issued ahead; a buffer is refilled one step after its own
    static constexpr int kBuf = MBS * 32 * kLdsRow * 16;           // bytes of an activation tile
    static_assert(R * kBuf <= kLdsBytes, "the activation tiles fit the LDS");
    static constexpr int first(int u) { return (u % H) * RB / H; }               // first 16-row block of unit u
    static constexpr int count(int u) { return (u % H + 1) * RB / H - first(u); }   // and how many it has
};

template <int LO, int HI, class F>
__device__ inline void static_for(F&& f) {
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>{});
        static_for<LO + 1, HI>(f);
    }
}

// Everything a pipeline step does besides its MFMAs is spread over them, one instruction after each
// MFMA: a load or an LDS access holds the wave's issue slot for some 16 cycles and the matrix pipe
// has only one instruction queued, so a run of them lets it run dry, and a wait that directly follows
// the LDS writes of the whole tile stalls the wave for their full latency.
// Loads done after the units 0..u of a step that spreads n of them evenly over U units:
constexpr int loads_upto(int u, int n, int U) { return u < 0 ? 0 : ((u + 1) * n + U - 1) / U < n ? ((u + 1) * n + U - 1) / U : n; }
// Global loads a step has issued before those of unit u: one activation load per unit while there are
// row blocks left, then the unit's share of the nb weight loads.
constexpr int issued_before(int u, int MBS, int nb, int U) { return (u < MBS ? u : MBS) + loads_upto(u - 1, nb, U); }

// fragment I of unit UNIT, from the activation tile at `tile`: lane 16 g + c holds row c of its 16-row block, piece 4 ks + g
template <int RB, int UNIT, int I>
__device__ inline void read_frag(uint4 (&af)[Units<RB>::G], const uint4* tile, int lane) {
    constexpr int ks = UNIT / Units<RB>::H, rb = Units<RB>::first(UNIT) + I;
    const int at = (lane & 15) * kLdsRow + (((lane >> 4) ^ (lane & 3)) | (lane & 4));      // ((lane >> 4) + 4 ks) ^ (lane % 8) without ks
    af[I] = tile[(at ^ (4 * ks)) + rb * 16 * kLdsRow];
}
// Row blocks whose sums fill the 256 accumulation registers (four fragments of four registers each).  Those of further blocks stay in vector registers: the
// instruction takes its sums from either kind, but the compiler only from the first and would move these there and back in every step, hence the
// assembly; nothing but the same instruction, dozens of others later, uses a sum before the end of the loop.
constexpr int acc_blocks(int RB) { return RB > 18 ? 15 : 16; }
// MFMA M of unit UNIT: 16-row block M / (2 NF) of the unit, weight fragment M % (2 NF)
template <int NF, int RB, int UNIT, int M>
__device__ inline void mma_one(f32x4 (&acc)[RB][2 * NF], const uint4 (&af)[Units<RB>::G], const BFrags<NF>& b) {
    constexpr int ks = UNIT / Units<RB>::H, i = M / (2 * NF), j = M % (2 * NF), rb = Units<RB>::first(UNIT) + i;
    if constexpr (rb < acc_blocks(RB))
        acc[rb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b.v[ks][j]), as_bf16x8(af[i]), acc[rb][j], 0, 0, 0);
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[rb][j]) : "v"(as_bf16x8(b.v[ks][j])), "v"(as_bf16x8(af[i])));
}
// One pipeline step.  Entering, af[0] holds the fragments of unit 0 of this step; leaving, those of
// unit 0 of the next step.
//   cur, nxt : activation tiles of this and of the next step
//   b        : weight fragments of this step
//   b_next   : registers of the next step's weights (loads in flight)
//   issue_a  : issue_a(integral_constant mb) issues the activation load of row block mb this step prefetches
//   issue_b  : issue_b(integral_constant i) issues load i of the kKS * 2 NF weight loads this step prefetches
// After MFMA s of a unit comes its s-th other instruction, in this order: the LDS reads of the next
// unit's fragments, the unit's activation load, its weight loads.  The last unit holds the wait for the next step's loads and the
// barrier after its fourth MFMA (after its second if it has no more than four): all fragments of this step were requested a unit earlier,
// so nothing but those loads is waited for, and the first fragments of the next step are read under the remaining MFMAs.
// The tile this step prefetches may be overwritten from its start on: its last readers passed the barrier of the step before.
template <int NF, int RB, class IssueA, class IssueB>
__device__ inline void run_step(f32x4 (&acc)[RB][2 * NF], uint4 (&af)[2][Units<RB>::G], const uint4* cur, const uint4* nxt,
                                const BFrags<NF>& b, BFrags<NF>& b_next, int lane, IssueA issue_a, IssueB issue_b) {
    constexpr int MBS = Units<RB>::MBS, U = Units<RB>::U, kB = kKS * 2 * NF;
    static_for<0, U>([&](auto uc) {
        constexpr int UU = decltype(uc)::value;
        constexpr bool kLast = UU + 1 == U;
        constexpr int M = Units<RB>::count(UU) * 2 * NF;           // MFMAs of this unit
        constexpr int NU = kLast ? 0 : UU + 1;                     // the unit whose fragments are fetched meanwhile
        constexpr int nR = Units<RB>::count(NU);
        constexpr int nA = UU < MBS ? 1 : 0;
        constexpr int b0 = loads_upto(UU - 1, kB, U), nB = loads_upto(UU, kB, U) - b0;
        constexpr int nOther = nR + nA + nB;
        constexpr int kFirst = !kLast ? 0 : M > 4 ? 3 : 1;         // other instruction s follows MFMA kFirst + kEvery s
        constexpr int kEvery = M - kFirst >= 2 * nOther ? 2 : 1;
        auto other = [&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if constexpr (s < nR)
                read_frag<RB, NU, s>(af[NU & 1], kLast ? nxt : cur, lane);
            else if constexpr (s < nR + nA)
                issue_a(std::integral_constant<int, UU + 0 * s>{});     // (made dependent on s: only instantiated when taken)
            else
                issue_b(std::integral_constant<int, b0 + s - nR - nA>{});
        };
        static_for<0, M>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            mma_one<NF, RB, UU, m>(acc, af[UU & 1], b);
            if constexpr (kLast && m == kFirst) {
                // younger than the loads of the next step: those of the D - 2 steps after it and what this step has issued
                wait_loads<(Units<RB>::D - 2) * (MBS + kB) + issued_before(UU, MBS, kB, U)>(b_next);
                __syncthreads();
            }
            if constexpr (m >= kFirst) {
                constexpr int before = (m - kFirst + kEvery - 1) / kEvery, lo = before < nOther ? before : nOther;
                constexpr int upto = (m - kFirst) / kEvery + 1, hi = m == M - 1 || upto > nOther ? nOther : upto;
                static_for<lo, hi>(other);
            }
        });
    });
}

// The id of this thread inside its block, rebuilt from the wave number (which sits in a scalar
// register) and the lane number, by instructions the compiler can neither hoist nor keep alive: a
// vector register that holds the id across the main loop is one the loop does not have.
__device__ inline unsigned thread_id(int wave) {
    unsigned lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return static_cast<unsigned>(wave) * 64u + lane;
}

// ---- work items.  A launch's items are positions of 8 queues (one per XCD; see ffn_mfma_kernel); everything a
// block needs to take one and to find out what it means, all of it uniform (scalar registers):
struct ItemQueue {
    unsigned* counters;            // positions taken of each queue beyond the first ones (see first_positions)
    unsigned total_q, home;        // positions per queue; this block's own queue
    const int4* tile_list;         // (expert, first row, rows, row tiles of the expert) per row tile
    int tiles, y_chunks, y_shift, mt_shift;
    const char* W;                 // packed weights of expert e_first (+ block_offset_bytes: the up or the down block)
    size_t expert_stride_bytes, block_offset_bytes;
    int e_first;
};
struct Item {
    bool real;                     // false: padding of the queue (past the last tile or column group)
    int e, row_begin, rows, tiles_of_expert, block_y;
};

__device__ inline Item decode_item(const ItemQueue& Q, unsigned q, unsigned xcd, int units) {
    // a run: 1 << mt_shift row tiles x 1 << y_shift column groups
    const unsigned yg = q & ((1u << Q.y_shift) - 1u), mt = (q >> Q.y_shift) & ((1u << Q.mt_shift) - 1u), rest = q >> (Q.y_shift + Q.mt_shift);
    const unsigned y_chunk = rest % static_cast<unsigned>(Q.y_chunks), tile_group = rest / static_cast<unsigned>(Q.y_chunks);
    const int slot = static_cast<int>((((tile_group << 3) + xcd) << Q.mt_shift) + mt);
    Item it;
    it.block_y = static_cast<int>((y_chunk << Q.y_shift) + yg);
    it.real = slot < Q.tiles && it.block_y * 4 < units;
    it.e = it.row_begin = it.rows = it.tiles_of_expert = 0;
    if (it.real) {
        // the same for all lanes, and written by an earlier kernel: read through the scalar cache
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(4))) i32x4 constant_i32x4;
        const i32x4 tile = ((constant_i32x4*)Q.tile_list)[slot];
        it.e = __builtin_amdgcn_readfirstlane(tile.x);
        it.row_begin = __builtin_amdgcn_readfirstlane(tile.y);
        it.rows = __builtin_amdgcn_readfirstlane(tile.z);
        it.tiles_of_expert = __builtin_amdgcn_readfirstlane(tile.w);
    }
    return it;
}

// Start of a wave's fragment stream in an item and the key that fixes where its sweep over the reduction dimension
// starts: the sweep starts at a step that depends on the expert and on the chunk of 8 column groups only, so blocks that
// share a weight stream or an activation tile walk it together; neighbouring chunks are one step apart (measured:
// far-apart chunks fetch the activation tile again, chunks in step collide on their weight streams), other experts
// anywhere.  The same for all lanes, so the address is handed over in scalar registers.
template <bool GATED, int NF>
__device__ inline const void* wave_stream(const ItemQueue& Q, int e, int block_y, int wave, int units, int K, unsigned& key) {
    const int unit = block_y * 4 + wave;
    const int u = unit < units ? unit : units - 1;     // a wave past the last unit recomputes the last one, stores nothing
    const int steps16 = K / 16;
    // fragment pair index and which half of the pair this wave reads
    const int pair = (GATED || NF == 2) ? u : (u >> 1);
    const int half = (GATED || NF == 2) ? 0 : (u & 1);
    const char* wb = Q.W + static_cast<size_t>(e - Q.e_first) * Q.expert_stride_bytes + Q.block_offset_bytes +
                     (static_cast<size_t>(pair) * steps16 * 128 + half * 64) * 16;
    const uintptr_t wbi = reinterpret_cast<uintptr_t>(wb);
    const uint32_t wb_lo = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(wbi))));
    const uint32_t wb_hi = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<uint32_t>(wbi >> 32))));
    key = sweep_key(e, static_cast<unsigned>(block_y) >> ((GATED || NF == 2) ? 3 : 4));   // 128 or 256 columns per group
    return reinterpret_cast<const void*>((static_cast<uintptr_t>(wb_hi) << 32) | static_cast<uintptr_t>(wb_lo));
}

// The first positions of a queue belong to the blocks that call it home, in order, without asking: a block starts on
// position blockIdx / 8.  The counters count what is taken after those.
__device__ inline unsigned first_positions(unsigned x) { return (gridDim.x + 7u - x) >> 3; }
// Thread 0 takes the next position: first from the block's own queue, and when that is empty from the others.
// The first attempt is split from the rest so that its answer can arrive under other work.  Before it asks another queue
// it looks at all counters at once (they only grow, so an old value costs a vain attempt and nothing else): at the end of a
// launch every block finds every queue empty, and seven questions one after the other take some 10 us.
// (Addresses and the one that is added are made opaque where they are used: constants and parts of addresses would be kept in
// vector registers across the main loop.)
template <class T>
__device__ inline T opaque(T v) {
    asm volatile("" : "+v"(v));
    return v;
}
// p + offset, for a uniform p (spelled out: a zero upper half of the offset would be such a constant)
__device__ inline const char* add_offset(const char* p, unsigned offset) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    unsigned lo, hi = opaque(static_cast<unsigned>(v >> 32));
    asm volatile("v_add_co_u32 %0, vcc, %2, %3\n\tv_addc_co_u32 %1, vcc, 0, %1, vcc" : "=&v"(lo), "+v"(hi) : "s"(static_cast<unsigned>(v)), "v"(offset) : "vcc");
    return reinterpret_cast<const char*>(static_cast<uint64_t>(hi) << 32 | lo);
}
// (addressed as global memory: a flat atomic's answer would be waited for at the next barrier)
typedef __attribute__((address_space(1))) unsigned global_counter;
__device__ inline unsigned take_from(const ItemQueue& Q, unsigned queue) {
    return first_positions(queue) + __hip_atomic_fetch_add(opaque((global_counter*)(Q.counters + queue)), opaque(1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline unsigned take_first(const ItemQueue& Q) { return take_from(Q, Q.home); }
__device__ inline void take_finish(const ItemQueue& Q, unsigned v, int* sh_q, int* sh_x) {
    int got = -1;
    unsigned x = Q.home;
    if (v < Q.total_q) {
        got = static_cast<int>(v);
    } else {
        unsigned seen[8];
#pragma unroll
        for (unsigned i = 1; i < 8u; ++i)
            seen[i] = __hip_atomic_load(opaque((global_counter*)(Q.counters + ((Q.home + i) & 7u))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (unsigned i = 1; i < 8u; ++i) {
            const unsigned y = (Q.home + i) & 7u;
            if (got < 0 && first_positions(y) + seen[i] < Q.total_q) {
                const unsigned w = take_from(Q, y);
                if (w < Q.total_q) { got = static_cast<int>(w); x = y; }
            }
        }
    }
    *sh_q = got;
    *sh_x = static_cast<int>(x);
}

// One tile of RB blocks of 16 rows: the whole reduction loop and the epilogue.
// Loads past the end are clamped to valid addresses (rows to the last row of the tile, pipeline steps
// to the last step) instead of being skipped, so every step issues the same loads.  Rows that are
// clamped duplicates only produce output rows that are never stored (an output row depends on its own
// input row only).
// GATHER: A is not the batched row array but the token array it was gathered from, and row r of the batched
// order is token gather[r] / gather_k of A (the batching of Section 6.2 done on the fly: the batched copy of the
// activations is never written); every thread then keeps one byte offset per row block instead of two in all.
template <bool GATED, int NF, int RB, bool KEEP, bool GATHER = false>
__device__ inline void ffn_tile(uint4 (&lds)[kLdsBytes / 16], const uint16_t* __restrict__ A, int row_begin, int rows,
                                const void* wave_base, uint16_t* __restrict__ C, int K, int N, int unit,
                                bool active, int act, unsigned phase_key, int wave_s, const int32_t* __restrict__ row_map,
                                const int32_t* __restrict__ gather, int gather_k, const ItemQueue& Q, int units, int* sh_q,
                                int* sh_x, int h_rows) {
    constexpr int MBS = Units<RB>::MBS;
    unsigned tid = thread_id(wave_s);
    const int lane = tid & 63;
    // every tile height gets its own copy of the loop bounds: shared ones would be computed once for all
    // heights and stay in registers across this one
    asm volatile("" : "+s"(K), "+s"(N), "+s"(phase_key));
    const int chunks = K / kKC, last = chunks - 1;

    // this thread's activation sources (byte offsets from A): row mb*32 + t/8 of every block, the piece that lies at place t%8.
    // All blocks but the last hold 32 rows, so their rows lie a fixed stride apart; rows past the end
    // of the last block re-read the tile's last row.
    const int r0 = tid >> 3;
    const uint32_t piece = 16u * ((tid ^ (tid >> 3)) & 7);
    // Layout of A.  The up-projection reads row-major rows (K elements each).  The down-projection reads the
    // intermediate H, which only these two kernels see and which is therefore kept in the order they touch it:
    // [chunk of 64 columns][row][64 columns], all h_rows rows of a chunk back to back, so that a tile's rows of one
    // chunk are one contiguous run, for the up-projection's stores (scattered 256-byte pieces cost the memory far
    // more than their bytes) as for these loads.
    const uint32_t a_row_bytes = GATED ? static_cast<uint32_t>(K) * 2u : static_cast<uint32_t>(kKC * 2);
    const size_t a_chunk_bytes = GATED ? static_cast<size_t>(kKC * 2) : static_cast<size_t>(h_rows) * (kKC * 2);
    const uint32_t a_first = static_cast<uint32_t>(row_begin + r0) * a_row_bytes + piece;
    const uint32_t a_last = static_cast<uint32_t>(row_begin + min((MBS - 1) * 32 + r0, rows - 1)) * a_row_bytes + piece;
    const uint32_t a_stride = 32u * a_row_bytes;        // 32 rows, in bytes
    uint32_t a_off[GATHER ? MBS : 1];           // GATHER: this thread's source row of every block, as a byte offset from A
    if constexpr (GATHER) {
#pragma unroll
        for (int mb = 0; mb < MBS; ++mb) {
            const int row = row_begin + min(mb * 32 + r0, rows - 1);
            a_off[mb] = static_cast<uint32_t>(gather[row] / gather_k) * K * 2u + piece;
        }
    }

    f32x4 acc[RB][2 * NF];
    // cleared in place, in the accumulation registers: a zero constant would be parked in 16 registers for all
    // tile heights and copied from there
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int j = 0; j < 2 * NF; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (rb < acc_blocks(RB)) asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(acc[rb][j][v]));
                else asm volatile("v_mov_b32 %0, 0" : "=v"(acc[rb][j][v]));
            }

    constexpr int D = Units<RB>::D, R = Units<RB>::R, kBuf = Units<RB>::kBuf;       // register indices and tiles repeat with period R
    constexpr int kB = kKS * 2 * NF;            // loads of one weight step
    static_assert(MBS <= Units<RB>::U, "one activation load per unit");
    BFrags<NF> ring[R];
    uint4 af[2][Units<RB>::G];
    auto tile_of = [&](int buf) { return reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(&lds[0]) + buf * kBuf); };
    const uint32_t lds_wave = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(reinterpret_cast<__attribute__((address_space(3))) char*>(
                                  (__attribute__((address_space(3))) uint4*)&lds[0]))) + static_cast<uint32_t>(wave_s) * 1024u;
    const uint32_t lane_off = weight_lane_offset(lane);
    // Blocks that share a weight stream or an activation tile start their sweep over the reduction
    // dimension at the same step (and wrap around), other blocks at other steps, so that concurrent
    // waves do not all walk their weight streams, which lie a power of two apart, in lockstep.  The
    // phase never depends on the launch shape, so a launch over all experts and a launch over one
    // expert sum in the same order (bitwise equal results).
    const int phase = static_cast<int>(phase_key % static_cast<unsigned>(chunks));
    auto at = [&](int i) { const int c = phase + i; return c >= chunks ? c - chunks : c; };   // i < chunks
    // Loads of step i, row block mb / weight load i of the step, into buffer / set BUF.  The per-block and per-step parts of the address
    // are uniform: they go into the scalar base, and the per-thread part is the same register for every block but the last.  Past the
    // last step there is nothing left to prefetch: the loads still issue (the waits count them), but all lanes read the
    // same 16 bytes, one cache line instead of a KiB per load.
    struct Source { const char* a; uint32_t first, last, keep, voff; };
    auto source = [&](int i) __attribute__((always_inline)) {
        const int k = at(min(i, last));
        return Source{reinterpret_cast<const char*>(A) + static_cast<size_t>(k) * a_chunk_bytes, i > last ? 0u : a_first, i > last ? 0u : a_last,
                      i > last ? 0u : ~0u, static_cast<uint32_t>(k) * kStepBytes + (i > last ? 0u : lane_off)};
    };
    auto issue_a = [&](const Source& f, auto buf, auto mbc) __attribute__((always_inline)) {
        constexpr int mb = decltype(mbc)::value, kTo = decltype(buf)::value * kBuf + mb * 4096;
        if constexpr (GATHER)
            ld_to_lds<kTo>(lds_wave, a_off[mb] & f.keep, f.a);
        else if constexpr (mb + 1 < MBS)
            ld_to_lds<kTo>(lds_wave, f.first, f.a + static_cast<size_t>(mb) * a_stride);
        else
            ld_to_lds<kTo>(lds_wave, f.last, f.a);
    };
    auto issue_b = [&](const Source& f, auto buf, auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, ks = i / (2 * NF), j = i % (2 * NF);
        ld_pinned_stream<(j >> 1) * 1024 + (j & 1) * 256, KEEP>(ring[decltype(buf)::value].v[ks][j], f.voff + ks * 4096, wave_base);
    };
    int c = 0;
    auto step = [&](auto ic) __attribute__((always_inline)) {      // step c + I, c a multiple of R: all register indices are static
        constexpr int I = decltype(ic)::value;
        const Source f = source(c + I + D);
        run_step<NF, RB>(acc, af, tile_of(I % R), tile_of((I + 1) % R), ring[I % R], ring[(I + 1) % R], lane,
                         [&](auto mb) __attribute__((always_inline)) { issue_a(f, std::integral_constant<int, (I + D) % R>{}, mb); },
                         [&](auto i) __attribute__((always_inline)) { issue_b(f, std::integral_constant<int, (I + D) % R>{}, i); });
    };
    asm volatile("; pipeline begin");           // from here to the matching end the build allows no spill code
    static_for<0, D>([&](auto jc) __attribute__((always_inline)) {
        const Source f = source(decltype(jc)::value);
        static_for<0, MBS>([&](auto mb) __attribute__((always_inline)) { issue_a(f, jc, mb); });
        static_for<0, kB>([&](auto i) __attribute__((always_inline)) { issue_b(f, jc, i); });
    });
    wait_loads<(D - 1) * (MBS + kB)>(ring[0]);
    __syncthreads();
    static_for<0, Units<RB>::count(0)>([&](auto i) __attribute__((always_inline)) { read_frag<RB, 0, decltype(i)::value>(af[0], tile_of(0), lane); });
    for (; c + R <= chunks; c += R) static_for<0, R>(step);
    // (the sums written by assembly, of whose latency the compiler knows nothing: 18 wait states before anything else reads them)
    if constexpr (RB > acc_blocks(RB)) asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
    asm volatile("; pipeline end");
    // All loads have landed, those past the last step included, and only now are their destination registers let go of: one the compiler
    // considers dead would be handed to something else (an LDS read, say) while the load into it is still in flight.
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
            for (int j = 0; j < 2 * NF; ++j) asm volatile("" : "+v"(ring[r].v[ks][j]));
    // the steps that do not fill a round of the loop, fewer than R and so all here: without overlap, the weights moved up after each
    if (c < chunks) {
        __syncthreads();                        // every wave's share of their activation tiles has landed
        for (const uint4* tile = tile_of(0); c < chunks; ++c, tile += kBuf / 16) {
            static_for<0, Units<RB>::U>([&](auto uc) __attribute__((always_inline)) {
                constexpr int UU = decltype(uc)::value;
                static_for<0, Units<RB>::count(UU)>([&](auto i) __attribute__((always_inline)) { read_frag<RB, UU, decltype(i)::value>(af[0], tile, lane); });
                static_for<0, Units<RB>::count(UU) * 2 * NF>([&](auto m) __attribute__((always_inline)) { mma_one<NF, RB, UU, decltype(m)::value>(acc, af[0], ring[0]); });
            });
#pragma unroll
            for (int r = 0; r + 1 < R; ++r) ring[r] = ring[r + 1];
        }
        if constexpr (RB > acc_blocks(RB)) asm volatile("s_nop 15\n\ts_nop 15" : : : "memory");
    }
    __syncthreads();                            // the last LDS reads are done before the epilogue reuses the LDS
    tid = thread_id(wave_s);                    // rebuilt: the first copy need not survive the main loop
    // The block's next work item is taken now, by thread 0: the queue's answer arrives while the output tile is
    // filled, is published with the barrier that follows the filling, and lets every wave request the first weights
    // of its next item before it stores the tile, so that they are in the L2 (and the memory system has had this
    // compute unit's requests) by the time the next item's own first loads ask for them.  An item is taken only a
    // few microseconds before the block turns to it, so the balance of the queues is what it was.
    unsigned taken = 0u;
    if (tid == 0) taken = take_first(Q);
    constexpr int kWarm = 2 * kKS * (GATED ? 2 : NF);       // 16-byte pieces per lane of one pipeline step of this wave's stream
    u32x4 warm[kWarm];
#pragma unroll
    for (int i = 0; i < kWarm; ++i) warm[i] = u32x4{0u, 0u, 0u, 0u};
    // Epilogue through LDS (the activation buffers are free now).  The weight fragment is the first MFMA
    // operand and the activation fragment the second, so the accumulators hold the transposed tile: lane l
    // has token row l%16 of its 16-row block and the four neighbouring output columns 4(l/16) + 0..3 of 16.
    // Every wave applies the activation, rounds four neighbours to bf16 and writes them
    // as one 8-byte piece into a row-major tile of the block's columns; then the whole block stores that tile
    // with 16 bytes per lane, whole 64-byte segments per row.  All rows are computed (clamped duplicates
    // give finite values), only real rows are stored.
    constexpr int W = 32 * (GATED ? 1 : NF);            // output columns per wave
    constexpr int kTileRowBytes = 4 * W * 2 + 16;       // padded: neighbouring rows start 4 dwords apart mod 32
    constexpr int kRowsPerPass = W == 32 ? kTileM : 128;   // tile rows that fit the LDS
    constexpr int kLanesPerRow = W / 2;                 // 16-byte stores per tile row
    constexpr int kRowsPerIter = 256 / kLanesPerRow;
    char* tile = reinterpret_cast<char*>(&lds[0]);
    static_assert(kRowsPerPass * kTileRowBytes <= static_cast<int>(sizeof(lds)), "epilogue tile must fit the LDS buffers");
    const int wave = wave_s;
    const int row_in = (tid & 15), col_in = 4 * ((tid & 63) >> 4);
    // the first step of this wave's weight stream in the block's next item (plain loads: they stay in the L2).  The end of the item waits for them, which
    // low tiles with short reductions lose more by than the next item gains: none up to 12 steps (300, 600 and 1000 tokens on 33 experts, d 768, f 3072
    // 116.3 -> 113.7, 119.1 -> 117.0 and 126.8 -> 122.4 us; d 1024 equal, 1000 tokens 206 -> 209; d 2048 and 4096 lose 0.5-0.8 % without them, and tall
    // tiles lose 3-6 % at 4 and 8 steps: the two products of 20000 rows on 64 experts, d 256, f 512 27.7 -> 28.4 and 20.0 -> 21.2).
    auto warm_next = [&]() {
        if (RB <= 4 && chunks <= 12) return;            // uniform
        const int nq = __builtin_amdgcn_readfirstlane(*sh_q);
        if (nq < 0) return;
        const Item nx = decode_item(Q, static_cast<unsigned>(nq), static_cast<unsigned>(__builtin_amdgcn_readfirstlane(*sh_x)), units);
        if (!nx.real) return;
        unsigned nkey;
        const char* nw = static_cast<const char*>(wave_stream<GATED, NF>(Q, nx.e, nx.block_y, wave_s, units, K, nkey));
        // (addressed as global memory, so that the loads return in order with the other global loads and the stores
        // that follow wait for their own operands only)
        typedef const __attribute__((address_space(1))) u32x4 global_u32x4;
        global_u32x4* src = (global_u32x4*)add_offset(nw + static_cast<size_t>(nkey % static_cast<unsigned>(chunks)) * kStepBytes, 16u * (tid & 63));
#pragma unroll
        for (int i = 0; i < kWarm; ++i) warm[i] = src[(GATED || NF == 2) ? i * 64 : i * 128];
    };
#pragma unroll
    for (int p0 = 0; p0 < RB * 16; p0 += kRowsPerPass) {
        if (p0 > 0) __syncthreads();                    // the previous pass has been stored
        // the choice of activation is taken once per pass, outside the value loops, so that the independent
        // evaluations of a wave can overlap
        auto fill = [&](auto exact) {
#pragma unroll
            for (int rb = p0 / 16; rb < RB && rb < (p0 + kRowsPerPass) / 16; ++rb) {
                char* trow = tile + (rb * 16 + row_in - p0) * kTileRowBytes + (wave * W + col_in) * 2;
#pragma unroll
                for (int j = 0; j < (GATED ? 2 : 2 * NF); ++j) {        // 16 columns each
                    float h[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (GATED)
                            h[i] = act_fn_bf16(acc[rb][j][i], decltype(exact)::value ? 0 : 1) * acc[rb][2 * NF - 2 + j][i];
                        else
                            h[i] = acc[rb][j][i];
                    }
                    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                    const bf16x4 packed = {static_cast<__bf16>(h[0]), static_cast<__bf16>(h[1]), static_cast<__bf16>(h[2]),
                                           static_cast<__bf16>(h[3])};
                    *reinterpret_cast<uint2*>(trow + 32 * j) = __builtin_bit_cast(uint2, packed);
                }
            }
        };
        if (!GATED || act == 0) fill(std::true_type{});
        else fill(std::false_type{});
        if (p0 == 0 && tid == 0) take_finish(Q, taken, sh_q, sh_x);
        __syncthreads();
        const int seg = (tid % kLanesPerRow) * 8;       // first of this lane's 8 columns inside the block
        const int src_wave = seg / W;
        const int out_unit = unit - wave + src_wave;            // unit of the wave that produced them
        if (out_unit < N / W) {
            // first of this lane's 8 columns, and the distance between rows, in elements: row-major output, or
            // (the up-projection's) the chunked order of H described above
            const int col = out_unit * W + (seg % W);
            uint16_t* cbase = GATED ? C + static_cast<size_t>(col >> 6) * h_rows * kKC + (col & (kKC - 1)) : C + col;
            const size_t c_row_elems = GATED ? static_cast<size_t>(kKC) : static_cast<size_t>(N);
            // All pieces of the pass are read from the tile (and their output rows looked up) before the first
            // is stored: one LDS and one look-up latency per pass instead of one per piece.
            //   row_map: where each row of the batched order goes (the layer's output rows, when the rows
            //   need no weighting afterwards); none: the batched order itself
            constexpr int kPieces = kRowsPerPass / kRowsPerIter;
            uint4 val[kPieces];
            int out_row[kPieces];
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                if (i * kRowsPerIter < RB * 16 - p0) {                   // rows this tile height has
                    const int r = static_cast<int>(tid) / kLanesPerRow + i * kRowsPerIter;
                    val[i] = *reinterpret_cast<const uint4*>(tile + r * kTileRowBytes + seg * 2);
                    const int row = row_begin + min(p0 + r, rows - 1);    // past the end: the last row again, not stored
                    out_row[i] = row_map != nullptr ? row_map[row] : row;
                }
            }
            if (p0 == 0) warm_next();
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                if (i * kRowsPerIter < RB * 16 - p0) {
                    const int r = static_cast<int>(tid) / kLanesPerRow + i * kRowsPerIter;
                    // written once and next read by another kernel, after far more traffic than the L2 holds: stored
                    // non-temporal, so that the rows do not take the place of weights and activation tiles there
                    // (5 % of the layer's time at 128 tokens per expert)
                    if (p0 + r < rows)
                        __builtin_nontemporal_store(u32x4{val[i].x, val[i].y, val[i].z, val[i].w},
                                                    reinterpret_cast<u32x4*>(cbase + static_cast<size_t>(out_row[i]) * c_row_elems));
                }
            }
        } else if (p0 == 0) {
            warm_next();
        }
    }
    // the requested pieces are only wanted in the cache; their registers are given up once they have arrived
#pragma unroll
    for (int i = 0; i < kWarm; ++i) asm volatile("" : : "v"(warm[i]));
}

constexpr int kKeepFromTiles = 2;       // row tiles of an expert from which its weights are worth keeping in the L2

// C[rows of one expert tile, N] = A[rows, K] * B_e, B_e in packed fragment order.
// A work item is one row tile (up to 320 rows of one expert; only the 16-row blocks that hold rows are
// computed) by one column group of 4 units, one unit per wave, for all rows.
// GATED (NF = 2): a unit is 32 output columns whose two fragments per k-step are (W_gate, W_in); the
//   epilogue writes act(gate) * in.
// otherwise a unit is 32 * NF output columns of W_out.
// Weight fragments stream HBM -> registers and activation tiles HBM -> LDS through rings of buffers, so that several KiB per
// wave are always in flight.
//
// One block per compute unit stays resident and takes work items from 8 queues, one per XCD (blocks go
// round-robin to the XCDs, each with its own L2, so blockIdx % 8 names the XCD): position q of a
// queue decodes into runs of 2^mt_shift neighbouring row tiles x 2^y_shift neighbouring column groups (32 items, or
// fewer where that leaves no position without an item).  Tiles of one expert then share its weight stream, and the column groups of a tile
// share its activation tile, in that XCD's L2; groups of tiles are dealt to the queues in turn.  A
// block whose own queue is empty helps with the others.
// GATHER (up-projection only): A is the token array x and the rows of a tile are looked up through `gather`
// (the permutation written by the batching step; row r is token gather[r] / gather_k); tiles then have at most
// kGatherTileM rows.
template <bool GATED, int NF, bool GATHER = false>
__global__ __launch_bounds__(256) void ffn_mfma_kernel(const uint16_t* __restrict__ A, int32_t* __restrict__ plan,
                                                       int counter_base, int e_first, const char* __restrict__ W,
                                                       size_t expert_stride_bytes, size_t block_offset_bytes,
                                                       uint16_t* __restrict__ C, int K, int N, int act, int y_chunks,
                                                       int y_shift, int mt_shift, const int32_t* __restrict__ row_map,
                                                       const int32_t* __restrict__ gather, int gather_k, int h_rows,
                                                       int list, int max_tiles) {
    __shared__ uint4 lds[kLdsBytes / 16];          // activation tiles; between items, the output tile
    __shared__ int sh_q, sh_x;
    ItemQueue Q;
    Q.tiles = plan[16 + list];
    Q.y_chunks = y_chunks;
    Q.y_shift = y_shift;
    Q.mt_shift = mt_shift;
    const unsigned per_group = 8u << mt_shift;
    Q.total_q = ((static_cast<unsigned>(Q.tiles) + per_group - 1u) / per_group * static_cast<unsigned>(y_chunks)) << (mt_shift + y_shift);
    Q.tile_list = reinterpret_cast<const int4*>(plan + kPlanHeader + 4 * list * max_tiles);
    Q.counters = reinterpret_cast<unsigned*>(plan) + counter_base;
    Q.home = blockIdx.x & 7u;
    Q.W = W;
    Q.expert_stride_bytes = expert_stride_bytes;
    Q.block_offset_bytes = block_offset_bytes;
    Q.e_first = e_first;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    // an item taken with nothing to do meanwhile: the one after a padding position
    auto take_now = [&]() {
        __syncthreads();                           // everybody has read the previous position
        if (thread_id(wave) == 0) take_finish(Q, take_first(Q), &sh_q, &sh_x);
        __syncthreads();
    };
    if (thread_id(wave) == 0) take_finish(Q, blockIdx.x >> 3, &sh_q, &sh_x);      // the block's own first position
    __syncthreads();
    for (;;) {
        if (sh_q < 0) return;                      // every queue is empty (uniform for the block)
        // The tile code below is compiled for 12 or 18 tile heights; values that do not change from item to
        // item would be hoisted out of this loop and held in registers across all of them.  The inputs
        // are made opaque per iteration instead.  (In the up-projection that does not gather, most heights still keep one or two 8-byte values in
        // scratch memory over their main loop, outside of which they are stored and loaded: twice per item, of some 100 us.)
        int Kl = K, Nl = N;
        asm volatile("" : "+s"(Kl), "+s"(Nl));
        const int units = Nl / (32 * (GATED ? 1 : NF));
        const Item it = decode_item(Q, static_cast<unsigned>(__builtin_amdgcn_readfirstlane(sh_q)),
                                    static_cast<unsigned>(__builtin_amdgcn_readfirstlane(sh_x)), units);
        if (!it.real) { take_now(); continue; }    // past the last tile or column group (uniform)
        const int e = it.e, row_begin = it.row_begin, rows = it.rows, tiles_of_expert = it.tiles_of_expert;
        const int unit = it.block_y * 4 + wave;
        const bool active = unit < units;          // a wave past the last unit recomputes the last one, stores nothing
        unsigned key;
        const void* wave_w = wave_stream<GATED, NF>(Q, e, it.block_y, wave, units, Kl, key);
        // weights of an expert with two row tiles or more are left in the L2 for its other tiles
        const bool keep = tiles_of_expert >= kKeepFromTiles;
        // A single block runs as two: its steps of four MFMAs per unit are too short (600 tokens, d 768, f 3072, 33 experts 122 -> 120 us).  Three run as
        // four: a height of their own gains nothing where the weights are the bound, and costs a short launch the fetching of its code (1500 tokens,
        // d 512, f 1024, 33 experts of 45 rows 52.8 -> 51.3 us, 1200 53.1 -> 52.0; with seven as eight too 900 tokens on 8 experts, d 4096 381 -> 386).
        const int blocks = min((rows + 15) >> 4, (GATHER ? kGatherTileM : kTileM) / 16);
#define FFN_TILE(RB, KP)                                                                                             \
    ffn_tile<GATED, NF, RB, KP, GATHER>(lds, A, row_begin, rows, wave_w, C, Kl, Nl, unit, active, act, key, wave, row_map, \
                                        gather, gather_k, Q, units, &sh_q, &sh_x, h_rows)
#define FFN_CASE(RB)                                                                                                 \
    case RB:                                                                                                         \
        if (keep) FFN_TILE(RB, true); else FFN_TILE(RB, false);                                                      \
        break;
        if constexpr (GATHER) {
            switch (blocks) {
                case 1: FFN_CASE(2) case 3: FFN_CASE(4) FFN_CASE(5) FFN_CASE(6) FFN_CASE(7) FFN_CASE(8) FFN_CASE(9)
                FFN_CASE(10) FFN_CASE(11) FFN_CASE(12) FFN_CASE(13)
                default: if (keep) FFN_TILE(kGatherTileM / 16, true); else FFN_TILE(kGatherTileM / 16, false); break;
            }
        } else {
            switch (blocks) {
                case 1: FFN_CASE(2) case 3: FFN_CASE(4) FFN_CASE(5) FFN_CASE(6) FFN_CASE(7) FFN_CASE(8) FFN_CASE(9)
                FFN_CASE(10) FFN_CASE(11) FFN_CASE(12) FFN_CASE(13) FFN_CASE(14) FFN_CASE(15) FFN_CASE(16) FFN_CASE(17) FFN_CASE(18) FFN_CASE(19)
                default: if (keep) FFN_TILE(kTileM / 16, true); else FFN_TILE(kTileM / 16, false); break;
            }
        }
#undef FFN_CASE
#undef FFN_TILE
        __syncthreads();                           // the tile has been read out of the LDS; the next position is in sh_q
    }
}

template <bool GATED, int NF, bool GATHER>
void launch_mfma(const FfnLaunch& a, hipStream_t s) {
    hipLaunchKernelGGL((ffn_mfma_kernel<GATED, NF, GATHER>), dim3(a.grid), dim3(256), 0, s, static_cast<const uint16_t*>(a.A), a.plan,
                       a.counter_base, a.e_first, static_cast<const char*>(a.W), a.expert_stride_bytes, a.block_offset_bytes,
                       static_cast<uint16_t*>(a.C), a.K, a.N, a.act, a.y_chunks, a.y_shift, a.mt_shift, a.row_map, a.gather, a.gather_k,
                       a.h_rows, a.list, a.max_tiles);
}
#endif  // FFN_PART

}  // namespace

#if FFN_PART == 1
void launch_ffn_up(const FfnLaunch& a, hipStream_t s) { launch_mfma<true, 2, false>(a, s); }
#elif FFN_PART == 2
void launch_ffn_up_gather(const FfnLaunch& a, hipStream_t s) { launch_mfma<true, 2, true>(a, s); }
#elif FFN_PART == 3
void launch_ffn_down(const FfnLaunch& a, hipStream_t s) { launch_mfma<false, 2, false>(a, s); }
#elif FFN_PART == 4
void launch_ffn_down_narrow(const FfnLaunch& a, hipStream_t s) { launch_mfma<false, 1, false>(a, s); }
#else
size_t ffn_plan_tiles(const moe_cfg& c) { return static_cast<size_t>(c.T) * c.k / kMinTileM + c.E; }   // room for the lowest tiles
bool ffn_reads_idx(const moe_cfg& c, int n_cu) {
    return static_cast<long>(c.T) * c.k <= kDirectRows && (c.dtype == MOE_F32 || few_rows(c, n_cu));
}

size_t ffn_plan_bytes(const moe_cfg& c) { return (kPlanHeader + 2 * 4 * ffn_plan_tiles(c)) * sizeof(int32_t); }

int launch_pack(const moe_cfg& c, const void* Win, const void* Wgate, const void* Wout, void* packed, hipStream_t s) {
    const size_t df = static_cast<size_t>(c.d) * c.f;
    if (c.dtype == MOE_BF16) {
        const long frags = static_cast<long>(c.f / 32) * (c.d / 16) * 2 + static_cast<long>(c.d / 64) * (c.f / 16) * 2;
        const long threads = frags * 64;
        hipLaunchKernelGGL(pack_bf16_kernel, dim3(static_cast<unsigned>((threads + 255) / 256)), dim3(256), 0, s,
                           static_cast<const uint16_t*>(Win), static_cast<const uint16_t*>(Wgate),
                           static_cast<const uint16_t*>(Wout), static_cast<uint4*>(packed), c.d, c.f);
        MOE_LAUNCH_CHECK("pack_bf16_kernel");
        return MOE_OK;
    }
    // fp32: W_gate | W_in | W_out, row-major, unchanged
    const size_t vecs = df * 4 / 16;
    const void* srcs[3] = {Wgate, Win, Wout};
    for (int i = 0; i < 3; ++i) {
        hipLaunchKernelGGL(copy_vec_kernel, dim3(static_cast<unsigned>((vecs + 255) / 256)), dim3(256), 0, s,
                           static_cast<const uint4*>(srcs[i]), static_cast<uint4*>(packed) + i * vecs, vecs);
        MOE_LAUNCH_CHECK("copy_vec_kernel");
    }
    return MOE_OK;
}

int launch_expert_ffn(const moe_cfg& c, const void* Xp, const int32_t* offsets, int e_first, int e_count,
                      const void* W, size_t expert_stride_bytes, long max_rows, void* H, void* Yp, int32_t* plan,
                      hipStream_t s, hipEvent_t between, hipEvent_t before_up, const int32_t* row_map, const FfnTiles* listed,
                      const int32_t* gather, const int32_t* idx) {
    if (max_rows <= 0 || e_count <= 0) return MOE_OK;
    const size_t df = static_cast<size_t>(c.d) * c.f;
    if (c.dtype == MOE_BF16) {
        // Work items: 8 queues x (groups of row tiles per queue) x (chunks of column groups) x 32; the
        // resident blocks take them until the queues are empty.
        int dev = 0;
        const DeviceInfo* info = nullptr;
        if (int rc = device_info(&dev, &info)) return rc;
        const int n_cu = info->compute_units;
        const FfnTiles cut = listed != nullptr ? *listed : ffn_tiles(c, gather != nullptr, n_cu, e_count, max_rows);
        const int tile_m = cut.up, tile_m_down = cut.down;
        if (tile_m > (gather != nullptr ? kGatherTileM : kTileM) || tile_m_down > kTileM)       // rows past those the kernel has code for would be left out
            return fail(MOE_ERR_INVALID_ARG, "row tiles of %d and %d rows are too high for the expert kernels", tile_m, tile_m_down);
        const long slots = max_rows / tile_m + e_count;                // upper bound of the number of row tiles
        const long slots_down = max_rows / tile_m_down + e_count;
        if (slots_down > static_cast<long>(ffn_plan_tiles(c)))
            return fail(MOE_ERR_INVALID_ARG, "more row tiles (%ld) than the workspace plans for", slots_down);
        if (slots > static_cast<long>(ffn_plan_tiles(c)))
            return fail(MOE_ERR_INVALID_ARG, "more row tiles (%ld) than the workspace plans for", slots);
        // Row tiles per group (4, 2 or 1): neighbouring tiles in the list belong to one expert when experts have
        // several tiles, and then a group shares the expert's weight stream in one XCD's L2; when experts have
        // a single tile each, a group of several would only put several activation tiles into that L2 at once
        // (measured at 128 tokens per expert: 3 % of the layer's time).  Decided from the mean rows per expert,
        // all the host knows.
        const long mean_rows = max_rows / e_count;
        const int by_rows = mean_rows > 384 ? 2 : mean_rows > 192 ? 1 : 0;
        auto shift_for = [&](long n_slots) {
            const int by_tiles = n_slots >= 32 ? 2 : n_slots >= 16 ? 1 : 0;
            return by_rows < by_tiles ? by_rows : by_tiles;
        };
        const int mt_shift = shift_for(slots), mt_shift_down = shift_for(slots_down);
        // positions of all queues.  Runs hold 32 items; narrower ones are taken where they leave fewer positions without an
        // item (80 column groups: five runs of 16 and not three of 32).
        auto items_for = [&](long n_slots, int shift, int col_groups, int& y_shift, int& y_chunks) {
            const long tile_groups = (n_slots + (8L << shift) - 1) / (8L << shift);   // per queue
            y_shift = 5 - shift;
            auto padded = [&](int ys) { return (col_groups + (1 << ys) - 1) >> ys << ys; };
            for (int ys = y_shift - 1; ys >= 0; --ys)
                if (padded(ys) < padded(y_shift)) y_shift = ys;
            y_chunks = padded(y_shift) >> y_shift;
            return ((tile_groups * 8) << (shift + y_shift)) * y_chunks;
        };
        const int max_tiles = static_cast<int>(ffn_plan_tiles(c));
        const int down_list = tile_m_down != tile_m ? 1 : 0;       // equal heights: one list serves both kernels
        if (listed == nullptr && idx == nullptr) {          // else the kernel that batched the tokens has written the work list as well
            hipLaunchKernelGGL(ffn_plan_kernel, dim3(1), dim3(256), 0, s, offsets, e_first, e_count, tile_m, tile_m_down, plan,
                               c.T * c.k, max_tiles);
            MOE_LAUNCH_CHECK("ffn_plan_kernel");
        }
        if (before_up != nullptr) MOE_HIP_CHECK(hipEventRecord(before_up, s));
        const size_t down_off = 2 * df * 2;
        if (few_rows(c, n_cu)) {
            const unsigned n_tiles = static_cast<unsigned>(max_rows < slots ? max_rows : slots);
            // Up-projection in blocks of two waves, whose units are neighbours in memory, for 16 experts and more; with fewer experts
            // to fill the chip, or all rows on one of them, smaller blocks spread better.  us, one / two waves: 40 tokens on 32
            // experts 869 / 856, 128 on 16 641 / 629, 64 on 8 319 / 319; 64 rows on one expert (FFN alone) 109 / 126.
            const int up_waves = c.T * c.k > 16 && c.E >= 16 ? 2 : 1;
// (few_depth: the rows have an expert each at most)
            const bool deep = static_cast<long>(n_tiles) * (c.d / few_columns(false, true)) <= n_cu && c.f >= 4096;
#define MOE_FFN_FEW_DOWN(SMALL, DIRECT, DEEP)                                                                                 \
    hipLaunchKernelGGL((ffn_few_kernel<false, SMALL, DIRECT, DEEP>), dim3(c.d / few_columns(false, SMALL), n_tiles), dim3(64), 0, s, \
                       static_cast<const uint16_t*>(H), plan, e_first, static_cast<const char*>(W),                           \
                       expert_stride_bytes, down_off, static_cast<uint16_t*>(Yp), c.f, c.d, c.act, row_map,                   \
                       static_cast<const int32_t*>(nullptr), 1, c.T * c.k, idx, c.E)
#define MOE_FFN_FEW(SMALL, DIRECT)                                                                                            \
    {                                                                                                                 \
        hipLaunchKernelGGL((ffn_few_kernel<true, SMALL, DIRECT>), dim3(c.f / few_columns(true, SMALL) / up_waves, n_tiles), dim3(64 * up_waves), 0, s, \
                           static_cast<const uint16_t*>(Xp), plan, e_first, static_cast<const char*>(W),              \
                           expert_stride_bytes, size_t(0), static_cast<uint16_t*>(H), c.d, c.f, c.act,                \
                           static_cast<const int32_t*>(nullptr), gather, c.k, c.T * c.k, idx, c.E);                   \
        MOE_LAUNCH_CHECK("ffn_few_kernel<up>");                                                                       \
        if (between != nullptr) MOE_HIP_CHECK(hipEventRecord(between, s));                                            \
        if (SMALL && deep) MOE_FFN_FEW_DOWN(SMALL, DIRECT, SMALL);                                                    \
        else MOE_FFN_FEW_DOWN(SMALL, DIRECT, false);                                                                  \
        MOE_LAUNCH_CHECK("ffn_few_kernel<down>");                                                                     \
    }
            if (idx != nullptr) {
                if (c.T * c.k <= 16) MOE_FFN_FEW(true, true) else MOE_FFN_FEW(false, true)
            } else {
                if (c.T * c.k <= 16) MOE_FFN_FEW(true, false) else MOE_FFN_FEW(false, false)
            }
#undef MOE_FFN_FEW_DOWN
#undef MOE_FFN_FEW
            return MOE_OK;
        }
        FfnLaunch up{Xp, plan, 0, e_first, W, expert_stride_bytes, 0, H, c.d, c.f, c.act, 0, 0, mt_shift, nullptr, gather,
                     gather != nullptr ? c.k : 1, c.T * c.k, 0, max_tiles, 0};
        long items = items_for(slots, mt_shift, (c.f / 32 + 3) / 4, up.y_shift, up.y_chunks);
        if (items > 0x7fffffffL) return fail(MOE_ERR_UNSUPPORTED, "too many work items for one launch (%ld)", items);
        up.grid = static_cast<unsigned>(items < n_cu ? items : n_cu);
        // (with `gather`, Xp is the token array and the kernel looks its rows up itself)
        if (gather != nullptr) launch_ffn_up_gather(up, s);
        else launch_ffn_up(up, s);
        MOE_LAUNCH_CHECK("ffn_mfma_kernel<up>");
        if (between != nullptr) MOE_HIP_CHECK(hipEventRecord(between, s));
        FfnLaunch down{H, plan, 8, e_first, W, expert_stride_bytes, down_off, Yp, c.f, c.d, c.act, 0, 0, mt_shift_down, row_map, nullptr,
                       1, c.T * c.k, down_list, max_tiles, 0};
        items = items_for(slots_down, mt_shift_down, ((cut.narrow ? c.d / 32 : c.d / 64) + 3) / 4, down.y_shift, down.y_chunks);
        if (items > 0x7fffffffL) return fail(MOE_ERR_UNSUPPORTED, "too many work items for one launch (%ld)", items);
        down.grid = static_cast<unsigned>(items < n_cu ? items : n_cu);
        if (cut.narrow) launch_ffn_down_narrow(down, s);
        else launch_ffn_down(down, s);
        MOE_LAUNCH_CHECK("ffn_mfma_kernel<down>");
        return MOE_OK;
    }
    return launch_expert_ffn_f32(c, static_cast<const float*>(Xp), offsets, e_first, e_count, static_cast<const float*>(W),
                                 expert_stride_bytes / 4, max_rows, static_cast<float*>(H), static_cast<float*>(Yp), s, between,
                                 row_map, gather, idx);
}

#endif  // FFN_PART

}  // namespace moe
