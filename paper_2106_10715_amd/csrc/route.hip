// Gate of the MoE layer (CPM-2 Section 2.1: each token picks its expert from its hidden state;
// Section 2.3: the gate is a frozen random projection): logits = x W_g (+ bias), top-k with ties to
// the lower expert index, softmax combine weights.
//
// The selection must be the one exact arithmetic would make.  The kernel therefore accumulates
// in fp32 with a summation order whose rounding error has a small bound (rigorous for the fp32 path; for the matrix
// instruction of the bf16 path, whose inner rounding is not documented, the largest loss ever observed), compares the gaps
// between the k+1 best logits with that bound, and re-evaluates only the tokens that are too close to
// call: products of two bf16 or two fp32 values are exact in fp64, and their sum is carried in two doubles
// (value and rounding error), which holds it exactly for any inputs of comparable magnitude, so that
// columns whose exact projections tie do tie.
#include "common.h"

#include <type_traits>

namespace moe {
namespace {

constexpr int kWaves = 4;      // waves per block
constexpr int kBK = 32;        // terms of one blocked partial sum
constexpr int kNE = 4;         // experts per lane at most (E <= 256, 64 lanes)
constexpr int kSel = 9;        // k + 1 <= 9 ranks are looked at

__device__ inline float ldf(const float* p, size_t i) { return p[i]; }
__device__ inline float ldf(const __bf16* p, size_t i) { return static_cast<float>(p[i]); }

// (value, expert) order of the gate: larger logit first, equal logits -> lower expert index first.  A logit is a
// pair (v, l) whose sum is its value, |l| at most half a unit in the last place of v (l = 0 for logits that were
// not re-evaluated), so pairs compare like their values, part by part.
__device__ inline bool before(double va, double la, int ea, double vb, double lb, int eb) {
    return va > vb || (va == vb && (la > lb || (la == lb && ea < eb)));
}

// Sums in twice the working precision for the re-evaluated logits: the products of two stored values (at most 24
// significant bits each) are exact in fp64, every addition keeps its rounding error (which two floating-point
// numbers always represent exactly) in a second double, and the errors are added up there.  As long as the exact
// sum fits some hundred bits (it does unless the inputs span more than 2^50 in magnitude) the pair holds it without
// any rounding, whatever the order of the terms: columns whose exact projections are equal give identical pairs,
// and a tie is a tie.
__device__ inline void dd_add(double& hi, double& lo, double h2, double l2) {
    const double sum = hi + h2, bb = sum - hi;
    lo += ((hi - (sum - bb)) + (h2 - bb)) + l2;
    hi = sum;
}
__device__ inline void dd_add_product(double& hi, double& lo, double x, double w) { dd_add(hi, lo, x * w, 0.0); }
// (A sum with an infinity in it has no rounding error: what dd_add keeps then is a NaN, and the sum is the high part.)
__device__ inline void dd_normalise(double& hi, double& lo) {
    if (lo != lo) lo = 0.0;
    const double sum = hi + lo, bb = sum - hi;
    lo = fabs(sum) == INFINITY ? 0.0 : (hi - (sum - bb)) + (lo - bb);
    hi = sum;
}

// The kk best of the wave's candidates, in order.  Lane `eg` owns experts eg + 64 i (i < kNE) when
// `owner`; every lane receives the same result.  A NaN ranks with the smallest, so that there are always kk experts.
__device__ __attribute__((always_inline)) inline void wave_topk(const double (&lv)[kNE], const double (&ll)[kNE], int eg, bool owner, int E, int kk,
                                 double (&outv)[kSel], int (&oute)[kSel]) {
    unsigned taken = 0;
#pragma unroll
    for (int r = 0; r < kSel; ++r) {
        if (r < kk) {
            double v = -INFINITY, l = 0.0;
            int e = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < kNE; ++i) {
                const int ei = eg + 64 * i;
                const bool number = lv[i] == lv[i];
                const double lvi = number ? lv[i] : -INFINITY, lli = number ? ll[i] : 0.0;
                if (owner && ei < E && !((taken >> i) & 1u) && before(lvi, lli, ei, v, l, e)) { v = lvi; l = lli; e = ei; }
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double ov = __shfl_xor(v, off), ol = __shfl_xor(l, off);
                const int oe = __shfl_xor(e, off);
                if (before(ov, ol, oe, v, l, e)) { v = ov; l = ol; e = oe; }
            }
            outv[r] = v;
            oute[r] = e;
            if (owner && (e & 63) == eg) taken |= 1u << (e >> 6);
        }
    }
}

// Combine weights of one token from its ranked logits, written by lane 0.  lv: this lane's logits of
// the experts it owns (only read for the full-softmax denominator).
__device__ __attribute__((always_inline)) inline void emit_token(const double (&lv)[kNE], const double (&sv)[kSel], const int (&se)[kSel], int eg, bool owner,
                                  int E, int k, int renorm, int lane, int32_t* __restrict__ idx_row, float* __restrict__ w_row) {
    float wj[kSel];
    float denom = 0.f;
#pragma unroll
    for (int r = 0; r < kSel; ++r)
        if (r < k) wj[r] = expf(static_cast<float>(sv[r] - sv[0]));
    if (renorm) {
#pragma unroll
        for (int r = 0; r < kSel; ++r)
            if (r < k) denom += wj[r];
    } else {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < kNE; ++i)
            if (owner && eg + 64 * i < E) s += expf(static_cast<float>(lv[i] - sv[0]));
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        denom = s;
    }
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < kSel; ++r)
            if (r < k) {
                idx_row[r] = se[r];
                w_row[r] = wj[r] / denom;
            }
    }
}

// Sign-bit gate (the gate of Section 2.3 read as a hashing function): column j of the projection gives
// bit j of the expert id, set when the projection is positive.  Lane j < bits holds projection j in
// lv[0].  gap = the smallest |projection| (how close the token is to a boundary), vmax = the largest.
__device__ __attribute__((always_inline)) inline void sign_bits(const double (&lv)[kNE], const double (&ll)[kNE], int eg, bool owner, int bits, int& code,
                                 double& gap, double& vmax) {
    const bool mine = owner && eg < bits;
    const unsigned long long set = __ballot(mine && (lv[0] > 0.0 || (lv[0] == 0.0 && ll[0] > 0.0)));
    code = static_cast<int>(set & ((1ull << bits) - 1ull));
    double lo = mine ? fabs(lv[0]) : INFINITY, hi = mine ? fabs(lv[0]) : 0.0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off));
        hi = fmax(hi, __shfl_xor(hi, off));
    }
    gap = lo;
    vmax = hi;
}

// Smallest gap between consecutive ranks 0..kk-1 and the largest magnitude among them.
__device__ __attribute__((always_inline)) inline void rank_gaps(const double (&sv)[kSel], int kk, double& gap, double& vmax) {
    gap = INFINITY;
    vmax = 0.0;
#pragma unroll
    for (int r = 0; r < kSel; ++r) {
        if (r < kk) vmax = fmax(vmax, fabs(sv[r]));
        if (r + 1 < kk) gap = fmin(gap, sv[r] - sv[r + 1]);
    }
}

// ---- wave-wide reductions in the lanes' own registers: an inclusive scan by row shifts, then row
// broadcasts, leaves the total in lane 63 (a dozen vector instructions; a butterfly of lane exchanges goes
// through the LDS permute unit six times, some hundred cycles each, and the selection is a chain of them).
template <int CTRL, int ROW_MASK>
__device__ inline unsigned dpp_from(unsigned identity, unsigned v) {
    return static_cast<unsigned>(__builtin_amdgcn_update_dpp(static_cast<int>(identity), static_cast<int>(v), CTRL, ROW_MASK, 0xf, false));
}
__device__ inline unsigned wave_max_u32(unsigned v) {
    v = max(v, dpp_from<0x111, 0xf>(0u, v));      // row_shr:1
    v = max(v, dpp_from<0x112, 0xf>(0u, v));      // row_shr:2
    v = max(v, dpp_from<0x114, 0xf>(0u, v));      // row_shr:4
    v = max(v, dpp_from<0x118, 0xf>(0u, v));      // row_shr:8: lane 15 of every row of 16 holds the row's maximum
    v = max(v, dpp_from<0x142, 0xa>(0u, v));      // row_bcast:15 into rows 1 and 3
    v = max(v, dpp_from<0x143, 0xc>(0u, v));      // row_bcast:31 into rows 2 and 3: lane 63 holds the wave's
    return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
}
__device__ inline unsigned wave_min_u32(unsigned v) { return ~wave_max_u32(~v); }
// The same over a row of 16 lanes, by rotations inside the row: every lane of the row gets the result.
__device__ inline unsigned row_max_u32(unsigned v) {
    v = max(v, dpp_from<0x128, 0xf>(0u, v));      // row_ror:8
    v = max(v, dpp_from<0x124, 0xf>(0u, v));
    v = max(v, dpp_from<0x122, 0xf>(0u, v));
    return max(v, dpp_from<0x121, 0xf>(0u, v));
}
__device__ inline unsigned row_min_u32(unsigned v) { return ~row_max_u32(~v); }
__device__ inline float row_sum_f32(float x) {          // neighbours first: pairs, quads, eights, the row
    auto step = [](float v, unsigned got) { return v + __uint_as_float(got); };
    x = step(x, dpp_from<0xb1, 0xf>(0u, __float_as_uint(x)));      // quad_perm:[1,0,3,2]
    x = step(x, dpp_from<0x4e, 0xf>(0u, __float_as_uint(x)));      // quad_perm:[2,3,0,1]
    x = step(x, dpp_from<0x141, 0xf>(0u, __float_as_uint(x)));     // row_half_mirror: the other quad of the eight
    return step(x, dpp_from<0x128, 0xf>(0u, __float_as_uint(x)));  // row_ror:8: the other eight
}
// fp32 values as unsigned keys of the same order (finite values; -0 must have been turned into +0)
__device__ inline unsigned order_key(float v) {
    const unsigned u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float from_order_key(unsigned key) {
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// The kk largest of the wave's fp32 logits, rank by rank: the largest key of the wave, then the lowest expert that has
// it.  Lane `eg` holds experts eg + 64 i (i < NE) when `owner`; every lane receives the same result.
template <int NE>
__device__ __attribute__((always_inline)) inline void rank_f32(const float (&fv)[NE], int eg, bool owner, int E, int kk,
                                                               double (&sv)[kSel], int (&se)[kSel]) {
    unsigned key[NE], taken = 0;
#pragma unroll
    for (int i = 0; i < NE; ++i) key[i] = owner && eg + 64 * i < E ? order_key(fv[i]) : 0u;
#pragma unroll
    for (int r = 0; r < kSel; ++r) {
        if (r < kk) {
            unsigned bk = 0u, be = 0xffffffffu;
#pragma unroll
            for (int i = 0; i < NE; ++i)
                if (owner && eg + 64 * i < E && !((taken >> i) & 1u) && key[i] > bk) { bk = key[i]; be = static_cast<unsigned>(eg + 64 * i); }
            const unsigned top = wave_max_u32(bk);
            const unsigned who = wave_min_u32(bk == top ? be : 0xffffffffu);
            sv[r] = static_cast<double>(from_order_key(top));
            se[r] = static_cast<int>(who);
            if ((who & 63u) == static_cast<unsigned>(eg)) taken |= 1u << (who >> 6);
        }
    }
}

// TPW: tokens per wave (they share the W_g loads); NE: experts per lane at most.  The kernel is bound by the latency of
// its loads: kUnroll terms are requested at a time (one memory latency for all of them), and a batch too short to give
// every compute unit several waves is handled one token per wave.
// QUADS (fp32; quads of terms requested at a time, 0: single ones): a lane takes four columns and four neighbouring terms at a time, 5 loads of 16 bytes for 16 products
// instead of 32 of 4, wherever W_g has a multiple of four columns, at any address and in every batch, so that a token's bits are the same everywhere.  us, single
// terms / quads: 64 tokens, d 256, 4 experts 5.3 / 4.0, d 1024, 8 11.6 / 5.5, 1100, d 1024, 16 21.8 / 9.4, 4096, d 192, 16 10.6 / 7.4, d 1024, 16 28.6 / 14.6, 5000, d 4096, 32
// 769 / 573; of 441 sizes none is slower. As many at a time as a lane has in all, but no more than 8 (207 registers, two waves of a SIMD), or 4 (116) where there are more blocks than
// two per compute unit: with 8 everywhere 64 tokens, d 256, 4 experts take 0.3 us longer and 4096, d 256, 8 14.4 us instead of 7.0. Four tokens per wave have registers for 2.
template <typename XT, int TPW, int NE, int QUADS = 0>
__global__ __launch_bounds__(kWaves * 64) void route_kernel(const XT* __restrict__ x, const XT* __restrict__ Wg,
                                                            const float* __restrict__ bias,
                                                            int32_t* __restrict__ idx, float* __restrict__ w,
                                                            int T, int d, int E, int k, int renorm, int hash) {
    // hash: E is the number of sign bits (columns of the projection), one expert id per token, weight 1
    constexpr int kUnroll = TPW * NE == 1 ? 32 : NE == 1 ? 16 : 8;
    static_assert(kBK % kUnroll == 0, "a partial sum is a whole number of load batches");
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int t0 = (blockIdx.x * kWaves + wave) * TPW;
    if (t0 >= T) return;                       // whole wave leaves; the kernel has no block-wide barrier

    int EP = 1;                                // lanes that hold distinct experts (power of two, <= 64)
    while (EP < E && EP < 64) EP <<= 1;
    const int KS = 64 / EP;                    // lane groups that split the reduction dimension
    const int eg = lane & (EP - 1);
    const int ks = lane / EP;
    const bool owner = ks == 0;

    size_t xrow[TPW];
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) xrow[tt] = static_cast<size_t>(min(t0 + tt, T - 1)) * d;

    float tot[TPW][NE], wsq[NE], xsq[TPW];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        wsq[i] = 0.f;
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) tot[tt][i] = 0.f;
    }
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) xsq[tt] = 0.f;

    // Blocked summation: partial sums of kBK terms are added into the running total, so a logit goes
    // through at most kBK + ceil(d / (KS kBK)) + log2(KS) + 1 roundings instead of d.
    int span, log2ks = 0;
    if constexpr (QUADS > 0) {
        typedef float quad __attribute__((ext_vector_type(4)));
        typedef float quad_at_4 __attribute__((ext_vector_type(4), aligned(4)));
        constexpr int kAtOnce = QUADS;                             // quads of terms requested at a time, of the kBK / 4 of a partial sum
        static_assert(kBK / 4 % kAtOnce == 0, "a partial sum is a whole number of load batches");
        int EQ = 1;                                // lanes that hold different columns
        while (4 * EQ < E) EQ <<= 1;
        const int KQ = 64 / EQ, cq = lane & (EQ - 1), kq = lane / EQ, col = min(4 * cq, E - 4);
        const bool has_columns = 4 * cq < E;
        span = KQ * kBK;
        quad sum[TPW], wsum = quad{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) sum[tt] = quad{0.f, 0.f, 0.f, 0.f};
        for (int kb = 0; kb < d; kb += span) {
            quad part[TPW];
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) part[tt] = quad{0.f, 0.f, 0.f, 0.f};
            for (int q0 = 0; q0 < kBK / 4 && kb + 4 * KQ * q0 < d; q0 += kAtOnce) {
                // (terms past the end are read from the start of the row and the column and enter as zeros, columns past the last one as well)
                quad xv[kAtOnce][TPW], wv[kAtOnce][4];
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const int k0 = kb + 4 * (kq + KQ * (q0 + u)), at = k0 < d ? k0 : 0;
#pragma unroll
                    for (int tt = 0; tt < TPW; ++tt) xv[u][tt] = *reinterpret_cast<const quad*>(x + xrow[tt] + at);
#pragma unroll
                    for (int r = 0; r < 4; ++r) wv[u][r] = *reinterpret_cast<const quad_at_4*>(Wg + static_cast<size_t>(at + r) * E + col);
                }
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const bool in = kb + 4 * (kq + KQ * (q0 + u)) < d;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        quad wr = wv[u][r];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            wr[c] = in && has_columns ? wr[c] : 0.f;
                            wsum[c] = fmaf(wr[c], wr[c], wsum[c]);
                        }
#pragma unroll
                        for (int tt = 0; tt < TPW; ++tt) {
                            const float xr = in ? xv[u][tt][r] : 0.f;
                            xsq[tt] = fmaf(xr, xr, xsq[tt]);
#pragma unroll
                            for (int c = 0; c < 4; ++c) part[tt][c] = fmaf(xr, wr[c], part[tt][c]);
                        }
                    }
                }
            }
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[tt][c] += part[tt][c];
        }
        if constexpr (NE == 1) {                   // (at most 16 lanes of columns: 4 or more that a column is added up over)
            // In each of the first two steps a lane hands half of its columns over and keeps the sums of the others, the same ones as if both kept all of them: column c ends in the lanes
            // with bits c / 2 and c % 2 in those places. 21 exchanges instead of 58 for a token at 4 columns, 63 instead of 160 for four.
            const bool high = (lane & EQ) != 0, odd = (lane & 2 * EQ) != 0;
            float r[TPW + 1];                      // of the tokens, and the column's square
#pragma unroll
            for (int tt = 0; tt <= TPW; ++tt) {
                const quad v = tt < TPW ? sum[tt < TPW ? tt : 0] : wsum;
                const float k0 = (high ? v[2] : v[0]) + __shfl_xor(high ? v[0] : v[2], EQ), k1 = (high ? v[3] : v[1]) + __shfl_xor(high ? v[1] : v[3], EQ);
                r[tt] = (odd ? k1 : k0) + __shfl_xor(odd ? k0 : k1, 2 * EQ);
                if (tt < TPW) xsq[tt] += __shfl_xor(xsq[tt], EQ);
                if (tt < TPW) xsq[tt] += __shfl_xor(xsq[tt], 2 * EQ);
            }
            log2ks = 2;
            for (int off = 4 * EQ; off < 64; off <<= 1) {
                ++log2ks;
#pragma unroll
                for (int tt = 0; tt <= TPW; ++tt) {
                    r[tt] += __shfl_xor(r[tt], off);
                    if (tt < TPW) xsq[tt] += __shfl_xor(xsq[tt], off);
                }
            }
            wsq[0] = r[TPW];                       // (only their largest is wanted)
            // every column to the lane that ranks it
            const int ei = min(eg, E - 1), from = (ei >> 2) + ((ei & 2) >> 1) * EQ + (ei & 1) * 2 * EQ;
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) {
                const float v = __shfl(r[tt], from);
                tot[tt][0] = eg < E ? v : 0.f;
            }
        } else {
            for (int off = EQ; off < 64; off <<= 1) {
                ++log2ks;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    wsum[c] += __shfl_xor(wsum[c], off);
#pragma unroll
                    for (int tt = 0; tt < TPW; ++tt) sum[tt][c] += __shfl_xor(sum[tt][c], off);
                }
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) xsq[tt] += __shfl_xor(xsq[tt], off);
            }
            // every column to the lanes that rank it: expert e lies in part e % 4 of lane e / 4
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int ei = min(eg + 64 * i, E - 1), from = ei >> 2, c = ei & 3;
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) {
                    const float v0 = __shfl(sum[tt][0], from), v1 = __shfl(sum[tt][1], from), v2 = __shfl(sum[tt][2], from), v3 = __shfl(sum[tt][3], from);
                    tot[tt][i] = eg + 64 * i < E ? (c & 2 ? (c & 1 ? v3 : v2) : (c & 1 ? v1 : v0)) : 0.f;
                }
            }
            wsq[0] = fmaxf(fmaxf(wsum[0], wsum[1]), fmaxf(wsum[2], wsum[3]));       // (only their largest is wanted)
        }
    } else {
        span = KS * kBK;
        for (int kb = 0; kb < d; kb += span) {
            float part[TPW][NE];
#pragma unroll
            for (int i = 0; i < NE; ++i)
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) part[tt][i] = 0.f;
            for (int ii = 0; ii < kBK && kb + ii * KS < d; ii += kUnroll) {
                // d is a multiple of 64 and so of KS: a term is past the end for all lanes or for none.  Such terms are
                // read from the start of the row and the column and enter as zeros.
                float xv[kUnroll][TPW], wv[kUnroll][NE];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const bool in = kb + (ii + u) * KS < d;
                    const int kk = (in ? kb + (ii + u) * KS : 0) + ks;
#pragma unroll
                    for (int tt = 0; tt < TPW; ++tt) xv[u][tt] = in ? ldf(x, xrow[tt] + kk) : 0.f;
#pragma unroll
                    for (int i = 0; i < NE; ++i) {
                        const int ei = eg + 64 * i;
                        const float v = ldf(Wg, static_cast<size_t>(kk) * E + min(ei, E - 1));
                        wv[u][i] = in && ei < E ? v : 0.f;
                    }
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
#pragma unroll
                    for (int tt = 0; tt < TPW; ++tt) {
                        xsq[tt] = fmaf(xv[u][tt], xv[u][tt], xsq[tt]);
#pragma unroll
                        for (int i = 0; i < NE; ++i) part[tt][i] = fmaf(xv[u][tt], wv[u][i], part[tt][i]);
                    }
#pragma unroll
                    for (int i = 0; i < NE; ++i) wsq[i] = fmaf(wv[u][i], wv[u][i], wsq[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < NE; ++i)
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) tot[tt][i] += part[tt][i];
        }
        for (int off = EP; off < 64; off <<= 1) {
            ++log2ks;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                wsq[i] += __shfl_xor(wsq[i], off);
#pragma unroll
                for (int tt = 0; tt < TPW; ++tt) tot[tt][i] += __shfl_xor(tot[tt][i], off);
            }
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt) xsq[tt] += __shfl_xor(xsq[tt], off);
        }
    }
    // largest column norm of W_g among this wave's experts (all lanes end with the wave maximum)
    float wn2 = 0.f;
#pragma unroll
    for (int i = 0; i < NE; ++i) wn2 = fmaxf(wn2, wsq[i]);
    wn2 = __uint_as_float(wave_max_u32(__float_as_uint(wn2)));      // sums of squares: not negative, ordered like their bits
    const float n_round = static_cast<float>(kBK + (d + span - 1) / span + log2ks + 2);

    float bl[kNE];
#pragma unroll
    for (int i = 0; i < kNE; ++i) {
        const int ei = eg + 64 * i;
        bl[i] = (i < NE && bias != nullptr && ei < E) ? bias[ei] : 0.f;
    }

    const int kk_sel = min(k + 1, E);
#pragma unroll
    for (int tt = 0; tt < TPW; ++tt) {
        const int t = t0 + tt;
        if (t >= T) continue;
        double lv[kNE], ll[kNE];                // logits as pairs (value, low part); the low part is 0 for fp32 logits
#pragma unroll
        for (int i = 0; i < kNE; ++i) { lv[i] = i < NE ? static_cast<double>(tot[tt][i < NE ? i : 0] + bl[i]) : 0.0; ll[i] = 0.0; }
        double sv[kSel];
        int se[kSel];
        int code = 0;
        double vmax, gap;
        if (hash) {
            sign_bits(lv, ll, eg, owner, E, code, gap, vmax);
        } else {
            float fv[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) fv[i] = (tot[tt][i] + bl[i]) + 0.0f;      // a -0 becomes +0: equal logits must compare equal
            rank_f32<NE>(fv, eg, owner, E, kk_sel, sv, se);
            rank_gaps(sv, kk_sel, gap, vmax);
        }
        // |computed - exact| <= n_round u |x_t| |W_g col| + u |logit| for every logit that matters
        // (Cauchy-Schwarz bounds the sum of |products|); 1/16 of slack covers the fp32 norms themselves.
        const double delta = 1.0625 * 5.9604644775390625e-8 *
                             (static_cast<double>(n_round) * sqrt(static_cast<double>(xsq[tt]) * static_cast<double>(wn2)) + vmax);
        if (gap <= 2.0 * delta) {
            // too close to call in fp32: exact products, sums in twice the fp64 precision
            double acc[NE], low[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) { acc[i] = 0.0; low[i] = 0.0; }
            for (int kk = ks; kk < d; kk += KS) {
                const double xv = static_cast<double>(ldf(x, xrow[tt] + kk));
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    const int ei = eg + 64 * i;
                    if (ei < E) dd_add_product(acc[i], low[i], xv, static_cast<double>(ldf(Wg, static_cast<size_t>(kk) * E + ei)));
                }
            }
            for (int off = EP; off < 64; off <<= 1)
#pragma unroll
                for (int i = 0; i < NE; ++i) {
                    const double oh = __shfl_xor(acc[i], off), ol = __shfl_xor(low[i], off);
                    dd_add(acc[i], low[i], oh, ol);
                }
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                dd_add(acc[i], low[i], static_cast<double>(bl[i]), 0.0);
                dd_normalise(acc[i], low[i]);
                lv[i] = acc[i];
                ll[i] = low[i];
            }
            if (hash) sign_bits(lv, ll, eg, owner, E, code, gap, vmax);
            else wave_topk(lv, ll, eg, owner, E, kk_sel, sv, se);
        }
        if (hash) {
            if (lane == 0) { idx[t] = code; w[t] = 1.f; }
        } else {
            emit_token(lv, sv, se, eg, owner, E, k, renorm, lane, idx + static_cast<size_t>(t) * k,
                       w + static_cast<size_t>(t) * k);
        }
    }
}

// ------------------------------------------------------------------------------------------ bf16: MFMA gate
//
// logits tile = 32 tokens (64, 16) x E on 16x16x32 bf16 MFMAs.  The eight waves of a block split the reduction
// dimension (wave w takes the 64-element groups S = w, w+8, ...), the partial tiles are added in wave
// order through LDS.  W_g is first rewritten (gate_prep_kernel) into fragments whose 16-byte pieces are
// operand pieces: fragment (nb, S, q), slot l, element j holds
//     W_g[64 S + 32 (l / 32) + 8 q + j, 32 nb + l % 32]            (0 beyond E).
//
// Error bound of an MFMA logit, empirical in one constant: the addends of an instruction (accumulator and products) behave as if
// aligned to the largest of them and cut to fp32 precision, so that one 16x16x32 instruction, 33 addends, loses at most 34 x 2^-24
// of its largest addend, which is at most the sum of |products|.  34.0 is also the largest loss seen over 10^8 random
// instructions (with all addends of one sign, whose sum is then some thirty times the largest); it is used without a margin of
// its own, beside the 1/16 on the whole bound.  |error| <= (17 n + 8) 2^-24 |x_t| |W_g column| with n = two per instruction a
// wave chains per logit.  Tokens whose k+1 best logits are not separated by twice that are re-evaluated from exact products by
// the whole block.

constexpr int kGateWaves = 8;    // waves of a gate block; they split the reduction dimension

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Block b packs the 64-row group S = b of W_g for every 32-expert block and writes the sums of squares
// of those 64 rows per expert column: part[b][E_pad].
__global__ __launch_bounds__(256) void gate_prep_kernel(const uint16_t* __restrict__ Wg, int d, int E, int NB,
                                                        uint4* __restrict__ pack, float* __restrict__ part) {
    __shared__ float sq[4][32];
    const int S = blockIdx.x, nS = d / 64;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;      // wave q packs fragment q of the group
    const int col_in = lane & 31, row0 = 64 * S + 32 * (lane >> 5) + 8 * q;
    for (int nb = 0; nb < NB; ++nb) {
        const int col = 32 * nb + col_in;
        uint16_t v[8];
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            v[j] = col < E ? Wg[static_cast<size_t>(row0 + j) * E + col] : uint16_t(0);
            const float f = __uint_as_float(static_cast<uint32_t>(v[j]) << 16);
            ss = fmaf(f, f, ss);
        }
        uint4 o;
        o.x = v[0] | (static_cast<uint32_t>(v[1]) << 16);
        o.y = v[2] | (static_cast<uint32_t>(v[3]) << 16);
        o.z = v[4] | (static_cast<uint32_t>(v[5]) << 16);
        o.w = v[6] | (static_cast<uint32_t>(v[7]) << 16);
        pack[((static_cast<size_t>(nb) * nS + S) * 4 + q) * 64 + lane] = o;
        ss += __shfl_xor(ss, 32);
        if (lane < 32) sq[q][lane] = ss;
        __syncthreads();
        if (threadIdx.x < 32)
            part[static_cast<size_t>(S) * NB * 32 + col] = ((sq[0][col_in] + sq[1][col_in]) + sq[2][col_in]) + sq[3][col_in];
        __syncthreads();
    }
}

// Where the gate kernel finds the gate: the packed fragments, or (RAW) W_g itself, whose 16-byte pieces it then puts together.
template <bool RAW>
struct Gate {
    const void* gate;
    int nS, E;
    // the piece of rows 64 S + 32 h + 8 q .. + 8 of a column (0 beyond E)
    __device__ __attribute__((always_inline)) uint4 piece(int col, int S, int q, int h) const {
        if constexpr (!RAW) return static_cast<const uint4*>(gate)[((static_cast<size_t>(col >> 5) * nS + S) * 4 + q) * 64 + h * 32 + (col & 31)];
        const uint16_t* from = static_cast<const uint16_t*>(gate) + static_cast<size_t>(64 * S + 32 * h + 8 * q) * E + min(col, E - 1);
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = from[static_cast<size_t>(j) * E];
        const uint32_t keep = col < E ? ~0u : 0u;
        return uint4{(v[0] | v[1] << 16) & keep, (v[2] | v[3] << 16) & keep, (v[4] | v[5] << 16) & keep, (v[6] | v[7] << 16) & keep};
    }
};

// Values of two columns of the projection of token t from exact products, by one wave, from the packed fragments: lane j
// takes the 8-row pieces j, j + 64, ... of the columns; sums in twice the fp64 precision, the pairs (hi, lo) not yet normalised.
// Every lane gets the sums.
template <bool RAW>
__device__ __attribute__((always_inline)) inline void exact_dots(const uint16_t* __restrict__ x, const Gate<RAW>& gate, size_t t,
                                                     const int (&col)[2], int nS, int d, int lane, double (&hi)[2], double (&lo)[2]) {
    constexpr int U = 4;                   // pieces requested at once
    const uint4* xr = reinterpret_cast<const uint4*>(x + t * d);
    const int pieces = nS * 8;
    hi[0] = hi[1] = lo[0] = lo[1] = 0.0;
    for (int j0 = 0; j0 < pieces; j0 += 64 * U) {
        uint4 xq[U], wq[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + 64 * u < pieces) {                                 // uniform
                const int j = min(j0 + 64 * u + lane, pieces - 1);
                const int S = j >> 3, q = (j & 7) >> 1, h = j & 1;      // rows 64 S + 32 h + 8 q .. + 8
                xq[u] = xr[S * 8 + h * 4 + q];
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    wq[u][c] = gate.piece(col[c], S, q, h);
            }
        }
        asm volatile("" : : : "memory");
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (j0 + 64 * u < pieces) {
                const bool in = j0 + 64 * u + lane < pieces;            // past the end: zeros, which change nothing
                const uint32_t xu[4] = {in ? xq[u].x : 0u, in ? xq[u].y : 0u, in ? xq[u].z : 0u, in ? xq[u].w : 0u};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const double x0 = static_cast<double>(__uint_as_float(xu[i] << 16)), x1 = static_cast<double>(__uint_as_float(xu[i] & 0xffff0000u));
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const uint32_t wu = i == 0 ? wq[u][c].x : i == 1 ? wq[u][c].y : i == 2 ? wq[u][c].z : wq[u][c].w;
                        dd_add_product(hi[c], lo[c], x0, static_cast<double>(__uint_as_float(wu << 16)));
                        dd_add_product(hi[c], lo[c], x1, static_cast<double>(__uint_as_float(wu & 0xffff0000u)));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double oh = __shfl_xor(hi[c], off), ol = __shfl_xor(lo[c], off);
            dd_add(hi[c], lo[c], oh, ol);
        }
    }
}

constexpr int kMaxCand = 12;     // columns of one token that are re-evaluated one by one; more than that: all columns

constexpr int gate_row(int columns) { return columns + 4; }      // floats per tile row: the four lane groups of a tile write hit different banks
template <int NB>
constexpr int gate_parts() { return NB <= 4 ? kGateWaves : 1; }      // one partial tile per wave while they fit the LDS
constexpr int gate_rows(int tok) { return tok > 32 ? tok : 32; }     // token rows of a tile
// TOK: tokens of a block (64, 32, 16 or 8; with 8, the 16 rows of a matrix tile repeat them).  A short batch gets more,
// smaller blocks: a block's time is mostly its own loads through one compute unit, and 128 blocks leave half the chip idle.
// A long one gets fewer, larger ones: every block reads the whole gate from the L2, beside its own tokens.
// PAIRS: two blocks per compute unit, of 128 registers a thread, where there are that many: one ranks its tokens and decides the close ones while the other loads.
// The gate fragments are then requested half a group ahead, the token pieces two groups.  us, one block / two (64 experts): 16384 tokens, d 4096 57.3 / 54.5, 32768
// 95.7 / 88.2, 16384, d 2048 32.6 / 29.7, 20000, d 1024 34.6 / 25.0; with a block more per compute unit for some only, 10000, d 4096 44.1 / 45.8, 8192 28.6 /
// 29.9; 32 experts, whose blocks of 64 tokens take less of the gate, 16384 42.4 / 44.5.  (On another box 16384, d 4096 49.1 / 43.2, d 1024 26.3 / 18.2.)  The 128
// registers are not quite enough: 92 bytes per thread go to scratch memory and come back, in the loops over close tokens.
// RAW: `pack` is W_g itself, for a matrix that is not packed and of at most 512 rows, one group of 64 for each wave: its pieces are put together from single
// values, all requested at once, and its column norms are added up on the way, in the order of gate_prep_kernel, whose launch that saves. us, packed by the call / RAW: 1025
// tokens, d 320, 33 experts 11.0 / 8.3, 500, d 512, 64 10.5 / 7.8, 300, d 512, 8 10.7 / 8.0, 4000, d 512, 31 13.1 / 11.1, 2500, d 448, 64 13.2 / 12.2.
template <int NB, int TOK, bool PAIRS = false, bool RAW = false>
__global__ __launch_bounds__(kGateWaves * 64, PAIRS ? 4 : 2) void route_mfma_kernel(const uint16_t* __restrict__ x,
                                                         const uint4* __restrict__ pack, const float* __restrict__ part,
                                                         const float* __restrict__ bias, int32_t* __restrict__ idx,
                                                         float* __restrict__ w, int T, int d, int E, int k, int renorm,
                                                         int hash) {
    // hash: E is the number of sign bits (columns of the projection), one expert id per token, weight 1
    constexpr int EP = NB * 32;
    constexpr int kParts = gate_parts<NB>(), kRows = gate_rows(TOK);
    __shared__ __align__(16) float part_tile[kParts * kRows * gate_row(EP)];     // [kParts][kRows][gate_row(EP)]: partial logit tiles
    __shared__ float xsq_w[kGateWaves][kRows];
    __shared__ float colpart[kGateWaves * 64];             // partial column sums of squares (up to 512 columns' worth)
    __shared__ unsigned long long close_sh;                     // tokens fp32 cannot decide, one bit each
    __shared__ unsigned long long many_sh;                      // and those with more columns in reach than are evaluated one by one
    __shared__ unsigned long long tied_sh;                      // close tokens that fp64 cannot decide either
    __shared__ uint8_t reach_count[kRows], reach_col[kRows][kMaxCand];    // columns of a close token that can change its answer
    // their sums from exact products, eight tokens at a time: fp64 by slices of the reduction, or pairs (high, low)
    __shared__ double close_sum[kGateWaves][kGateWaves][kMaxCand];
    // partial sums of all columns, value and low part, of kMany tokens: in the logit tiles, which are not needed any more then
    constexpr int kMany = kParts == kGateWaves ? kGateWaves : 1;
    static_assert(kMany == 1 || kMany * kGateWaves * EP * 4 <= kParts * kRows * gate_row(EP), "the sums fit the tiles");
    __shared__ double2 pair_sh[kMany == 1 ? kGateWaves * EP : 1];
    auto tile_at = [&](int p, int tok, int e) -> float& { return part_tile[(p * kRows + tok) * gate_row(EP) + e]; };

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int t0 = blockIdx.x * TOK;
    const int nS = d / 64;
    const Gate<RAW> gate{pack, nS, E};

    // ---- column norms of W_g, for the error bound: thread (g, c) adds the per-group sums S = g, g + G, ... of column c; the
    // partial sums are added up where they are used, after the barrier that publishes the logits.  The first kNorm
    // are requested before everything else and added once the loads below are on their way.
    constexpr int G = EP >= kGateWaves * 64 ? 1 : kGateWaves * 64 / EP, kNorm = 8;
    const int norm_c = static_cast<int>(threadIdx.x) % EP, norm_g = static_cast<int>(threadIdx.x) / EP;
    float norm[kNorm];                     // (threads past the last whole group of columns, EP = 96 and others, hold unused sums)
#pragma unroll
    for (int i = 0; i < kNorm && !RAW; ++i) {
        const int S = norm_g + i * G;
        norm[i] = part[static_cast<size_t>(S < nS ? S : 0) * EP + norm_c];
    }
    asm volatile("" : : : "memory");

    // A wave's groups of 64 reduction elements are S = wave, wave + 8, ...  Products on 16x16x32: in k-step m of a group, lane
    // 16 g + c holds elements 64 S + 32 m + 8 g + j of token row c (and of column c), so that a load of token pieces covers 64
    // contiguous bytes of 16 rows (one lane per 16 bytes of 32 rows, as 32x32x16 wants it, takes the address unit twice as
    // long: 40 cycles per load, which bounded the kernel); the gate fragment holds those elements at slot 32 m + 16 cb + c of its part g.
    constexpr int RB = TOK > 16 ? TOK / 16 : 1;                  // 16-row blocks; 8 tokens: every row twice
    const int c15 = lane & 15, g4 = lane >> 4;
    uint32_t x_lane[RB];                                   // byte offsets from x (T d 2 < 2^32)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
        x_lane[rb] = static_cast<uint32_t>(min(t0 + ((16 * rb + c15) & (TOK - 1)), T - 1)) * static_cast<uint32_t>(d) * 2u + 64u * (g4 & 1) + 16u * (g4 >> 1);
    const uint32_t w_lane = 1024u * (g4 >> 1) + 512u * (g4 & 1) + 16u * c15;
    auto x_piece = [&](int S, int m, int rb) __attribute__((always_inline)) {
        return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(x) + static_cast<size_t>(S) * 128 + 32 * m + x_lane[rb]);
    };
    auto w_piece = [&](int S, int nb, int m, int cb) __attribute__((always_inline)) {
        if constexpr (RAW) return gate.piece(32 * nb + 16 * cb + c15, S, 2 * m + (g4 >> 1), g4 & 1);
        return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(pack) + (static_cast<size_t>(nb) * nS + S) * 4096 + 2048 * m + 256 * cb + w_lane);
    };
    struct XGroup { uint4 v[2][RB]; };
    struct WHalf { uint4 v[NB][2]; };                      // of one k-step
    struct WGroup { uint4 v[NB][2][2]; };
    f32x4 acc[RB][NB][2];
    float xs[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        xs[rb] = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[rb][nb][0] = acc[rb][nb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // k-step m of a group; gate(nb, cb): the fragment of column half cb of block nb
    auto multiply_step = [&](const XGroup& xg, int m, auto&& gate) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const uint4 piece = xg.v[m][rb];
            const uint32_t u[4] = {piece.x, piece.y, piece.z, piece.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float lo = __uint_as_float(u[i] << 16), hi = __uint_as_float(u[i] & 0xffff0000u);
                xs[rb] = fmaf(lo, lo, xs[rb]);
                xs[rb] = fmaf(hi, hi, xs[rb]);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                    acc[rb][nb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, piece),
                                                                              __builtin_bit_cast(bf16x8, gate(nb, cb)), acc[rb][nb][cb], 0, 0, 0);
        }
    };
    auto multiply = [&](const XGroup& xg, const WGroup& wg) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 2; ++m) multiply_step(xg, m, [&](int nb, int cb) __attribute__((always_inline)) { return wg.v[nb][m][cb]; });
    };
    auto load_x = [&](int S, XGroup& dst) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int m = 0; m < 2; ++m) dst.v[m][rb] = x_piece(S, m, rb);
    };
    auto load_w = [&](int S, WGroup& dst) __attribute__((always_inline)) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) dst.v[nb][m][cb] = w_piece(S, nb, m, cb);
    };
    // RAW: the sums of squares of the wave's one group, the block's place for column c of wave w
    auto norms_of_group = [&](const WGroup& wg, bool has) __attribute__((always_inline)) {
        float mine = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                float ss[2];                                   // rows 8 q .. of both halves, q = 2 m + g / 2
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const uint4 v = wg.v[nb][m][cb];
                    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
                    ss[m] = 0.f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float lo = __uint_as_float(u[i] << 16), hi = __uint_as_float(u[i] & 0xffff0000u);
                        ss[m] = fmaf(lo, lo, ss[m]);
                        ss[m] = fmaf(hi, hi, ss[m]);
                    }
                    ss[m] += __shfl_xor(ss[m], 16);
                }
                const float other = __shfl_xor(ss[1], 32), q2 = g4 >> 1 ? other : ss[1], q3 = g4 >> 1 ? ss[1] : other;
                const float total = ((ss[0] + __shfl_xor(ss[0], 32)) + q2) + q3;
                if (EP == 64 ? (lane >> 5 == nb && ((lane >> 4) & 1) == cb) : lane >> 4 == cb) mine = total;
            }
        colpart[threadIdx.x] = has ? mine : 0.f;               // (32 columns: the wave's other 32 lanes add zeros)
        if (threadIdx.x == 0) close_sh = many_sh = tied_sh = 0ull;
    };
    auto norms_to_lds = [&]() __attribute__((always_inline)) {
        float ssum = 0.f;
#pragma unroll
        for (int i = 0; i < kNorm; ++i) ssum += norm_g + i * G < nS ? norm[i] : 0.f;
        for (int S = norm_g + kNorm * G; S < nS; S += G) ssum += part[static_cast<size_t>(S) * EP + norm_c];
        colpart[threadIdx.x] = ssum;
        if (threadIdx.x == 0) close_sh = many_sh = tied_sh = 0ull;
    };

    // ---- MFMA partial tiles
    if constexpr (NB <= 2) {
        // The token pieces come from HBM: a ring of kXDepth groups is requested ahead, for as many groups as the registers
        // hold (at d_model 4096 a wave has eight).  The gate fragments, which every block re-reads from the L2, are requested
        // kWRing - 1 groups ahead, the first ones before the token pieces (loads return in order).
        constexpr int kXDepth = PAIRS || TOK == 64 ? 2 : TOK == 32 && NB == 2 ? 4 : 8, kWRing = 2;
        const int n_mine = (nS - wave + kGateWaves - 1) / kGateWaves;      // this wave's groups (0 when d is short)
        XGroup xv[kXDepth];
        // The odd waves take their groups from the middle on: with all waves of all blocks at the same place of rows that lie a
        // power of two apart, half of the memory channels would idle (8192 tokens, d 4096: 31.6 -> 25.2 us at 8 experts, 34.4 ->
        // 29.7 at 64).  The order depends on the wave only, so a logit has the same bits wherever its token lies in the batch.
        const int phase = wave & 1 ? n_mine / 2 : 0;
        auto group_of = [&](int i) {
            const int r = i + phase < n_mine ? i + phase : i + phase - n_mine;
            return i < n_mine ? wave + r * kGateWaves : 0;                 // past the end: group 0, unused
        };
        // (a fence after every batch of loads: the compiler would move them down to their use)
        auto fetch_x = [&](int i, XGroup& dst) __attribute__((always_inline)) {
            load_x(group_of(i), dst);
            asm volatile("" : : : "memory");
        };
        auto fetch_w = [&](int i, WGroup& dst) __attribute__((always_inline)) {
            load_w(group_of(i), dst);
            asm volatile("" : : : "memory");
        };
        if constexpr (RAW) {
            static_assert(EP <= 64, "a column for each lane of a wave");
            WGroup wg;
            fetch_w(0, wg);
            fetch_x(0, xv[0]);
            norms_of_group(wg, n_mine > 0);
            if (n_mine > 0) multiply(xv[0], wg);                           // uniform for the wave
        } else if constexpr (PAIRS) {
            WHalf half[2];
            auto fetch_half = [&](int i, int m, WHalf& dst) __attribute__((always_inline)) {
                const int S = group_of(i);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) dst.v[nb][cb] = w_piece(S, nb, m, cb);
                asm volatile("" : : : "memory");
            };
            auto gate_of = [](const WHalf& h) __attribute__((always_inline)) { return [&h](int nb, int cb) __attribute__((always_inline)) { return h.v[nb][cb]; }; };
            fetch_half(0, 0, half[0]);
#pragma unroll
            for (int p = 0; p < kXDepth; ++p) fetch_x(p, xv[p]);
            norms_to_lds();
            for (int i0 = 0; i0 < n_mine; i0 += kXDepth) {
#pragma unroll
                for (int p = 0; p < kXDepth; ++p) {
                    const int i = i0 + p;
                    fetch_half(i, 1, half[1]);
                    if (i < n_mine) multiply_step(xv[p], 0, gate_of(half[0]));     // uniform for the wave
                    fetch_half(i + 1, 0, half[0]);
                    if (i < n_mine) multiply_step(xv[p], 1, gate_of(half[1]));
                    fetch_x(i + kXDepth, xv[p]);
                }
            }
        } else {
            WGroup wv[kWRing];
#pragma unroll
            for (int p = 0; p + 1 < kWRing; ++p) fetch_w(p, wv[p]);
            fetch_x(0, xv[0]);
            if (TOK >= 32 || n_mine > 1) {               // (short batches: nothing to request ahead when d is short)
#pragma unroll
                for (int p = 1; p < kXDepth; ++p) fetch_x(p, xv[p]);
            }
            norms_to_lds();
            for (int i0 = 0; i0 < n_mine; i0 += kXDepth) {
                auto groups = [&](auto more) __attribute__((always_inline)) {  // more: the ring is refilled behind the groups used
#pragma unroll
                    for (int p = 0; p < kXDepth; ++p) {
                        const int i = i0 + p;
                        if ((p + kWRing - 1 < kXDepth && (TOK >= 32 || n_mine > 1)) || decltype(more)::value) fetch_w(i + kWRing - 1, wv[(p + kWRing - 1) % kWRing]);
                        if (i < n_mine) multiply(xv[p], wv[p % kWRing]);       // uniform for the wave
                        if (decltype(more)::value) fetch_x(i + kXDepth, xv[p]);
                    }
                };
                if (i0 + kXDepth < n_mine) groups(std::true_type{});
                else groups(std::false_type{});
            }
        }
    } else {
        // more expert blocks: as many groups of token pieces at a time and gate fragments ahead as the registers hold
        constexpr int kAhead = NB <= 4 ? 2 : 1;
        norms_to_lds();
        for (int S0 = wave; S0 < nS; S0 += kGateWaves * kAhead) {
            XGroup xv[kAhead];
            WGroup wv[2];
            auto group_of = [&](int p) { return S0 + p * kGateWaves < nS ? S0 + p * kGateWaves : S0; };
#pragma unroll
            for (int p = 0; p < kAhead; ++p) load_x(group_of(p), xv[p]);
            load_w(S0, wv[0]);
#pragma unroll
            for (int p = 0; p < kAhead; ++p) {
                if (p + 1 < kAhead) load_w(group_of(p + 1), wv[(p + 1) % 2]);
                if (S0 + p * kGateWaves < nS) multiply(xv[p], wv[p % 2]);  // uniform for the wave
            }
        }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        xs[rb] += __shfl_xor(xs[rb], 16);
        xs[rb] += __shfl_xor(xs[rb], 32);
        if (lane < 16) xsq_w[wave][16 * rb + lane] = xs[rb];
    }
    // accumulator v of lane 16 g + c: token 4 g + v of its row block, column c of its half block
    // The partial tiles are added in wave order: by the lane that reads a logit when every wave has a tile of its own,
    // else wave after wave into one tile.
    auto each_value = [&](auto&& put) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) put(16 * rb + 4 * g4 + v, 32 * nb + 16 * cb + c15, acc[rb][nb][cb][v]);
    };
    if (kParts == kGateWaves) {
        each_value([&](int tok, int col, float v) { tile_at(wave, tok, col) = v; });
        __syncthreads();
    } else {
        for (int turn = 0; turn < kGateWaves; ++turn) {
            if (wave == turn)
                each_value([&](int tok, int col, float v) {
                    float& at = tile_at(0, tok, col);
                    at = turn == 0 ? v : at + v;
                });
            __syncthreads();
        }
    }

    // ---- selection
    // largest column norm: every wave adds up the partial sums for itself
    float wn2_f = 0.f;
    for (int c = lane; c < EP; c += 64) {
        float tot = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g) tot += colpart[g * EP + c];
        wn2_f = fmaxf(wn2_f, tot);
    }
    wn2_f = __uint_as_float(wave_max_u32(__float_as_uint(wn2_f)));         // sums of squares: not negative, ordered like their bits
    const int n_chain = ((nS + kGateWaves - 1) / kGateWaves) * 4;                               // 16-row steps a wave chains per logit
    const double gamma = 1.0625 * 5.9604644775390625e-8 * static_cast<double>(17 * n_chain + 8);
    constexpr int NE = (NB + 1) / 2;         // experts a lane holds: eg, eg + 64, ... (kNE at most)
    const int eg = lane;
    const int kk_sel = min(k + 1, E);
    const double wn2 = static_cast<double>(wn2_f);
    // logit of (token, column): the partial tiles added in wave order, ((w0 + w1) + w2) + ..., and the bias
    auto logit = [&](int tt, int e) __attribute__((always_inline)) {
        float sum = tile_at(0, tt, e);
        if (kParts > 1) {
#pragma unroll
            for (int pw = 1; pw < kParts; ++pw) sum += tile_at(pw, tt, e);
        }
        return sum;
    };
    auto token_norm2 = [&](int tt) __attribute__((always_inline)) {
        float v = xsq_w[0][tt];
#pragma unroll
        for (int wv = 1; wv < kGateWaves; ++wv) v += xsq_w[wv][tt];
        return static_cast<double>(v);
    };
    // Sixteen lanes (one row of the cross-lane moves) per token, lane j of the row holds columns j, j + 16, ...: a wave ranks
    // four tokens at once, a block 32.  The selection is a latency chain per rank (largest key
    // of the row, then the lowest column that has it); one token per wave after the other, it took longer than the products.
    for (int first = wave * 4; first < TOK; first += 4 * kGateWaves) {
        constexpr int NL = EP / 16;
        const int j0 = lane & 15, tt = first + (lane >> 4), t = t0 + tt;
        const bool real = t < T;
        const int tr = real ? t : T - 1;             // past the end: as the last token, nothing is written
        float fv[NL];
        unsigned key[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int c = j0 + 16 * i, cc = c < E ? c : 0;                 // columns past the end read column 0 and drop it
            fv[i] = (logit(tt, cc) + (bias != nullptr && c < E ? bias[cc] : 0.f)) + 0.0f;   // a -0 becomes +0: equal logits must compare equal
            key[i] = c < E ? order_key(fv[i]) : 0u;
        }
        double gap, vmax, reach_from = 0.0;
        if (hash) {
            unsigned set = 0u, least = 0x7f800000u, most = 0u;
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (j0 + 16 * i < E) {
                    const unsigned mag = __float_as_uint(fabsf(fv[i]));
                    set |= fv[i] > 0.f ? 1u << (j0 + 16 * i) : 0u;
                    least = min(least, mag);
                    most = max(most, mag);
                }
            set |= dpp_from<0x128, 0xf>(0u, set);
            set |= dpp_from<0x124, 0xf>(0u, set);
            set |= dpp_from<0x122, 0xf>(0u, set);
            set |= dpp_from<0x121, 0xf>(0u, set);
            gap = static_cast<double>(__uint_as_float(row_min_u32(least)));
            vmax = static_cast<double>(__uint_as_float(row_max_u32(most)));
            if (real && j0 == 0) { idx[tr] = static_cast<int>(set); w[tr] = 1.f; }
        } else {
            double sv[kSel];
            int se[kSel];
            unsigned taken = 0;
#pragma unroll
            for (int r = 0; r < kSel; ++r) {
                if (r < kk_sel) {
                    unsigned bk = 0u, be = 0xffffffffu;
#pragma unroll
                    for (int i = 0; i < NL; ++i)
                        if (!((taken >> i) & 1u) && key[i] > bk) { bk = key[i]; be = static_cast<unsigned>(j0 + 16 * i); }
                    const unsigned top = row_max_u32(bk);
                    const unsigned who = row_min_u32(bk == top ? be : 0xffffffffu);
                    sv[r] = static_cast<double>(from_order_key(top));
                    se[r] = static_cast<int>(who);
                    if ((who & 15u) == static_cast<unsigned>(j0)) taken |= 1u << (who >> 4);
                }
            }
            rank_gaps(sv, kk_sel, gap, vmax);
#pragma unroll
            for (int r = 0; r < kSel; ++r)
                if (r + 1 == kk_sel) reach_from = sv[r];
            float wj[kSel], denom = 0.f;
#pragma unroll
            for (int r = 0; r < kSel; ++r)
                if (r < k) wj[r] = expf(static_cast<float>(sv[r] - sv[0]));
            if (renorm) {
#pragma unroll
                for (int r = 0; r < kSel; ++r)
                    if (r < k) denom += wj[r];
            } else {
                // in the order a wave adds 64 columns at a time: columns 16 r .. 16 r + 15 of every 64, then the four of them
                float part_sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < NL; ++i)
                    if (j0 + 16 * i < E) part_sum[i & 3] += expf(static_cast<float>(static_cast<double>(fv[i]) - sv[0]));
#pragma unroll
                for (int r = 0; r < 4; ++r) part_sum[r] = row_sum_f32(part_sum[r]);
                denom = (part_sum[3] + part_sum[2]) + (part_sum[1] + part_sum[0]);
            }
            if (real && j0 == 0) {
#pragma unroll
                for (int r = 0; r < kSel; ++r)
                    if (r < k) {
                        idx[static_cast<size_t>(tr) * k + r] = se[r];
                        w[static_cast<size_t>(tr) * k + r] = wj[r] / denom;
                    }
            }
        }
        // Too close to call in fp32 (the answer is written above all the same, and again below).  Which columns can exact
        // arithmetic still change it for?  Top-k: every logit within 2 delta of the (k+1)-th best, or above it (anything
        // lower stays below all of those even with both errors against it).  Sign bits: every projection within 2 delta
        // of zero.  Usually two or three columns; the others keep their fp32 values, which cannot reach the selected ones.
        const double delta = gamma * sqrt(token_norm2(tt) * wn2) + 1.0625 * 5.9604644775390625e-8 * vmax;
        const bool close = real && gap <= 2.0 * delta;                     // the same in the whole row
        if (__any(close)) {
            const double reach = hash ? 2.0 * delta : reach_from - 2.0 * delta;
            int count = 0;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const double v = static_cast<double>(fv[i]);
                const bool in = close && j0 + 16 * i < E && (hash ? fabs(v) <= reach : v >= reach);
                const unsigned in_row = static_cast<unsigned>(__ballot(in) >> (lane & 48)) & 0xffffu;
                const int at = count + __popc(in_row & ((1u << j0) - 1u));
                if (in && at < kMaxCand) reach_col[tt][at] = static_cast<uint8_t>(j0 + 16 * i);
                count += __popc(in_row);
            }
            if (close && j0 == 0) {
                reach_count[tt] = static_cast<uint8_t>(count);             // (looked at up to kMaxCand only; E = 256 in reach: many_sh)
                atomicOr(count > kMaxCand ? &many_sh : &close_sh, 1ull << tt);
            }
        }
    }
    float bl[kNE];
#pragma unroll
    for (int i = 0; i < kNE; ++i) bl[i] = i >= NE ? 0.f : (bias != nullptr && eg + 64 * i < E) ? bias[eg + 64 * i] : 0.f;
    __syncthreads();

    // ---- the tokens fp32 cannot decide, by the whole block: one of them in a block would otherwise keep a single wave busy for
    // longer than all the rest of the kernel takes
    auto uniform64 = [](unsigned long long v) {
        const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
        const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)));
        return static_cast<unsigned long long>(hi) << 32 | lo;
    };
    unsigned long long todo = uniform64(close_sh);
    // Eight tokens at a time: all waves take the exact products of their columns in reach in turn, then wave i decides for token i.
    // In fp64 a job is four columns in one slice of the reduction (at d_model 4096 an eighth, one 8-row piece per lane), and
    // wave i adds the slices in order.  Where that leaves the decision inside its rounding error (in practice: exact ties), a job
    // is two whole columns in twice the precision.  A sum is the same whichever wave takes it.
    // Against eighths of every sum, empty ones too, and all pairs of a token by one wave, column by column: 16384 tokens, d 4096,
    // 32 experts 46 -> 40 us; 16384 tokens that all tie, d 1024, 8 experts 465 -> 240, 32 experts (all columns) 480 -> 249.
    const int slices = min(kGateWaves, (nS + 7) / 8);
    while (todo != 0ull) {                           // the same in every wave
        const unsigned long long batch = todo;
        int tokens = 0;
        for (; tokens < kGateWaves && todo != 0ull; ++tokens) todo &= todo - 1ull;
        auto token = [&](int n) {                    // the n-th token of the batch
            unsigned long long m = batch;
            for (int skip = n; skip > 0; --skip) m &= m - 1ull;
            return __ffsll(static_cast<long long>(m)) - 1;
        };
        auto columns_of = [&](int tt) { return __builtin_amdgcn_readfirstlane(static_cast<int>(reach_count[tt])); };
        auto column = [&](int tt, int c) { return __builtin_amdgcn_readfirstlane(static_cast<int>(reach_col[tt][c])); };
        int job = 0;
        for (int n = 0; n < tokens; ++n) {
            const int tt = token(n), cols = columns_of(tt);
            for (int c0 = 0; c0 < cols; c0 += 4, job += slices) {
                const int slice = (wave - job) & (kGateWaves - 1);                  // the one of these jobs that falls to this wave
                if (slice >= slices) continue;
                const uint4* xr = reinterpret_cast<const uint4*>(x + static_cast<size_t>(t0 + tt) * d);
                int col[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) col[c] = column(tt, min(c0 + c, cols - 1));
                double sum[4] = {0.0, 0.0, 0.0, 0.0};
                for (int j0 = slice * 64; j0 < nS * 8; j0 += kGateWaves * 64) {
                    const int j = min(j0 + lane, nS * 8 - 1);
                    const bool in = j0 + lane < nS * 8;
                    const int S = j >> 3, q = (j & 7) >> 1, h = j & 1;               // rows 64 S + 32 h + 8 q .. + 8
                    const uint4 xq = xr[S * 8 + h * 4 + q];
                    const uint32_t xu[4] = {xq.x, xq.y, xq.z, xq.w};
                    uint4 wq[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        wq[c] = gate.piece(col[c], S, q, h);
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t wu[4] = {wq[c].x, wq[c].y, wq[c].z, wq[c].w};
                        double part_sum = 0.0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            part_sum = fma(static_cast<double>(__uint_as_float(xu[i] << 16)), static_cast<double>(__uint_as_float(wu[i] << 16)), part_sum);
                            part_sum = fma(static_cast<double>(__uint_as_float(xu[i] & 0xffff0000u)),
                                           static_cast<double>(__uint_as_float(wu[i] & 0xffff0000u)), part_sum);
                        }
                        sum[c] += in ? part_sum : 0.0;
                    }
                }
                // over the lanes; the columns part on the way: lanes 16 c .. 16 c + 15 end with column c
                const bool upper = lane >= 32, odd = (lane & 16) != 0;
                const double got0 = __shfl_xor(upper ? sum[0] : sum[2], 32), got1 = __shfl_xor(upper ? sum[1] : sum[3], 32);
                const double both0 = (upper ? sum[2] : sum[0]) + got0, both1 = (upper ? sum[3] : sum[1]) + got1;
                double total = (odd ? both1 : both0) + __shfl_xor(odd ? both0 : both1, 16);
#pragma unroll
                for (int off = 8; off >= 1; off >>= 1) total += __shfl_xor(total, off);
                if ((lane & 15) == 0 && c0 + (lane >> 4) < cols) close_sum[n][slice][c0 + (lane >> 4)] = total;
            }
        }
        const int tt = token(wave < tokens ? wave : 0), t = t0 + tt, cols = columns_of(tt);
        double sv[kSel];
        int se[kSel];
        int code = 0;
        double gap, vmax;
        double lv[kNE], ll[kNE];                     // value and low part of the columns this lane holds; from NE on: no expert, never looked at
#pragma unroll
        for (int i = 0; i < kNE; ++i) lv[i] = ll[i] = 0.0;
        // Lane c of the wave adds up column c in reach, and ranks it by looking at the others.  The columns out of reach stay below the
        // k + 1 best, so their logits are only needed for the sign bits, for the denominator of the full softmax, or where infinities and
        // NaNs leave the columns in reach without an order of their own; then all columns are gone through.
        // (Column by column and slice by slice, with an exchange among all lanes per rank, this took 4-6 us of the kernel: 1025 tokens x 2 on
        // 33 experts, d 320 11.6 -> 10.4 us; 4096 tokens on 32, d 4096 26 -> 21; 2048 on 8 22 -> 18.5; 16384 x 2 on 64 56 -> 52.)
        auto decide = [&](bool pairs) __attribute__((always_inline)) {
            const int c = min(lane, cols - 1), at = max(c, 0);
            const int mine = reach_col[tt][at];
            double slice_sum[kGateWaves];
#pragma unroll
            for (int v = 0; v < kGateWaves; ++v) slice_sum[v] = close_sum[wave][v][at];
            double hi = slice_sum[0], lo = pairs ? slice_sum[1] : 0.0;
#pragma unroll
            for (int v = 1; v < kGateWaves; ++v)
                if (!pairs && v < slices) hi += slice_sum[v];
            float b = 0.f;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const float got = __shfl(bl[i], mine & 63);
                if (mine >> 6 == i) b = got;
            }
            dd_add(hi, lo, static_cast<double>(b), 0.0);
            dd_normalise(hi, lo);
            if (!pairs) lo = 0.0;
            auto from_lane = [](double v, int l) __attribute__((always_inline)) {
                const uint64_t bits = __builtin_bit_cast(uint64_t, v);
                const unsigned low = __builtin_amdgcn_readlane(static_cast<int>(bits), l), high = __builtin_amdgcn_readlane(static_cast<int>(bits >> 32), l);
                return __builtin_bit_cast(double, static_cast<uint64_t>(high) << 32 | low);
            };
            bool ordered = false;
            if (!hash && cols >= kk_sel) {           // uniform
                int rank = 0;
                for (int j = 0; j < cols; ++j)
                    rank += before(from_lane(hi, j), from_lane(lo, j), __builtin_amdgcn_readlane(mine, j), hi, lo, mine) ? 1 : 0;
                if (lane >= cols) rank = kSel;
                ordered = true;
#pragma unroll
                for (int r = 0; r < kSel; ++r)
                    if (r < kk_sel) {
                        const unsigned long long who = __ballot(rank == r);
                        ordered = ordered && __popcll(who) == 1;
                        const int l = who != 0ull ? __ffsll(static_cast<long long>(who)) - 1 : 0;
                        sv[r] = from_lane(hi, l);
                        se[r] = __builtin_amdgcn_readlane(mine, l);
                    }
            }
            if (hash || !renorm || !ordered) {       // uniform
#pragma unroll
                for (int i = 0; i < NE; ++i) {       // fp32, a -0 becomes +0: equal logits must compare equal
                    const int ei = eg + 64 * i, ec = ei < E ? ei : 0;      // lanes without an expert read column 0 and drop it
                    lv[i] = ei < E ? static_cast<double>((logit(tt, ec) + bl[i]) + 0.0f) : 0.0;
                    ll[i] = 0.0;
                }
                for (int j = 0; j < cols; ++j) {
                    const double vj = from_lane(hi, j), lj = from_lane(lo, j);
                    const int col = __builtin_amdgcn_readlane(mine, j);
#pragma unroll
                    for (int i = 0; i < NE; ++i)
                        if (eg + 64 * i == col) { lv[i] = vj; ll[i] = lj; }
                }
                if (hash) sign_bits(lv, ll, eg, true, E, code, gap, vmax);
                else if (!ordered) wave_topk(lv, ll, eg, true, E, kk_sel, sv, se);
            }
            if (!hash) rank_gaps(sv, kk_sel, gap, vmax);
        };
        auto emit = [&]() __attribute__((always_inline)) {
            if (hash) {
                if (lane == 0) { idx[t] = code; w[t] = 1.f; }
            } else {
                emit_token(lv, sv, se, eg, true, E, k, renorm, lane, idx + static_cast<size_t>(t) * k, w + static_cast<size_t>(t) * k);
            }
        };
        __syncthreads();
        bool tied = false;
        if (wave < tokens) {
            decide(false);
            const double delta64 = 1.0625 * 1.1102230246251565e-16 * (static_cast<double>(d + 8) * sqrt(token_norm2(tt) * wn2) + 2.0 * vmax);
            tied = gap <= 2.0 * delta64;
            if (!tied) emit();
            else if (lane == 0) atomicOr(&tied_sh, 1ull << tt);
        }
        __syncthreads();
        const unsigned long long ties = uniform64(tied_sh) & batch;
        if (ties == 0ull) continue;
        job = 0;
        for (int n = 0; n < tokens; ++n) {
            const int t2 = token(n), cols2 = columns_of(t2);
            if (((ties >> t2) & 1ull) == 0ull) continue;
            for (int c = 0; c < cols2; c += 2, ++job) {
                if (job % kGateWaves != wave) continue;
                const int last = min(c + 1, cols2 - 1);
                const int col[2] = {column(t2, c), column(t2, last)};
                double hi[2], lo[2];
                exact_dots(x, gate, static_cast<size_t>(t0 + t2), col, nS, d, lane, hi, lo);
                if (lane == 0) {
                    close_sum[n][0][c] = hi[0];
                    close_sum[n][1][c] = lo[0];
                    if (last > c) { close_sum[n][0][last] = hi[1]; close_sum[n][1][last] = lo[1]; }
                }
            }
        }
        __syncthreads();
        if (tied) {
            decide(true);
            emit();
        }
        __syncthreads();                             // the sums have been read
    }
    unsigned long long many = uniform64(many_sh);
    auto pair_at = [&](int n, int wv, int c) -> double2& {
        return kMany == 1 ? pair_sh[wv * EP + c] : reinterpret_cast<double2*>(part_tile)[(n * kGateWaves + wv) * EP + c];
    };
    while (many != 0ull) {                           // the same in every wave
        const unsigned long long batch = many;
        int tokens = 0;
        for (; tokens < kMany && many != 0ull; ++tokens) {
            const int tt = __ffsll(static_cast<long long>(many)) - 1, t = t0 + tt;
            many &= many - 1ull;
            // More than kMaxCand columns in reach: all columns in fp64 pairs, from the same packed fragments and with the same split as
            // the MFMA pass: wave w takes the groups S = w, w+8, ..., lane (c, h) the 32 rows 64 S + 32 h .. of column c of
            // every expert block; the two halves are added by a lane exchange, the waves in wave order.
            const uint4* xr = reinterpret_cast<const uint4*>(x + static_cast<size_t>(t) * d + 32 * (lane >> 5));
            double a64[NB], l64[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) { a64[nb] = 0.0; l64[nb] = 0.0; }
            for (int S = wave; S < nS; S += kGateWaves) {
                uint4 xa[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) xa[q] = xr[S * 8 + q];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    uint4 wb[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) wb[q] = gate.piece(32 * nb + (lane & 31), S, q, lane >> 5);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t xu[4] = {xa[q].x, xa[q].y, xa[q].z, xa[q].w};
                        const uint32_t wu[4] = {wb[q].x, wb[q].y, wb[q].z, wb[q].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            dd_add_product(a64[nb], l64[nb], static_cast<double>(__uint_as_float(xu[i] << 16)),
                                           static_cast<double>(__uint_as_float(wu[i] << 16)));
                            dd_add_product(a64[nb], l64[nb], static_cast<double>(__uint_as_float(xu[i] & 0xffff0000u)),
                                           static_cast<double>(__uint_as_float(wu[i] & 0xffff0000u)));
                        }
                    }
                }
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const double oh = __shfl_xor(a64[nb], 32), ol = __shfl_xor(l64[nb], 32);
                dd_add(a64[nb], l64[nb], oh, ol);
                if (lane < 32) pair_at(tokens, wave, 32 * nb + lane) = double2{a64[nb], l64[nb]};
            }
        }
        __syncthreads();
        if (wave < tokens) {                         // wave i finishes token i
            unsigned long long mine = batch;
            for (int skip = wave; skip > 0; --skip) mine &= mine - 1ull;
            const int t = t0 + __ffsll(static_cast<long long>(mine)) - 1;
            double lv[kNE], ll[kNE];
#pragma unroll
            for (int i = 0; i < kNE; ++i) {
                const int ei = eg + 64 * i;
                double sum = 0.0, low = 0.0;
                if (ei < E) {
                    for (int wv = 0; wv < kGateWaves; ++wv) {
                        const double2 part_pair = pair_at(wave, wv, ei);
                        dd_add(sum, low, part_pair.x, part_pair.y);
                    }
                    dd_add(sum, low, static_cast<double>(bl[i]), 0.0);
                    dd_normalise(sum, low);
                }
                lv[i] = sum;
                ll[i] = low;
            }
            if (hash) {
                int code;
                double gap, vmax;
                sign_bits(lv, ll, eg, true, E, code, gap, vmax);
                if (lane == 0) { idx[t] = code; w[t] = 1.f; }
            } else {
                double sv[kSel];
                int se[kSel];
                wave_topk(lv, ll, eg, true, E, kk_sel, sv, se);
                emit_token(lv, sv, se, eg, true, E, k, renorm, lane, idx + static_cast<size_t>(t) * k, w + static_cast<size_t>(t) * k);
            }
        }
        __syncthreads();
    }
}

}  // namespace

int gate_columns(const moe_cfg& c) {
    if (c.gate != MOE_GATE_HASH) return c.E;
    int bits = 0;
    while ((1 << bits) < c.E) ++bits;
    return bits;
}

size_t route_scratch_bytes(const moe_cfg& c) {
    if (c.dtype != MOE_BF16) return 0;
    const size_t EP = static_cast<size_t>((gate_columns(c) + 31) / 32) * 32;
    return align256(EP * c.d * 2) + align256(static_cast<size_t>(c.d / 64) * EP * 4);
}

size_t gate_packed_bytes(const moe_cfg& c) {
    if (c.dtype == MOE_BF16) return route_scratch_bytes(c);
    return align256(static_cast<size_t>(c.d) * gate_columns(c) * 4);
}

// The gate in the form the gate kernel reads: bf16, fragments in MFMA operand order followed by the sums of
// squares of every 64-row group of every column; fp32, the matrix itself.
int launch_pack_gate(const moe_cfg& c, const void* Wg, void* packed, hipStream_t s) {
    const int cols = gate_columns(c);
    if (c.dtype == MOE_BF16) {
        const int NB = (cols + 31) / 32;
        const size_t EP = static_cast<size_t>(NB) * 32;
        float* part = reinterpret_cast<float*>(static_cast<char*>(packed) + align256(EP * c.d * 2));
        hipLaunchKernelGGL(gate_prep_kernel, dim3(c.d / 64), dim3(256), 0, s, static_cast<const uint16_t*>(Wg), c.d, cols, NB,
                           static_cast<uint4*>(packed), part);
        MOE_LAUNCH_CHECK("gate_prep_kernel");
        return MOE_OK;
    }
    MOE_HIP_CHECK(hipMemcpyAsync(packed, Wg, static_cast<size_t>(c.d) * cols * 4, hipMemcpyDeviceToDevice, s));
    return MOE_OK;
}

int launch_route(const moe_cfg& c, const void* x, const void* Wg, const float* bias, int32_t* idx, float* w,
                 void* scratch, hipStream_t s) {
    if (c.T == 0) return MOE_OK;
    const int hash = c.gate == MOE_GATE_HASH ? 1 : 0;
    const int cols = gate_columns(c);          // columns of the gate matrix: experts, or sign bits
    int dev = 0;
    const DeviceInfo* info = nullptr;
    if (int rc = device_info(&dev, &info)) return rc;
    const int n_cu = info->compute_units;
    if (c.dtype == MOE_BF16) {
        const int NB = (cols + 31) / 32;
        const size_t EP = static_cast<size_t>(NB) * 32;
        // a gate packed once by the caller (it is frozen: Section 2.3) is read where it lies; else it is packed
        // into the workspace first, by every call
        // (but for short reductions and batches, where the kernel is as well off with the matrix itself: RAW)
        const bool raw = !c.gate_packed && NB <= 2 && c.d <= 64 * kGateWaves && (c.T + 15) / 16 < n_cu;
        if (!c.gate_packed && !raw)
            if (int rc = launch_pack_gate(c, Wg, scratch, s)) return rc;
        const char* gate = static_cast<const char*>(c.gate_packed || raw ? Wg : scratch);
        const uint4* pack = reinterpret_cast<const uint4*>(gate);
        const float* part = reinterpret_cast<const float*>(gate + align256(EP * c.d * 2));
        // as many tokens per block as still give every compute unit a block
        const int tok = raw ? 8 : NB == 1 && (c.T + 63) / 64 >= n_cu ? 64 : (c.T + 31) / 32 >= n_cu ? 32 : (c.T + 15) / 16 >= n_cu ? 16 : 8;
        dim3 grid((c.T + tok - 1) / tok), block(kGateWaves * 64);
        // (close to two blocks for every compute unit, or more)
        const bool pairs = NB == 2 && tok == 32 && 10L * grid.x >= 19L * n_cu;
#define MOE_ROUTE_LAUNCH(N, TK) MOE_ROUTE_LAUNCH_AS((route_mfma_kernel<N, TK>))
#define MOE_ROUTE_LAUNCH_AS(KERNEL)                                                                                   \
    hipLaunchKernelGGL(KERNEL, grid, block, 0, s, static_cast<const uint16_t*>(x), pack, part, bias, idx,  \
                       w, c.T, c.d, cols, c.k, c.renorm, hash)
#define MOE_ROUTE_CASE(N)                                                                                             \
    case N:                                                                                                           \
        if (raw) MOE_ROUTE_LAUNCH_AS((route_mfma_kernel<(N <= 2 ? N : 1), 8, false, true>));                          \
        else if (tok == 64) MOE_ROUTE_LAUNCH(1, 64);                                                                       \
        else if (pairs) MOE_ROUTE_LAUNCH_AS((route_mfma_kernel<2, 32, true>));                                        \
        else if (tok == 32) MOE_ROUTE_LAUNCH(N, 32);                                                                  \
        else if (tok == 16) MOE_ROUTE_LAUNCH(N, 16);                                                                  \
        else MOE_ROUTE_LAUNCH(N, 8);                                                                                  \
        break;
        switch (NB) {
            MOE_ROUTE_CASE(1) MOE_ROUTE_CASE(2) MOE_ROUTE_CASE(3) MOE_ROUTE_CASE(4)
            MOE_ROUTE_CASE(5) MOE_ROUTE_CASE(6) MOE_ROUTE_CASE(7) MOE_ROUTE_CASE(8)
            default: return fail(MOE_ERR_UNSUPPORTED, "E = %d is out of range", c.E);
        }
#undef MOE_ROUTE_LAUNCH
#undef MOE_ROUTE_LAUNCH_AS
#undef MOE_ROUTE_CASE
        MOE_LAUNCH_CHECK("route_mfma_kernel");
        return MOE_OK;
    }
    // one token per wave up to 16 waves per compute unit, then four
    const int tpw = c.T <= 4096 ? 1 : 4;
    const int per_block = kWaves * tpw;
    dim3 grid((c.T + per_block - 1) / per_block), block(kWaves * 64);
    const bool quads = cols % 4 == 0;
    const bool rounds = c.T > 2 * kWaves * n_cu;
    int lanes = 1;                             // that hold different columns
    while (4 * lanes < cols) lanes <<= 1;
#define MOE_ROUTE_F32(TPW, NE, QUADS)                                                                                 \
    hipLaunchKernelGGL((quads ? route_kernel<float, TPW, NE, QUADS> : route_kernel<float, TPW, NE, 0>), grid, block, 0, s, static_cast<const float*>(x),               \
                       static_cast<const float*>(Wg), bias, idx, w, c.T, c.d, cols, c.k, c.renorm, hash)
    if (tpw == 1) {
        if (cols <= 64) {
            if (static_cast<long>(c.d) * lanes <= 2 * 4 * 64) MOE_ROUTE_F32(1, 1, 2); else if (rounds) MOE_ROUTE_F32(1, 1, 4); else MOE_ROUTE_F32(1, 1, 8);
        } else {
            if (rounds) MOE_ROUTE_F32(1, kNE, 4); else MOE_ROUTE_F32(1, kNE, 8);
        }
    } else {
        if (cols <= 64) MOE_ROUTE_F32(4, 1, 2); else MOE_ROUTE_F32(4, kNE, 2);
    }
#undef MOE_ROUTE_F32
    MOE_LAUNCH_CHECK("route_kernel");
    return MOE_OK;
}

}  // namespace moe
