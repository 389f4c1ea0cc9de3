// Dense 16-bit attention of one agent's query rows over its private, uncompressed continuation: the work of one wave.
#pragma once
#include <hip/hip_fp16.h>

#include "polykv_internal.hpp"
#include "polykv_layout.hpp"

namespace polykv {

constexpr int kTailRows = 4;   // query rows of one wave

typedef _Float16 tail_half8 __attribute__((ext_vector_type(8)));
typedef __bf16 tail_bf8 __attribute__((ext_vector_type(8)));
typedef float tail_float4 __attribute__((ext_vector_type(4)));
typedef uint32_t tail_uint4 __attribute__((ext_vector_type(4)));

template <bool BF> __device__ __forceinline__ tail_float4 tail_mfma(const tail_uint4& a, const tail_uint4& b, const tail_float4& c) {
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(tail_bf8, a), __builtin_bit_cast(tail_bf8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(tail_half8, a), __builtin_bit_cast(tail_half8, b), c, 0, 0, 0);
}

template <int ROR> __device__ __forceinline__ float tail_ror(float x) {   // lane (i - ROR) % 16 of the 16-lane row
    const int xi = __float_as_int(x);
    return __int_as_float(__builtin_amdgcn_update_dpp(xi, xi, 0x120 + ROR, 0xF, 0xF, false));
}
// Two numbers, each to be added over lanes l and l ^ 32 (l ^ 16): lanes with that bit clear get a's sum, the others b's.
__device__ __forceinline__ float tail_add32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float tail_add16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float tail_max64(float x) {   // over the lanes that share lane % 4
    x = fmaxf(x, tail_ror<4>(x));
    x = fmaxf(x, tail_ror<8>(x));
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float tail_sum64(float x) {
    x += tail_ror<4>(x);
    x += tail_ror<8>(x);
    x = tail_add16(x, x);
    return tail_add32(x, x);
}

// A wave's tokens in one round: all their keys and values are requested at once.
constexpr int tail_block_tokens(int D) { return D == 256 ? 32 : 64; }

// Rows [4 zb, 4 zb + 4) of agent a, selected unit usel -> (m, l) in tail_ml and the unnormalized sum, in the original
// value domain, in tail_o.  `a`, `usel`, `zb` are wave-uniform; p_s: tail_block_tokens(D) * 4 floats of LDS of the wave's
// own.  No barriers: waves of one workgroup may run through here with different lengths.
//
// What bounds it: HBM at many tokens and agents, the chain request -> scores -> softmax -> sums of a single wave at few.
// Per block of 64 tokens (32 at head_dim 256):
//   loads   keys and values are all requested before the first one is used, through buffer resources that end with the
//           agent's tokens: lanes past the end read zeros and touch no memory;
//   scores  16 tokens x 16 columns per matrix instruction, key rows straight from memory as the A operand, no staging.
//           The four query rows fill the 16 columns four times over, so that each of a row's scores sits in four lanes, and
//           each of those takes a fourth of the exponentials; maxima and sums over tokens are two DPP steps and two lane
//           swaps.  (Packed dot products over key rows staged in LDS, with the queries broadcast from there and 48
//           ds_bpermute steps in the reductions: a call of 15 agents with 64-token tails over 7,194 tokens took 125.5 us,
//           116.3 us this way; a step of 32 one-layer calls with 32-token tails 673 and 573 us.)
//   P.V     in fp32 on the vector ALU: lane = (token slot, 8 coordinates), one 16-byte load covers a lane's 8
//           coordinates of a token; the slots are added once at the very end, by lane swaps that leave every lane with
//           the row it stores.
template <int D, bool BF>
__device__ __forceinline__ void tail_rows(const __half* __restrict__ Q, const TailPtrs& tails, float* __restrict__ tail_ml,
                                          float* __restrict__ tail_o, const AttendPlan& p, int a, int usel, int zb, int lane,
                                          float* p_s) {
    constexpr int LPR = D / 8;             // lanes per value row
    constexpr int TPL = 64 / LPR;          // tokens per wave load (token slots)
    constexpr int TB = tail_block_tokens(D), NT = TB / 16, NJ = D / 32, NLD = TB / TPL;
    int kvh, in_group;
    const int ls = p.div_H.divide(usel, &kvh);
    const int rows_a = p.nq * p.G;         // rows of this agent within the KV head, contiguous
    const int r0 = a * rows_a + zb * kTailRows;
    const int r_end = min((a + 1) * rows_a, r0 + kTailRows);
    if (r0 >= r_end) return;
    const int len = tails.len[a];
    const int g = lane >> 4, col = lane & 15, row = col & 3, copy = col >> 2;
    // tokens the lane's row may see: all of them, or, for a causal multi-token step, one less for every query position
    // before the agent's last (row r0 + row is query (zb * 4 + row) / G)
    const int qi = p.div_G.divide(zb * kTailRows + row, &in_group);
    const int row_len = p.tail_causal ? max(0, len - (p.nq - 1 - min(qi, p.nq - 1))) : len;
    const size_t head_off = ((size_t)(p.layer_begin + ls) * p.H + kvh) * p.tail_capacity * D;
    uint16_t* Kt = const_cast<uint16_t*>(reinterpret_cast<const uint16_t*>(tails.K[a])) + head_off;
    uint16_t* Vt = const_cast<uint16_t*>(reinterpret_cast<const uint16_t*>(tails.V[a])) + head_off;

    tail_uint4 q[NJ];   // (rows past the agent's last repeat it; nothing of them is stored)
    {
        const __half* src = Q + q_row_index(p, ls, kvh, min(r0 + row, r_end - 1)) * D + 8 * g;
#pragma unroll
        for (int j = 0; j < NJ; ++j) q[j] = *reinterpret_cast<const tail_uint4*>(src + 32 * j);
    }
    const int slot = lane / LPR, piece = lane - slot * LPR;
    float m_run = -INFINITY, l_run = 0.0f, acc[kTailRows][8];
#pragma unroll
    for (int r = 0; r < kTailRows; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[r][c] = 0.0f;

    for (int t0 = 0; t0 < len; t0 += TB) {
        const int cnt = min(TB, len - t0);
        const auto rk = __builtin_amdgcn_make_buffer_rsrc(Kt + (size_t)t0 * D, 0, cnt * D * 2, 0x00020000);
        const auto rv = __builtin_amdgcn_make_buffer_rsrc(Vt + (size_t)t0 * D, 0, cnt * D * 2, 0x00020000);
        tail_uint4 k[NT][NJ], v[NLD];
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                k[i][j] = __builtin_amdgcn_raw_buffer_load_b128(rk, ((16 * i + col) * D + 32 * j + 8 * g) * 2, 0, 0);
#pragma unroll
        for (int u = 0; u < NLD; ++u) v[u] = __builtin_amdgcn_raw_buffer_load_b128(rv, ((u * TPL + slot) * D + 8 * piece) * 2, 0, 0);
        __builtin_amdgcn_sched_barrier(0);   // all requested before the first use
        float s[NT];
        float m_blk = -INFINITY;
#pragma unroll
        for (int i = 0; i < NT; ++i) {   // S: row `row`, tokens 16 i + 4 g + 0..3; the lane keeps token + copy
            tail_float4 S = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) S = tail_mfma<BF>(k[i][j], q[j], S);
            const float sv = (copy & 2) ? ((copy & 1) ? S[3] : S[2]) : ((copy & 1) ? S[1] : S[0]);
            s[i] = t0 + 16 * i + 4 * g + copy < row_len ? sv * p.qscale : -INFINITY;
            m_blk = fmaxf(m_blk, s[i]);
        }
        const float m_new = fmaxf(m_run, tail_max64(m_blk));
        // a row that has seen no token yet keeps m = -inf: nothing to rescale, every weight 0
        const float alpha = m_new == -INFINITY ? 1.0f : exp2f(m_run - m_new);
        float l_blk = 0.0f;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const float pr = m_new == -INFINITY ? 0.0f : exp2f(s[i] - m_new);
            l_blk += pr;
            p_s[64 * i + lane] = pr;     // [token][row]: (16 i + 4 g + copy) * 4 + row
        }
        l_run = l_run * alpha + tail_sum64(l_blk);
        m_run = m_new;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the wave's own LDS accesses complete in order
        __builtin_amdgcn_wave_barrier();
        if (t0 > 0) {
#pragma unroll
            for (int r = 0; r < kTailRows; ++r) {
                const float al = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(alpha), r));
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[r][c] *= al;
            }
        }
#pragma unroll
        for (int u0 = 0; u0 < NLD; u0 += 4) {
            if (u0 * TPL < cnt) {
#pragma unroll
                for (int u = u0; u < u0 + 4; ++u) {
                    const float4 pr4 = *reinterpret_cast<const float4*>(p_s + 4 * (u * TPL + slot));
                    const float pr[4] = {pr4.x, pr4.y, pr4.z, pr4.w};
#pragma unroll
                    for (int c2 = 0; c2 < 4; ++c2) {
                        const float2 f = pair16_to_float2(v[u][c2], BF);
#pragma unroll
                        for (int r = 0; r < kTailRows; ++r) {
                            acc[r][2 * c2] = fmaf(pr[r], f.x, acc[r][2 * c2]);
                            acc[r][2 * c2 + 1] = fmaf(pr[r], f.y, acc[r][2 * c2 + 1]);
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // read before the next block's probabilities replace them
        __builtin_amdgcn_wave_barrier();
    }

    // ---- the token slots' shares are added; lanes 16 r .. end up with row r (head_dim 256: a half wave with two rows)
    const size_t prow0 = (size_t)usel * p.R + r0;
    if (g == 0 && copy == 0 && r0 + row < r_end)
        *reinterpret_cast<float2*>(tail_ml + (prow0 + row) * 2) = make_float2(m_run, l_run);
    if constexpr (D == 256) {
        float y[2][8];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
#pragma unroll
            for (int c = 0; c < 8; ++c) y[x][c] = tail_add32(acc[x][c], acc[x + 2][c]);
            const int r = x + 2 * (lane >> 5);
            if (r0 + r < r_end) {
                float4* dst = reinterpret_cast<float4*>(tail_o + (prow0 + r) * D + 8 * piece);
                dst[0] = make_float4(y[x][0], y[x][1], y[x][2], y[x][3]);
                dst[1] = make_float4(y[x][4], y[x][5], y[x][6], y[x][7]);
            }
        }
    } else {
        float y[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (D == 64) {   // eight slots: lanes l and l ^ 8 first
#pragma unroll
                for (int r = 0; r < kTailRows; ++r) acc[r][c] += tail_ror<8>(acc[r][c]);
            }
            y[c] = tail_add16(tail_add32(acc[0][c], acc[2][c]), tail_add32(acc[1][c], acc[3][c]));
        }
        if (r0 + g < r_end) {
            float4* dst = reinterpret_cast<float4*>(tail_o + (prow0 + g) * D + 8 * piece);
            if (D == 64) {   // lanes l and l ^ 8 hold the same: a half each
                const bool up = lane & 8;
                dst[up ? 1 : 0] = make_float4(up ? y[4] : y[0], up ? y[5] : y[1], up ? y[6] : y[2], up ? y[7] : y[3]);
            } else {
                dst[0] = make_float4(y[0], y[1], y[2], y[3]);
                dst[1] = make_float4(y[4], y[5], y[6], y[7]);
            }
        }
    }
}

}  // namespace polykv
