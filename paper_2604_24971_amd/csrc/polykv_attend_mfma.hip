// Matrix-core decode attention over the packed pool (gfx950, v_mfma_f32_32x32x16_f16).
//
// One wave owns up to 64 query rows (NT tiles of 32) of one KV head and streams 32-token tile
// records.  Per tile, with tokens as the MFMA M dimension and query rows as N:
//
//   staging  a lane's share of a record (its key-code runs, a token's scales, its value codes -- every wave load
//            one contiguous run) is loaded into registers one step ahead of its use, piece by piece.
//   pipeline two tiles are in flight per wave: the scores of the next tile are computed on the matrix
//            cores while the vector ALUs run the softmax and value dequantization of the current one.
//   scores   S^T[t, r] = sum_j s[t,j] * (sum_{k in block j} code[t,k] * q[r,k]): the keys enter the matrix cores as
//            their integer codes, exact in fp16, and the q8_0 block scales are applied in fp32 to the products of a
//            block (two K=16 MFMAs) as they are summed.
//   softmax  online, per row, in base-2 units; a row's reference only moves when the row's probabilities
//            of one tile sum to more than 2^15 in a lane, so the accumulator rescale is rare, p fits
//            fp16, and the common case takes no maximum over the scores at all.
//   PV       O^T[v, r] += sum_t c[code[t, v]] * p[t, r]   with the score tile's accumulator layout
//            feeding the B operand directly (the value codes are stored in that k-order), centroids
//            looked up with byte permutes.  The softmax denominator is summed from the very same
//            fp16-rounded p with packed dot products.
//
// Why 32x32x16: a wave that interleaves MFMAs with vector work pays 5 to 8 issue cycles per MFMA whatever its shape and
// 4 to 5 per vector instruction, so the larger tile halves the MFMA share of the issue time for the same arithmetic.
//
// What bounds it: with 64 rows a workgroup, the issue of vector instructions by a lone wave per SIMD, at a clock that follows
// the operands.  15 agents over 4,096 tokens are 93,800 cycles a wave (14,770 vector and 1,024 matrix instructions; the matrix
// pipe is busy for 32,800, 17,600 are waits).  By its time that is a clock of 2.08 GHz behind the codec kernels of the bench
// step (45.1 us), 1.92 back to back (48.9 us), 2.29 over zeros (41.0 us).  Fewer cycles alone do not shorten it: deeper requests
// (two sets of tile data, every piece asked for two steps ahead) and a loop rearranged to 7 % fewer cycles changed nothing or
// lost 1 to 2 %.  With 32 rows, HBM and the fixed parts around the loop, 8 to 12 us of a call.
// What the forms of the scores took, us a call (15 agents x 4,096 tokens at R = 60; 64 agents x 4 queries x 7,194 tokens):
//   the exact dequantized key, 18 bits, as two fp16 terms and two products     61.4    1,624
//   codes less their offset (2 packed subtractions per 4 codes), fold          55      1,470 (1,165 in die order, 1,097 with own rows)
// Codes as stored, offset by 128 (fp16 subnormals, no subtraction), with 128 times the queries' sums taken away by a product of
// their own per score tile, ran 1,024 rows in 1,069 instead of 1,089 us, calls of 5 rows in 27.3 instead of 27.7 and 15 agents in
// the same time, but the fp32 sums lose up to log2(128 / |code|) bits, most where a block has one massive channel and small codes
// otherwise: with queries near 1,000 errors of 4.4e-4 to 1.8e-3, where the rounding of the probabilities makes 0.3e-4 or less.
// With accumulators and queries in vector registers where waves share a SIMD (see parks) and the codes' products folded in
// place, one statement an element, calls of 5 rows take 27.7 instead of 28.7 us and int8 values 42.2 instead of 42.7.
//
// The accumulation stays in the rotated value domain; the inverse Walsh-Hadamard rotation is done
// once per output row (sections "Compression Scheme" / "TurboQuant", dequantization), in this kernel
// when one workgroup covers the whole token range and there are no private tails, else in the merge
// kernel.  The four waves of a workgroup take interleaved tiles and are merged through LDS, or, where there
// are rows for it, have rows of their own (OWN, below).
#include <hip/hip_fp16.h>

#include <mutex>
#include <type_traits>

#include "polykv_internal.hpp"
#include "polykv_layout.hpp"
#include "polykv_tail.hpp"

namespace polykv {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

union H8 {
    half8 h;
    uint32_t u[4];
    half2v p[4];
};

__device__ __forceinline__ float16v mfma32(const half8& a, const half8& b, const float16v& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// The same with the result in vector registers (the compiler gives the builtin's result to accumulation registers in
// this kernel, which vector instructions cannot read): C = 0, and C = D.  The compiler does not know what is inside, so
// the call sites keep the distances the instruction asks for: two instructions between the vector write of an operand
// and the product that reads it, and at least twelve between the product and a vector read of its result.
// WAIT: with two wait states of its own in front, where an operand may have been moved just before.
// BA: the second operand is in accumulation registers.
template <bool WAIT, bool BA> __device__ __forceinline__ void mfma32_v0(float16v& d, const half8& a, const half8& b) {
    if constexpr (WAIT && BA) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
    else if constexpr (WAIT) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
    else if constexpr (BA) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
    else asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
template <bool WAIT, bool BA> __device__ __forceinline__ void mfma32_v(float16v& d, const half8& a, const half8& b) {
    if constexpr (WAIT && BA) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
    else if constexpr (WAIT) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
    else if constexpr (BA) asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
    else asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
// The lane's number, read again where it is needed: across the main loop it would hold a register.
__device__ __forceinline__ int lane_again() {
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(lane));
    return lane;
}
// lane <-> lane ^ 32 combinations
__device__ __forceinline__ float xor32_max(float x) {
    const uint32_t xi = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32_sum(float x) {
    const uint32_t xi = __float_as_uint(x);
    auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ---- tile loads: global -> registers, one step ahead --------------------------------------------
// A lane's share of a tile record: its 16 bytes of every key block (the A operands of the block's two K=16 slices), the
// key scales of one token, its value codes.  Every load is one contiguous run across the wave (the record is stored in
// exactly this order).  A piece is requested again, for the tile a step later, as soon as it has been used, so that one
// set of registers is enough and every load has a whole step to arrive.  (Records staged in LDS with direct loads,
// three tiles ahead, cost 5 % more time on the Llama-shaped pool: the loop does not wait for its loads.)
//
// The records of a KV head are read through a buffer resource: every load is "resource + wave-uniform byte
// offset of the tile (a scalar register) + the lane's constant offset (a vector register that never changes)
// + an immediate", so a step spends no vector instruction on addresses, and a load beyond the KV head's records
// would return zeros instead of touching memory.
typedef __amdgpu_buffer_rsrc_t TileRsrc;
__device__ __forceinline__ TileRsrc make_tile_rsrc(const uint8_t* unit_base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(unit_base), 0, bytes, 0x00020000);
}
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F&& f) {   // f(integral_constant<int, 0 .. N-1>)
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// How the scores over q8_0 block keys are formed.
//   FOLD (exact keys): the keys enter the matrix cores as their codes, every 32-element block has a product
//     of its own, and the block scale (times softmax scale * log2 e) is applied to the block's products in fp32 as
//     they are summed.  A score tile has its tokens in the accumulator's registers, the same 16 tokens for every
//     lane of a half wave, so a scale is handed out by DPP: position i of each 16-lane row holds the scale of the
//     token of register i, and one v_fmac with a row broadcast of lane i does the element.
//   otherwise (one scale per layer tensor, whose scale rides on the softmax scale; keys rounded to fp16): one product
//     over all blocks.
__host__ __device__ constexpr bool fold_scales(int KC, bool K16) { return KC == 0 && !K16; }
// The records of a KV head as a lane reads them; `tile` is a record's byte offset.
template <int D, int VC, int KC, bool K16> struct TileReader {
    using LY = Layout<D, VC, KC>;
    static constexpr int VB = vc_bits(VC);
    static constexpr int NS = D / 64;             // dwords of key scales per token
    static constexpr int NQ = D / 64;             // chunks of value codes: four coordinate groups each
    static constexpr int CW = VB == 8 ? 8 : VB;   // dwords per lane and chunk
    TileRsrc rs;
    // the lane's offsets: key codes, key scales, value codes, value scales (opaque, so that the compiler adds what is
    // constant in the instruction instead of keeping a register per load)
    uint32_t k, s, v, g;

    __device__ __forceinline__ TileReader(TileRsrc r, int lane) : rs(r) {
        k = (uint32_t)lane * 16;
        // FOLD: the scales of the token of accumulator register lane % 16 in the lane's half wave; else of the token
        // whose key codes the lane holds
        const int t = fold_scales(KC, K16) ? 8 * ((lane >> 2) & 3) + 4 * (lane >> 5) + (lane & 3) : lane & 31;
        s = (uint32_t)t * (D / 32) * 2;
        v = (uint32_t)lane * (VB == 8 ? 16 : VB == 3 ? 12 : VB == 4 ? D / 4 : D / 8);
        g = (uint32_t)(lane >> 5) * 8;
        asm volatile("" : "+v"(k), "+v"(v));
        if (KC == 0) asm volatile("" : "+v"(s));
        if (vc_has_scale(VC)) asm volatile("" : "+v"(g));
    }
    // key codes of token lane % 32, block j: elements 8h..8h+7 (x, y) and 16+8h.. (z, w), h = lane / 32
    __device__ __forceinline__ uint4v kcodes(uint32_t tile, int j) const {
        return __builtin_amdgcn_raw_buffer_load_b128(rs, k + j * 1024, tile, 0);
    }
    // key scales, blocks 2x and 2x + 1
    __device__ __forceinline__ void kscales(uint32_t tile, uint32_t (&sc)[NS]) const {
        if (KC != 0) return;
        if constexpr (NS == 1) {
            sc[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, LY::kscales_off + s, tile, 0);
        } else {
#pragma unroll
            for (int x = 0; x < NS; x += 2) {
                const auto two = __builtin_amdgcn_raw_buffer_load_b64(rs, LY::kscales_off + s + 4 * x, tile, 0);
                sc[x] = two[0], sc[x + 1] = two[1];
            }
        }
    }
    // value codes of coordinate groups 4q .. 4q + 3
    __device__ __forceinline__ void vcodes(uint32_t tile, int q, uint32_t (&w)[CW]) const {
        if constexpr (VB == 8) {
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const uint4v c = __builtin_amdgcn_raw_buffer_load_b128(rs, LY::vcodes_off + v + (2 * q + x) * 1024, tile, 0);
                w[4 * x] = c.x, w[4 * x + 1] = c.y, w[4 * x + 2] = c.z, w[4 * x + 3] = c.w;
            }
        } else if constexpr (VB == 3) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b96(rs, LY::vcodes_off + v + q * 768, tile, 0);
            w[0] = t[0], w[1] = t[1], w[2] = t[2];
        } else if constexpr (VB == 4) {
            const uint4v c = __builtin_amdgcn_raw_buffer_load_b128(rs, LY::vcodes_off + v + 16 * q, tile, 0);
            w[0] = c.x, w[1] = c.y, w[2] = c.z, w[3] = c.w;
        } else {
            const auto c = __builtin_amdgcn_raw_buffer_load_b64(rs, LY::vcodes_off + v + 8 * q, tile, 0);
            w[0] = c[0], w[1] = c[1];
        }
    }
    // value scales of the lane's 16 tokens as fp16 pairs, in the order in which the lane holds their probabilities
    // (tokens 8b + 4h + {0,1} in [2b], + {2,3} in [2b+1])
    __device__ __forceinline__ void vscales(uint32_t tile, uint32_t (&sc)[8]) const {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const auto two = __builtin_amdgcn_raw_buffer_load_b64(rs, LY::vscales_off + g + 16 * b, tile, 0);
            sc[2 * b] = two[0], sc[2 * b + 1] = two[1];
        }
    }
};

__device__ __forceinline__ _Float16 half_of(uint32_t w, int odd) {   // the lower or upper fp16 of a dword
    return __builtin_bit_cast(_Float16, (uint16_t)(odd ? w >> 16 : w));
}

// Half block s of a lane's 16 key codes -> the A operand of one score product: the codes as exact fp16 integers or, for
// keys rounded to fp16 (K16), code * scale; sc2: the dword that holds the block's scale, odd: in its upper half.
template <bool K16> __device__ __forceinline__ half8 key_operand(const uint4v& raw, int s, uint32_t sc2, int odd) {
    H8 a;
    codes4_to_half(s == 0 ? raw.x : raw.z, a.u[0], a.u[1]);
    codes4_to_half(s == 0 ? raw.y : raw.w, a.u[2], a.u[3]);
    a.h = a.h - (_Float16)1152.0f;
    if (!K16) return a.h;
    return a.h * (half8)half_of(sc2, odd);
}

// S[i] += scale of register i's token * P[i] (see fold_scales).  (A statement per element: with several in one the register
// allocator copies the tile, a matrix instruction's result, out of its 16 consecutive registers.)
template <int I> __device__ __forceinline__ float fold1(float s, float product, float scale) {
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(s) : "v"(scale), "v"(product), "n"(I));
    return s;
}
__device__ __forceinline__ void fold16(float16v& S, const float16v& P, float scale) {
    static_for<16>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        S[i] = fold1<i>(S[i], P[i], scale);
    });
}

// Constants the main loop keeps in scalar registers.  As 32-bit literals they would double the size of every
// instruction that uses them, and a lone wave's instruction fetch is what bounds the loop.
struct LoopConsts {
    uint32_t m7, m3, m4;   // byte masks 0x07070707, 0x03030303, 0x04040404 (value-code selectors)
    half2v one2;           // (1, 1): the packed dot product that sums a pair of probabilities
    float raise_sum;       // AttendPlan::raise_sum
};
__device__ __forceinline__ LoopConsts make_loop_consts(float raise_sum) {
    uint32_t m7 = 0x07070707u, m3 = 0x03030303u, m4 = 0x04040404u, one = 0x3c003c00u;
    asm volatile("" : "+s"(m7), "+s"(m3), "+s"(m4), "+s"(one));   // opaque: the compiler would fold them back
    union {
        uint32_t u;
        half2v h;
    } o;
    o.u = one;
    return LoopConsts{m7, m3, m4, o.h, raise_sum};
}

// Half hf (codes 4 hf .. 4 hf + 3) of coordinate group gi = 0..3 of a chunk of value codes -> fp16 centroids: half of
// the A operand of one P.V product.
template <int VC, int CW>
__device__ __forceinline__ void value_half(const uint32_t (&w)[CW], int gi, int hf, H8& va, const LoopConsts& lc) {
    uint32_t &o0 = va.u[2 * hf], &o1 = va.u[2 * hf + 1];
    if constexpr (vc_bits(VC) == 4) {
        half4_b4(w[gi], hf, o0, o1);
    } else if constexpr (vc_bits(VC) == 2) {
        half4_b2(w[gi >> 1], gi & 1, hf, o0, o1);
    } else if constexpr (vc_bits(VC) == 8) {
        // int8 codes -> exact fp16 integers (the scale rides on P)
        codes4_to_half(w[4 * (gi >> 1) + 2 * (gi & 1) + hf], o0, o1);
        va.p[2 * hf] = va.p[2 * hf] - (_Float16)1152.0f;
        va.p[2 * hf + 1] = va.p[2 * hf + 1] - (_Float16)1152.0f;
    } else {
        lookup4(vcode_selector(w[0], w[1], w[2], gi, hf, lc.m7, lc.m3, lc.m4), o0, o1);
    }
}

template <typename SV> __device__ __forceinline__ float max16(const SV& a) {
    float m = fmaxf(fmaxf(a[0], a[1]), a[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) m = fmaxf(fmaxf(m, a[i]), a[i + 1]);
    return fmaxf(m, a[15]);
}

// Four scores of a row -> fp16 probabilities (packed pairs) and their sum into lsum (the tile's sum).  FOLD: S holds
// the exponents themselves (base-2 units, relative to the row's reference), else raw scores.  With value scales (g, the
// lane's StepState::g) the P.V operand is p * scale of its token (formed in fp32, rounded to fp16 once), at most
// 2^8 * 2^7; the denominator sums the plain, unrounded p.
template <bool VS, bool FOLD, typename SV>
__device__ __forceinline__ void exp4(const SV& S, int c, float qscale, float mneg, H8 (&pb)[2], float& lsum,
                                     const uint32_t* g, half2v one2, float* gmax = nullptr) {
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const int i = 4 * c + 2 * pr;
        half2v p2;
        const float e0 = __builtin_amdgcn_exp2f(FOLD ? S[i] : fmaf(S[i], qscale, mneg));
        const float e1 = __builtin_amdgcn_exp2f(FOLD ? S[i + 1] : fmaf(S[i + 1], qscale, mneg));
        p2[0] = (_Float16)e0;
        p2[1] = (_Float16)e1;
        // The denominator sums the very numbers that enter the P.V product where those are the probabilities
        // themselves (their rounding errors then cancel in the quotient); with a value scale the products p * g
        // are what is rounded, so the denominator takes the unrounded probabilities.
        if (VS) lsum += e0 + e1;
        else lsum = __builtin_amdgcn_fdot2(p2, one2, lsum, false);
        if (VS) {   // p * g in fp32, rounded to fp16 once
            union {
                uint32_t u;
                _Float16 h[2];
            } g2;
            g2.u = g[i >> 1];
            const float g0 = (float)g2.h[0], g1 = (float)g2.h[1];
            p2[0] = (_Float16)(e0 * g0);
            p2[1] = (_Float16)(e1 * g1);
            if (gmax != nullptr) *gmax = fmaxf(fmaxf(*gmax, g0), g1);   // the largest scale among the lane's tokens
        }
        pb[i >> 3].p[(i & 7) >> 1] = p2;
    }
}

// One software-pipelined step.  While the matrix cores compute the scores of tile B (the next tile),
// the vector ALUs turn the scores of tile A (the current tile, computed one step earlier) into
// probabilities and dequantize A's values; then the matrix cores accumulate A's P.V.  Keeping two
// tiles in flight is what lets MFMA and VALU work overlap within a single wave: the MFMA stream of a
// step never depends on vector work of the same tile that has not had a full step to complete.
//
//   cur        what a step is handed by the one before: the scores of tile A and its values, tile B's first key operands,
//              its key codes and scales; on exit the same for the next step, requested from nextV (tile B), nextK (the
//              tile after B) and, for block 0, whose operands are formed at the end of the step before, nextK0
//   upper      the lane is one of 32 .. 63
//   masked     (LAST only: tile B may be the pool's last) tokens of tile B from `masked` on lie past the end of the pool
//   down       (REBASE only) rows whose maximum of tile A lies less than `down` below their reference take it for their reference
//
// Softmax bookkeeping: the reference m_ref (base-2 units) of a row only moves when the row's probabilities
// of a tile, taken against the old reference, sum to more than raise_sum = 2^15 in one of the row's two lanes --
// with value scales: when that sum times the largest scale among the lane's tokens of the tile does.  Every operand
// that reaches a P.V product (a probability, or a probability times its token's scale) is therefore at most 2^15:
// fp16 holds it; what matters for the result is the relative precision of a probability, which does not depend on
// its magnitude, down to fp16's smallest normal number: a probability less than 2^-14 of the row's reference (divided
// by its token's value scale) loses bits, one less than 2^-25 is flushed to zero.  The common case takes no
// maximum over the scores, and on keys with outlier channels, where a row's maximum keeps creeping up, the expensive
// rescale of the accumulators stays rare: with a threshold of 2^8 it was a tenth of the kernel's time on the
// Llama-shaped workload.
//
// Which tokens set a reference shows in the result.  A probability is rounded to fp16, except where it is a power of two:
// the token that set the row's reference is exact, and the tokens with the largest probabilities make most of a row's
// error.  Every split and every wave that shares a row brings a reference of its own.  A plan with fewer of them than the one
// that gives every CU a workgroup makes up for it:
//   - besides its first tile's, a wave takes the maxima of its last AttendPlan::references - 1 tiles for references, one after
//     the other, which costs a rescale of the accumulators each, about a step (the first ones would do as well, but take
//     steps of their own in front of the loop: 0.5 us of 25 in the SmolLM2-shaped call, which has no use for them);
//   - rows move their reference at sums of 2^11 (keys with outlier channels, where each of several waves would have moved
//     its own).
// And whoever has the pool's last tile takes references from it where it is not full, as its few tokens may hold a maximum.
// Error against float64, rms over outputs, 32 layers x 8 KV heads x 128, with shared rows / own rows and one reference /
// own rows as described: 512 rows over 300 tokens 1.32 / 1.51 / 1.32e-4; 1,024 rows over 7,194 tokens 1.51 / 1.53 / 1.48e-4.
//
// A reference moves down by kRebaseDown at most: a token further below the largest so far hardly shows in the result,
// and the accumulators stay in range (16 references, 2^64).
constexpr int kRebaseDown = 4, kNoRebase = -1;

template <int D, int NT, int VC, int KC, bool K16> struct StepState {
    using TR = TileReader<D, VC, KC, K16>;
    float16v S[NT];                                // scores of tile A
    half8 kop[2];                                  // tile B: key operands of block 0, both halves,
    uint4v k[D / 32];                              //   key codes (block 0: of the tile after B),
    uint32_t sc[TR::NS];                           //   key scales
    uint32_t v[TR::NQ][TR::CW];                    // tile A: value codes
    uint32_t g[vc_has_scale(VC) ? 8 : 1];          //   and value scales
    __device__ __forceinline__ void first_operands() {
        kop[0] = key_operand<K16>(k[0], 0, sc[0], 0);
        kop[1] = key_operand<K16>(k[0], 1, sc[0], 0);
    }
};

// Waves per SIMD the kernel is compiled for: one where it needs all 512 registers; three for 32-row blocks at
// head_dim 64 (the small-row shape of the SmolLM2-sized pool: 768 workgroups, all resident at once on 256 CUs,
// so that one workgroup's query fetch, pipeline ramp and merge overlap the others' main loops); two for 64-row blocks there
// (24 layers x 32 heads x 1,851 tokens: 40 rows 54.0 us with one, 43.0 with two, 100 rows 97.6 and 74.7).  Value scales take 268
// to 308 of the 256 registers that leaves.  4-bit values and waves with rows of their own come out at 256 or less by themselves,
// compiled for one; two workgroups then share a CU as well (256 rows, rows of their own: 168 -> 141 us).
constexpr int kernel_waves_per_simd(int D, int NT, int VC, bool OWN) {
    if (D != 64 || vc_has_scale(VC) || OWN) return 1;
    return NT == 2 ? (vc_bits(VC) == 4 ? 1 : 2) : vc_bits(VC) == 3 ? 3 : 1;
}
// Where several waves share a SIMD, queries and accumulators are in vector registers like everything else: with any
// accumulation registers in use the compiler has half of a wave's registers for either kind, and at three waves moved 80 values
// a step between them.
constexpr bool parks(int waves_per_simd) { return waves_per_simd == 1; }

template <int D, int NT, int VC, int KC, bool K16, int WPS, bool HAS_A, bool HAS_B, bool LOOP, bool LAST, bool REBASE>
__device__ __forceinline__ void pipeline_step(StepState<D, NT, VC, KC, K16>& cur, const TileReader<D, VC, KC, K16>& tr,
                                              uint32_t nextV, uint32_t nextK, uint32_t nextK0, int masked, int down, float qscale,
                                              bool upper, const half8 (&qb)[NT][D / 32][2], float16v (&O)[D / 32][NT],
                                              float (&Lsum)[NT], float* m_ref, float (&mneg)[NT], const LoopConsts& lc) {
    using TR = TileReader<D, VC, KC, K16>;
    constexpr int NB = D / 32, NG = D / 16, MG = D / 32;
    constexpr bool FOLD = fold_scales(KC, K16), VS = vc_has_scale(VC), PARK = parks(WPS);
    const half8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    auto& Sa = cur.S;
    float16v Sb[NT];
    float lt[NT];   // this tile's probability sums, per lane
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) lt[nt] = 0.0f;

    // The step is a sequence of short stretches, each one product (MFMA) followed by the vector work that shares its
    // time; scheduling barriers keep the compiler from moving work across.
    constexpr int NCH = 4 * NT;   // probability chunks of tile A: 4 scores each
    auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
    H8 pb[NT][2];      // probabilities of tile A: B operands of the P.V products, [row tile][k slice]
    float gmax = VS ? 5.9604645e-8f : 1.0f;   // (not 0: an infinite sum times it must still say "move")
    auto exp_chunk = [&](int c) {
        exp4<VS, FOLD>(Sa[c >> 2], c & 3, qscale, mneg[c >> 2], pb[c >> 2], lt[c >> 2], cur.g, lc.one2,
                       VS && c < 4 ? &gmax : nullptr);
    };
    uint32_t sc_next[TR::NS], g_next[VS ? 8 : 1];   // scales of the tiles a step later
    auto kdeq = [&](int k, half8& dst) {   // half block k's operand; after a block's second half its codes are reloaded
        dst = key_operand<K16>(cur.k[k >> 1], k & 1, cur.sc[k >> 2], (k >> 1) & 1);
    };
    auto scales_next = [&]() {
        tr.kscales(nextK, sc_next);
        if constexpr (VS) tr.vscales(nextV, g_next);
    };

    // the row's maximum of tile A in base-2 units (FOLD: the exponents are relative to the reference)
    auto row_max = [&](int nt, float m_old) {
        return FOLD ? m_old + xor32_max(max16(Sa[nt])) : xor32_max(max16(Sa[nt])) * qscale;
    };
    auto move_reference = [&](int nt, float m_old, float m_new, bool both) {
        const float alpha = m_new == m_old ? 1.0f : __builtin_amdgcn_exp2f(m_old - m_new);
        m_ref[32 * nt + (lane_again() & 31)] = m_new;
        mneg[nt] = -m_new;
        if constexpr (FOLD) {   // the exponents of the tiles in flight move along
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                Sa[nt][i] -= m_new - m_old;
                if (both) Sb[nt][i] -= m_new - m_old;
            }
        }
        // The accumulators live in accumulation registers that vector instructions cannot read; an MFMA with zero
        // operands (D = 0*0 + C) carries them to vector registers and back, so the hot path never copies them.
        Lsum[nt] *= alpha;
        if constexpr (!PARK) {
            asm volatile("s_nop 15" : "+v"(O[0][nt]));   // the last products
            fence();
        }
#pragma unroll
        for (int g = 0; g < MG; ++g) {
            if constexpr (!PARK) {
                O[g][nt] *= alpha;
                continue;
            }
            float16v y = mfma32(zero8, zero8, O[g][nt]);
            y *= alpha;
            O[g][nt] = mfma32(zero8, zero8, y);
        }
    };
    // A tile that sets references does so before anything is taken relative to them, so that nothing is done twice (1,024 rows
    // over 7,194 tokens 1,094 instead of 1,158 us, 512 over 300 tokens 57 instead of 59).  Without FOLD and with a tile B the
    // registers do not hold it here, and it is done with the rows that outgrew their references, further down.
    constexpr bool EARLY = REBASE && (FOLD || !HAS_B);
    if constexpr (EARLY) {
        if (__builtin_expect(down != kNoRebase, 0)) {   // (out of the way of the steps without)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float m_old = m_ref[32 * nt + (lane_again() & 31)], m = row_max(nt, m_old), m_new = m >= m_old - (float)down ? m : m_old;
                if (__any(m_new != m_old)) move_reference(nt, m_old, m_new, false);
            }
        }
    }

    // block j's products with row tile nt (FOLD): two of them take turns, one is folded while the other is formed
    // (with two waves a SIMD one: a unit is folded before the next is formed)
    constexpr int NP = FOLD && WPS != 2 ? 2 : 1;
    float16v P[NP];
    constexpr int NU = NB * NT;
    // (A DPP source must not have been written by the two instructions before: a block's scale is formed a unit ahead.)
    float fscale[2];
    auto fold_scale = [&](int j) { fscale[j & 1] = (float)half_of(cur.sc[j >> 1], j & 1) * qscale; };
    auto fold = [&](int u) { fold16(Sb[u % NT], P[u % NP], fscale[u / NT & 1]); };
    if (HAS_B) {
        if constexpr (FOLD) {
            // Unit u: block u / NT with row tile u % NT, two products.  The operand of a half block is formed as soon as
            // its predecessor's last product has been issued.
            static_for<NU>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                constexpr int j = u / NT, nt = u % NT;
                const bool last_nt = nt == NT - 1 && j + 1 < NB;
                // The unit's chunks of probabilities, in order, so that a tile's sum is the same where it is formed anew (the rows
                // that move their reference).  The first units have one each in front; NP == 1: the others behind the second
                // product, which is folded after them.
                constexpr bool behind = NP == 1 && u + 1 < NU;
                auto chunks_before = [](int x) {
                    const int first = x < NT ? x : NT, even = x * NCH / NU;
                    return NP == 2 ? (even > first ? even : first) : x < NU ? first + x * (NCH - NT) / (NU - 1) : NCH;
                };
                constexpr int c0 = chunks_before(u), c1 = chunks_before(u + 1);
                fence();
                // What the block products are added to.  (In front: 15 agents 53.6 us; behind the first product 54.5.  As a product
                // of the references with constants, one fp32 matrix instruction for 16 moves, 1,024 rows 1,108 instead of 1,097.)
                if (j == 0) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) Sb[nt][i] = mneg[nt];
                    fence();
                    if (HAS_A) exp_chunk(c0);
                    fence();
                }
                if (u == 0) mfma32_v0<true, PARK>(P[u % NP], cur.kop[0], qb[nt][j][0]);   // (operands handed over by the last step)
                else mfma32_v0<!LOOP, PARK>(P[u % NP], cur.kop[0], qb[nt][j][0]);
                fence();
                if (u == 0) scales_next();
                if (nt == 0) fold_scale(j);
                if (last_nt) kdeq(2 * (j + 1), cur.kop[0]);
                auto chunks = [&]() {
                    if (HAS_A) {
#pragma unroll
                        for (int c = c0 + (j == 0 ? 1 : 0); c < c1; ++c) exp_chunk(c);
                    }
                };
                if (!behind) chunks();
                fence();
                if (u == 0) mfma32_v<true, PARK>(P[u % NP], cur.kop[1], qb[nt][j][1]);
                else mfma32_v<!LOOP, PARK>(P[u % NP], cur.kop[1], qb[nt][j][1]);
                fence();
                if (behind) chunks();
                if (NP == 2 ? u > 0 : behind) {
                    if (!HAS_A) {   // (no probabilities in between)
                        if (NP == 2) asm volatile("s_nop 7");
                        else asm volatile("s_nop 15");
                    }
                    fence();
                    fold(NP == 2 ? u - 1 : u);
                }
                if (last_nt) {
                    kdeq(2 * (j + 1) + 1, cur.kop[1]);
                    cur.k[j + 1 < NB ? j + 1 : 0] = tr.kcodes(nextK, j + 1);
                }
                fence();
            });
            if (!HAS_A) {   // (else with the first product of P.V)
                asm volatile("s_nop 15");
                fence();
                fold(NU - 1);
            }
        } else {
            constexpr int NQK = 2 * NB;   // half blocks
            half8 kop2[2] = {cur.kop[0], cur.kop[1]};
            static_for<NQK>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    fence();
                    if (k == 0) mfma32_v0<true, PARK>(Sb[nt], kop2[0], qb[nt][0][0]);
                    else if (k == 1) mfma32_v<true, PARK>(Sb[nt], kop2[1], qb[nt][0][1]);
                    else mfma32_v<!LOOP || NT == 1, PARK>(Sb[nt], kop2[k & 1], qb[nt][k >> 1][k & 1]);
                    fence();
                    if (k == 0 && nt == 0) scales_next();
                    // the operand two half blocks on, once this one's last product has been issued
                    if (nt == NT - 1 && k + 2 < NQK) {
                        kdeq(k + 2, kop2[k & 1]);
                        if (k & 1) cur.k[(k + 2 < NQK ? k + 2 : 0) >> 1] = tr.kcodes(nextK, (k + 2) >> 1);
                    }
                    if (HAS_A) {
                        const int u = k * NT + nt, N = NQK * NT;
#pragma unroll
                        for (int c = u * NCH / N; c < (u + 1) * NCH / N; ++c) exp_chunk(c);
                    }
                    fence();
                }
            });
            if (!HAS_A) asm volatile("s_nop 15");
        }
    } else if (HAS_A) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) exp_chunk(c);
    }
    if (HAS_A) {
        // Does a row have to move its reference?  Rare after a row's first tiles.  The probabilities of the rows that
        // move are then recomputed against the new reference; those of the other rows come out as they were.  Only the
        // rows that outgrew their reference move it: a row's result depends on that row's scores alone, whatever other
        // agents' rows share the wave.
        // gmax: the largest value scale among the lane's 16 tokens of this tile (1 without value scales), collected
        // by the chunks of row tile 0; the products probability x scale stay below raise_sum if the tile's sum of
        // probabilities times gmax does
        bool raise = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) raise |= !(lt[nt] * gmax <= lc.raise_sum);   // (inf and NaN say yes)
        const bool set_here = REBASE && !EARLY && down != kNoRebase;
        if (__builtin_expect(__any(raise) || set_here, 0)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const bool row_raise = !(xor32_max(lt[nt] * gmax) <= lc.raise_sum);   // (+inf stays +inf through the max)
                const float m_old = m_ref[32 * nt + (lane_again() & 31)];
                const float m = row_max(nt, m_old), m_new = row_raise ? fmaxf(m_old, m) : set_here && m >= m_old - (float)down ? m : m_old;
                if (!__any(m_new != m_old)) continue;   // no row of this row tile moves: it keeps what it has
                move_reference(nt, m_old, m_new, HAS_B);
                lt[nt] = 0.0f;
#pragma unroll
                for (int c = 4 * nt; c < 4 * nt + 4; ++c) exp_chunk(c);
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) Lsum[nt] += lt[nt];

        // ---- P.V.  Group G's operand is formed a little ahead of its first product; NVA operands take turns.
        // (Three where the registers hold them: 15 agents with tails over 7,194 tokens 117.2 us with two, 113.2 with three.)
        constexpr int NVA = FOLD && D == 128 && !VS ? 3 : 2;
        H8 va[NVA];
        auto vhalf = [&](int i) {   // the i-th half operand
            if (i >= 2 * NG) return;
            const int G = i >> 1;
            value_half<VC>(cur.v[G >> 2], G & 3, i & 1, va[G % NVA], lc);
            if (HAS_B && (i & 7) == 7) tr.vcodes(nextV, G >> 2, cur.v[G >> 2]);   // the chunk has been used up
        };
        vhalf(0);
        vhalf(1);
        if (NVA == 3) vhalf(2);
        fence();
#pragma unroll
        for (int G = 0; G < NG; ++G) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                if constexpr (PARK) O[G >> 1][nt] = mfma32(va[G % NVA].h, pb[nt][G & 1].h, O[G >> 1][nt]);
                else mfma32_v<true, false>(O[G >> 1][nt], va[G % NVA].h, pb[nt][G & 1].h);
                fence();
                if (FOLD && HAS_B && G == 0 && nt == 0) fold(NU - 1);
                vhalf(2 * G + NVA + nt);
                if (NT == 1) vhalf(2 * G + NVA + 1);
                fence();
            }
        }
    }

    if (HAS_B) {
        // what the next step starts with
#pragma unroll
        for (int x = 0; x < TR::NS; ++x) cur.sc[x] = sc_next[x];
        if constexpr (VS) {
#pragma unroll
            for (int x = 0; x < 8; ++x) cur.g[x] = g_next[x];
        }
        cur.first_operands();
        cur.k[0] = tr.kcodes(nextK0, 0);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if (LAST && masked < kTile) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (8 * (i >> 2) + (upper ? 4 : 0) + (i & 3) >= masked) Sb[nt][i] = -INFINITY;
            }
            Sa[nt] = Sb[nt];
        }
    }
}

// ws_ml / ws_o: where the kernel leaves its split's partial (direct == 0); with direct == 1 and private tails,
// the tail kernel's partials (row maxima and denominators / unnormalized sums), read in the final pass.
// block: the workgroup's number among those that read the pool.
// OWN: every wave has 32 NT query rows of its own and walks the whole token range of the split, instead of four waves
// sharing the rows and taking every fourth tile: nothing to merge between the waves, a fourth of the workgroups, whose
// ramps and final passes (five steps' worth, see make_plan) are then spread over four times the steps, and one record
// serves the four waves from the L1.  Measured, shared rows and own rows, 32 layers x 8 KV heads x 128:
//   1,024 rows, 7,194 tokens   1,158 and 1,100 us       256 rows, 4,096 tokens   171 and 163 us
//   512 rows, 300 tokens          75 and 56 us          (head_dim 256, 128 rows, 2,500 tokens   133 and 118 us)
// (own rows with as many references as the shared ones have, see kRebaseDown)
template <int D, int NT, int VC, int KC, bool K16, bool OWN>
__device__ __forceinline__ void attend_mfma_block(const uint8_t* __restrict__ pool, const __half* __restrict__ Q,
                                                  float* __restrict__ ws_ml, float* __restrict__ ws_o,
                                                  float* __restrict__ out, const AttendPlan& p, int direct, uint32_t block) {
    using LY = Layout<D, VC, KC>;
    constexpr int NB = D / 32, MG = D / 32, ROWS = 32 * NT;
    constexpr int WG_ROWS = OWN ? 4 * ROWS : ROWS, STEP = OWN ? 1 : 4;   // rows of the workgroup; tiles from one of a wave's to its next
    constexpr int WPS = kernel_waves_per_simd(D, NT, VC, OWN);
    constexpr bool FOLD = fold_scales(KC, K16), PARK = parks(WPS);
    constexpr int OSTRIDE = D + 4;
    constexpr int TB = LY::tile_bytes;
    __shared__ float m_s[4][ROWS];
    __shared__ float l_s[4 * ROWS];
    extern __shared__ __align__(16) float o_s[];  // four merge buffers of ROWS x OSTRIDE floats

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
    const int h = lane >> 5, n = lane & 31;
    // Workgroup -> (token stream = split of a KV head, row block).  Consecutive workgroups go to the eight dies in turn,
    // each with an L2 of its own: the row blocks of a stream follow each other on one die, so that they read its records
    // from memory once.  (Row blocks in the outermost grid dimension read every record once per block from memory:
    // 1,450 us for 16 row blocks over 7,194 tokens, 1,165 us in this order.)
    int row_block, split, kvh;
    const int stream = p.div_row_blocks.divide((int)(block >> 3), &row_block) * 8 + (int)(block & 7);
    if (stream >= p.layers * p.H * p.nsplit) return;   // (the dies' rounding, or that of a grid of two dimensions)
    const int row0 = row_block * WG_ROWS + (OWN ? wave * ROWS : 0);
    const int usel = p.div_nsplit.divide(stream, &split), ls = p.div_H.divide(usel, &kvh);
    const int tps = p.split_tiles;
    const int t_begin = split * tps, t_end = min(p.tiles, t_begin + tps);
    const uint8_t* unit_base = pool + (size_t)((p.layer_begin + ls) * p.H + kvh) * p.tiles_cap * TB;
    // One key scale per layer tensor: the keys enter the products as their integer codes and the scale
    // rides on the softmax scale (an all-zero layer has only zero codes: any positive scale will do).
    float qscale = p.qscale;
    if (KC == 1) {
        const float s_tensor = (float)tensor_key_scale(p.kmax[p.layer_begin + ls]);
        qscale *= s_tensor > 0.0f ? s_tensor : 1.0f;
    }

    // this wave's tiles: t_begin + wave, +4, +8, ... (OWN: all); local index k <-> tile my_first + STEP k
    const int my_first = t_begin + (OWN ? 0 : wave);
    const int my_count = my_first < t_end && (!OWN || row0 < p.R) ? (t_end - my_first + STEP - 1) / STEP : 0;
    // Byte offset of local tile k; k past the end is clamped (the loads of the last steps then fetch the wave's own last
    // tile again, harmlessly, instead of needing a branch per load).
    // (From the KV head's first record; pool_create keeps a KV head's records under 4 GiB.)
    const int last_k = max(my_count - 1, 0);
    auto tile_off = [&](int k) { return (uint32_t)(my_first + STEP * min(k, last_k)) * (uint32_t)TB; };
    const TileReader<D, VC, KC, K16> tr(make_tile_rsrc(unit_base, (uint32_t)p.tiles_cap * (uint32_t)TB), lane);
    StepState<D, NT, VC, KC, K16> cur;
    if (my_count > 0) {
        const uint32_t t0 = tile_off(0);
#pragma unroll
        for (int j = 0; j < NB; ++j) cur.k[j] = tr.kcodes(t0, j);
        tr.kscales(t0, cur.sc);
    }

    // ---- query rows as MFMA B operands: lane (n, h) holds q[row 32nt+n][32j + 16s + 8h .. +7].
    // The block of rows is fetched with fully coalesced 16-byte loads (16 lanes to a row) into LDS
    // (the merge buffers are idle until the end) and picked up from there in operand order.
    constexpr int QS = D + 8;  // halves per staged row: 16-byte aligned, rotates the banks
    constexpr int QT = OWN ? 64 : 256;        // threads that fetch a block of rows
    const int qt = OWN ? lane : tid;
    _Float16* q_s = reinterpret_cast<_Float16*>(o_s + (OWN ? wave * ROWS * OSTRIDE : 0));   // (OWN: in the wave's own buffer)
    constexpr int QP = ROWS * (D / 8) / QT;   // 16-byte pieces per thread; all requested before any is used
    static_assert(QP * QT == ROWS * (D / 8), "");
    uint4v qraw[QP];
#pragma unroll
    for (int u = 0; u < QP; ++u) {
        // rows past the end re-read the last row (no branch between the loads) and are zeroed below
        const int i = qt + QT * u, rr = i / (D / 8), piece = i - rr * (D / 8), r = min(row0 + rr, p.R - 1);
        qraw[u] = *reinterpret_cast<const uint4v*>(Q + q_row_index(p, ls, kvh, r) * D + 8 * piece);
    }
    // the accumulators are cleared while the queries and the first tiles are on their way
    float16v O[MG][NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int g = 0; g < MG; ++g) {
#pragma unroll
            for (int i = 0; i < 16; ++i) O[g][nt][i] = 0.0f;
            if constexpr (PARK) asm volatile("" : "+a"(O[g][nt]));  // now, not where the first product needs them
        }
#pragma unroll
    for (int u = 0; u < QP; ++u) {
        const int i = qt + QT * u, rr = i / (D / 8), piece = i - rr * (D / 8);
        uint4v raw = row0 + rr < p.R ? qraw[u] : uint4v{0, 0, 0, 0};
        if (p.io_bf16) {  // bfloat16 queries become fp16 operands (exact for magnitudes fp16 holds)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float2 f = pair16_to_float2(raw[b], true);
                union {
                    uint32_t u;
                    _Float16 h[2];
                } o;
                o.h[0] = (_Float16)f.x;
                o.h[1] = (_Float16)f.y;
                raw[b] = o.u;
            }
        }
        *reinterpret_cast<uint4v*>(q_s + rr * QS + 8 * piece) = raw;
    }
    __syncthreads();
    half8 qb[NT][NB][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                qb[nt][j][s] = *reinterpret_cast<const half8*>(q_s + (32 * nt + n) * QS + 32 * j + 16 * s + 8 * h);
    __syncthreads();  // every wave has picked up its queries: the merge at the end reuses this memory
    // The queries are only ever MFMA operands: park them in accumulation registers so that the vector
    // registers are left for the scores and the dequantization temporaries (a second loop, so that the LDS
    // reads above are all in flight before the first one is waited for).
    if constexpr (PARK) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int s = 0; s < 2; ++s) asm volatile("" : "+a"(qb[nt][j][s]));
    }

    // The references themselves are only read where a row moves its reference and at the merge: they live in the
    // wave's row of m_s (LDS), not in registers.  Both lanes of a row hold the same value and write the same value;
    // a wave's LDS accesses complete in order, so a wave reading back what it wrote needs no barrier.
    float* const m_ref = m_s[wave];
    float Lsum[NT], mneg[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        m_ref[32 * nt + n] = -INFINITY;
        mneg[nt] = FOLD ? 0.0f : INFINITY;   // no reference yet: the first tile's maximum sets one
        Lsum[nt] = 0.0f;
    }
    const LoopConsts lc = make_loop_consts(p.raise_sum);

    // Local tile k is "B" in step k-1 (scores) and "A" in step k (softmax, PV).
    if (my_count > 0) {
        int k = 0;                                            // the step's tile A
        auto rest = [&](int b) { return p.T - (my_first + STEP * b) * kTile; };   // tokens from tile b's first one on
        cur.first_operands();
        cur.k[0] = tr.kcodes(tile_off(1), 0);
        // prologue: scores of tile 0; requests the values of tile 0 and the keys of tile 1
#pragma unroll
        for (int q = 0; q < TileReader<D, VC, KC, K16>::NQ; ++q) tr.vcodes(tile_off(0), q, cur.v[q]);
        pipeline_step<D, NT, VC, KC, K16, WPS, false, true, false, true, false>(cur, tr, tile_off(0), tile_off(1), tile_off(2), rest(0), kNoRebase,
                                                                   qscale, h == 1, qb, O, Lsum, m_ref, mneg, lc);
        // the rows' first references: the maxima of this first tile, taken here once instead of letting the first
        // step find out through infinite probabilities and compute its tile's probabilities twice
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const float m0 = xor32_max(max16(cur.S[nt])) * (FOLD ? 1.0f : qscale);
            m_ref[32 * nt + n] = m0;
            mneg[nt] = -m0;
            if constexpr (FOLD) {
#pragma unroll
                for (int i = 0; i < 16; ++i) cur.S[nt][i] -= m0;
            }
        }
        // The wave's last tiles set references besides the first, as many as the plan says, and one that is not full on top; by
        // itself the latter only raises them.
        const bool ragged = rest(my_count - 1) < kTile;
        const int setting = my_count - (p.references > 1 ? p.references - 1 + (ragged ? 1 : 0) : 0);   // from this tile on
        const int pairs_end = min(my_count - 3, setting - 1);
        auto main_step = [&]() {
            pipeline_step<D, NT, VC, KC, K16, WPS, true, true, true, false, false>(cur, tr, tile_off(k + 1), tile_off(k + 2), tile_off(k + 3),
                                                                              kTile, kNoRebase, qscale, h == 1, qb, O, Lsum, m_ref, mneg, lc);
            ++k;
        };
        while (k < pairs_end) {   // two steps a trip: the two tiles' scores swap registers without copies
            main_step();
            main_step();
        }
        for (; k + 1 < my_count; ++k)   // tile B may be the pool's last
            pipeline_step<D, NT, VC, KC, K16, WPS, true, true, true, true, true>(cur, tr, tile_off(k + 1), tile_off(k + 2), tile_off(k + 3),
                                                                            rest(k + 1), k > 0 && k >= setting ? kRebaseDown : kNoRebase,
                                                                            qscale, h == 1, qb, O, Lsum, m_ref, mneg, lc);
        const int down = k > 0 && k >= setting ? kRebaseDown : ragged ? 0 : kNoRebase;
        pipeline_step<D, NT, VC, KC, K16, WPS, true, false, false, false, true>(cur, tr, 0, 0, 0, kTile, down, qscale, h == 1, qb, O, Lsum,
                                                                           m_ref, mneg, lc);
    }

    // ---- merge the four waves through LDS: every wave stores its row maxima, denominators and accumulators
    // as they are into buffers of its own; the final pass rescales them to the common row maximum and adds
    // them in a fixed order, so the result is reproducible.
    const int elane = lane_again();
    {
        if constexpr (!PARK) {   // the last products
            asm volatile("s_nop 15" : "+v"(O[0][0]));
            __builtin_amdgcn_sched_barrier(0);
        }
        const int h = elane >> 5, n = elane & 31;
        float* obuf = o_s + wave * (ROWS * OSTRIDE);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int r = 32 * nt + n;
            const float l = xor32_sum(Lsum[nt]);  // the lane pair (n, h) shares a row
            if (h == 0) {
                l_s[wave * ROWS + r] = l;
            }
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    // registers 4b..4b+3 hold coordinates 32g + 8b + 4h + 0..3 of row r
                    float4* dst = reinterpret_cast<float4*>(&obuf[r * OSTRIDE + 32 * g + 8 * b + 4 * h]);
                    *dst = make_float4(O[g][nt][4 * b + 0], O[g][nt][4 * b + 1], O[g][nt][4 * b + 2], O[g][nt][4 * b + 3]);
                }
        }
    }
    if constexpr (OWN) {   // the wave's own buffer: its LDS accesses complete in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }

    // ---- final pass: every wave finishes ROWS/4 rows, LR lanes to a row.  Lane qd of a row takes every
    // LR-th 4-coordinate piece (piece LR i + qd), so that the lanes of a row read and write LR * 16 contiguous bytes per
    // instruction; the rotation is then log2(D/LR) in-register stages and log2(LR) DPP stages, whichever index bits
    // sit in the lane.  Four lanes for 16 rows; eight for the 8 rows of a 32-row workgroup's wave, of which each sixteen
    // lanes take two that lie 8 rows apart, in different halves of the LDS banks.  (With four lanes there, half of a wave idle:
    // 7,000 of 92,000 cycles of a wave at head_dim 256, 4,000 with eight; 26 layers x 8 heads x 2,500 tokens 46.1 -> 44.7 us,
    // 32 one-layer calls 435 -> 412, one layer of 600 tokens 7.5 -> 7.3, SmolLM2 shape with 5 rows 28.4 -> 27.8.)
    // (OWN: a wave finishes its own rows, 16 at a time, from its own buffer.)
    constexpr int LR = OWN || NT == 2 ? 4 : 8, CPL = D / LR;
    const int qd = LR == 8 ? codec_chunk(elane) : elane & 3;
    const int ri = LR == 8 ? ((elane >> 1) & 2) | ((elane >> 4) & 1) | ((elane >> 3) & 4) : elane >> 2;
    const float entry_sign = LR == 8 ? codec_entry_sign(elane) : quad_entry_sign(elane);
#pragma unroll 1
    for (int pass = 0; pass < (OWN ? ROWS / 16 : 1); ++pass) {
        const int rr = OWN ? 16 * pass + ri : wave + 4 * ri, r = row0 + rr;
        constexpr int NW = OWN ? 1 : 4;   // the waves that hold a share of the row
        const int w0 = OWN ? wave : 0;
        float Mr = m_s[w0][rr];
#pragma unroll
        for (int w = 1; w < NW; ++w) Mr = fmaxf(Mr, m_s[w][rr]);
        float fw[NW];  // a wave's weight: 2^(its maximum - the common one); 0 if it saw no tile
#pragma unroll
        for (int w = 0; w < NW; ++w)
            fw[w] = m_s[w0 + w][rr] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_s[w0 + w][rr] - Mr);
        float l;
        if constexpr (OWN) l = l_s[wave * ROWS + rr] * fw[0];
        else l = (l_s[rr] * fw[0] + l_s[ROWS + rr] * fw[1]) + (l_s[2 * ROWS + rr] * fw[2] + l_s[3 * ROWS + rr] * fw[3]);
        // Direct output with private tails: the row's tail partial (maximum in base-2 units, denominator and
        // unnormalized sum in the original value domain; written by the tail kernel, which ran before this one
        // and whose buffers arrive in ws_ml / ws_o) joins by log-sum-exp weights: the pool part gets wa / den
        // instead of 1 / l, the tail part wb / den once the pool part has been rotated back.
        float inv_l = __builtin_amdgcn_rcpf(l), tail_w = 0.0f;
        size_t tail_row = 0;
        if (direct && p.has_tails) {
            tail_row = (size_t)usel * p.R + min(r, p.R - 1);
            const float tm = ws_ml[tail_row * 2], tl = ws_ml[tail_row * 2 + 1];
            if (tl > 0.0f) {
                const float M2 = fmaxf(Mr, tm);
                const float wa = __builtin_amdgcn_exp2f(Mr - M2), wb = __builtin_amdgcn_exp2f(tm - M2);
                const float inv = 1.0f / (wa * l + wb * tl);
                inv_l = wa * inv;
                tail_w = wb * inv;
            }
        }
        // direct: 1/l, the centroid scale, 1/sqrt(D) and the entry sign of the DPP stages in one factor
        // int8 values are accumulated unrotated and unscaled: 1/l is all that is left to do
        constexpr float kCS = inv_centroid_scale<vc_bits(VC)>();
        const float f = VC == 2 ? (direct ? inv_l : 1.0f)
                        : direct ? entry_sign * (kCS * (D == 64 ? 0.125f : D == 128 ? 0.08838834764831845f : 0.0625f)) *
                                       inv_l
                                 : kCS;
#pragma unroll
        for (int w = 0; w < NW; ++w) fw[w] *= f;
        float x[CPL];  // x[4i + k] = coordinate 4 (LR i + qd) + k
        constexpr int BUF4 = ROWS * OSTRIDE / 4;  // one wave's buffer, in float4 units
        const float4* a4 = reinterpret_cast<const float4*>(&o_s[rr * OSTRIDE]) + w0 * BUF4 + qd;
#pragma unroll
        for (int i = 0; i < CPL / 4; ++i) {
            const float4 a = a4[LR * i];
            if constexpr (OWN) {
                x[4 * i + 0] = a.x * fw[0];
                x[4 * i + 1] = a.y * fw[0];
                x[4 * i + 2] = a.z * fw[0];
                x[4 * i + 3] = a.w * fw[0];
            } else {
                const float4 b = a4[BUF4 + LR * i], c = a4[2 * BUF4 + LR * i], d = a4[3 * BUF4 + LR * i];
                x[4 * i + 0] = (a.x * fw[0] + b.x * fw[1]) + (c.x * fw[2] + d.x * fw[3]);
                x[4 * i + 1] = (a.y * fw[0] + b.y * fw[1]) + (c.y * fw[2] + d.y * fw[3]);
                x[4 * i + 2] = (a.z * fw[0] + b.z * fw[1]) + (c.z * fw[2] + d.z * fw[3]);
                x[4 * i + 3] = (a.w * fw[0] + b.w * fw[1]) + (c.w * fw[2] + d.w * fw[3]);
            }
        }
        if (direct) {
            if (VC != 2) {
                if constexpr (LR == 8) wht_cross_chunks<CPL>(x, elane);
                else wht_cross_quad<CPL>(x, elane);
                wht_inlane<CPL>(x);
                // rotation variant H.D
                if (p.signs.on) {
#pragma unroll
                    for (int i = 0; i < CPL / 4; ++i) {
                        float(&x4)[4] = *reinterpret_cast<float(*)[4]>(&x[4 * i]);
                        const int at = LR == 8 ? 4 * qd : 16 * (i & 1) + 4 * qd;
                        flip_signs<4>(x4, sign_word(p.signs, LR == 8 ? i : i >> 1) >> at);
                    }
                }
            }
            if (tail_w != 0.0f) {
                const float4* t4 = reinterpret_cast<const float4*>(ws_o + tail_row * D) + qd;
#pragma unroll
                for (int i = 0; i < CPL / 4; ++i) {
                    const float4 t = t4[LR * i];
                    x[4 * i] = fmaf(tail_w, t.x, x[4 * i]);
                    x[4 * i + 1] = fmaf(tail_w, t.y, x[4 * i + 1]);
                    x[4 * i + 2] = fmaf(tail_w, t.z, x[4 * i + 2]);
                    x[4 * i + 3] = fmaf(tail_w, t.w, x[4 * i + 3]);
                }
            }
            if (r < p.R) {
                float4* dst = reinterpret_cast<float4*>(out + q_row_index(p, ls, kvh, r) * D) + qd;
#pragma unroll
                for (int i = 0; i < CPL / 4; ++i) dst[LR * i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
            }
        } else if (r < p.R) {
            const size_t prow = ((size_t)usel * p.nsplit + split) * p.R + r;
            float4* dst = reinterpret_cast<float4*>(ws_o + prow * D) + qd;
#pragma unroll
            for (int i = 0; i < CPL / 4; ++i) dst[LR * i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
            if (qd == 0) {
                ws_ml[prow * 2] = Mr;
                ws_ml[prow * 2 + 1] = l;
            }
        }
    }
}

template <int D, int NT, int VC, int KC, bool K16, bool OWN>
__global__ __launch_bounds__(256, kernel_waves_per_simd(D, NT, VC, OWN)) void attend_mfma_kernel(
    const uint8_t* __restrict__ pool, const __half* __restrict__ Q, float* __restrict__ ws_ml, float* __restrict__ ws_o,
    float* __restrict__ out, AttendPlan p, int direct) {
    attend_mfma_block<D, NT, VC, KC, K16, OWN>(pool, Q, ws_ml, ws_o, out, p, direct, blockIdx.y * p.grid_x + blockIdx.x);
}

// Two workgroups a CU wherever the pool's part fits 256 registers (left alone, the tails' part takes 324 at head_dim 128).
constexpr int tails_waves_per_simd(int D, int VC, int KC) {
    return D == 128 && vc_has_scale(VC) && KC == 0 ? 1 : kernel_waves_per_simd(D, 1, VC, false) == 3 ? 3 : 2;
}
// The same for a call whose token range is split, with the private tails in the same launch: the workgroups from
// pool_blocks on do the tails, a wave each.  Neither part needs the other before the merge kernel, and two workgroups of
// 32 rows fit a CU, so the tails run beside the pool instead of in a launch of their own in front of it: 32 one-layer calls with 32-token
// tails, 15 agents, 573 us with two launches, 442 us with one.
template <int D, int VC, int KC, bool K16>
__global__ __launch_bounds__(256, tails_waves_per_simd(D, VC, KC)) void attend_mfma_tails_kernel(
    const uint8_t* __restrict__ pool, const __half* __restrict__ Q, float* __restrict__ ws_ml, float* __restrict__ ws_o,
    AttendPlan p, TailPtrs tails, float* __restrict__ tail_ml, float* __restrict__ tail_o, uint32_t pool_blocks) {
    const uint32_t block = blockIdx.y * p.grid_x + blockIdx.x;
    if (block < pool_blocks) {
        attend_mfma_block<D, 1, VC, KC, K16, false>(pool, Q, ws_ml, ws_o, nullptr, p, 0, block);
        return;
    }
    extern __shared__ __align__(16) float o_s[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int units = p.layers * p.H;
    const int job = (int)(block - pool_blocks) * 4 + wave;   // agents of a unit follow each other
    const int a = job % p.A, usel = job / p.A % units, zb = job / p.A / units;
    float* p_s = o_s + wave * tail_block_tokens(D) * kTailRows;
    // (a job past the last has no rows)
    if (p.io_bf16) tail_rows<D, true>(Q, tails, tail_ml, tail_o, p, a, usel, zb, threadIdx.x & 63, p_s);
    else tail_rows<D, false>(Q, tails, tail_ml, tail_o, p, a, usel, zb, threadIdx.x & 63, p_s);
}

// int8 values at head_dim 256 stay with the vector kernel: it keeps queries and probabilities in 32 bits, and takes bfloat16
// queries of any magnitude; the matrix kernel would have both in fp16 (its registers hold the pair, it is not a matter of fit).
bool matrix_kernel_supports(int head_dim, int value_codec) { return head_dim != 256 || value_codec != POLYKV_VALUES_INT8; }

// Query rows per workgroup: 64 (32 at head_dim 256, where 64 rows' accumulators alone would fill the registers).
int matrix_kernel_block_rows(int head_dim) { return head_dim == 256 ? 32 : 64; }

bool matrix_kernel_direct(const AttendPlan& plan) { return plan.nsplit == 1; }

int matrix_kernel_row_tiles(const AttendPlan& plan) { return plan.D != 256 && plan.R > 32 && plan.block_rows == 64 ? 2 : 1; }

int matrix_kernel_row_blocks(const AttendPlan& plan) {
    const int rows = 32 * matrix_kernel_row_tiles(plan) * (plan.own_rows ? 4 : 1);
    return (plan.R + rows - 1) / rows;
}

static long tail_waves(const AttendPlan& plan) {
    return (long)plan.A * plan.layers * plan.H * ((plan.nq * plan.G + kTailRows - 1) / kTailRows);
}

// Tails in the pool's launch: where the merge kernel runs anyway, with 32-row workgroups at head_dim 64 and 128 (of
// which two fit a CU; a call of 64-row workgroups fills the CUs with them, and the tails would follow), and no more of them than
// all CUs hold beside one pool workgroup each.
bool matrix_kernel_takes_tails(const AttendPlan& plan) {
    return plan.has_tails && plan.kernel == POLYKV_KERNEL_MATRIX && !matrix_kernel_direct(plan) && plan.D != 256 &&
           matrix_kernel_row_tiles(plan) == 1 && tail_waves(plan) <= 4 * 256;
}

static uint64_t pool_workgroups(const AttendPlan& plan) {
    const uint64_t streams = (uint64_t)plan.layers * plan.H * plan.nsplit;
    return (streams + 7) / 8 * 8 * plan.div_row_blocks.d;
}

// A grid dimension holds less than 2^32 threads, 16.7 million workgroups; beyond 2^23 of them (only splits asked for by number
// over pools near 100 GB come there) the launch gets a second dimension.  Whole multiples of eight keep the order of the dies.
dim3 matrix_kernel_grid(const AttendPlan& plan) {
    const uint64_t all = pool_workgroups(plan) + (matrix_kernel_takes_tails(plan) ? (tail_waves(plan) + 3) / 4 : 0), most = 1u << 23;
    return all <= most ? dim3((uint32_t)all) : dim3((uint32_t)most, (uint32_t)((all + most - 1) / most));
}

template <int D, int NT, int VC, int KC, bool K16, bool OWN>
static hipError_t launch_one(const uint8_t* storage, const AttendPlan& plan, const void* Q, float* ws_ml,
                             float* ws_o, float* out, int direct, const TailPart* tails, hipStream_t s) {
    constexpr int kShared = 4 * 32 * NT * (D + 4) * (int)sizeof(float);   // the merge buffers
    auto kern = attend_mfma_kernel<D, NT, VC, KC, K16, OWN>;
    static std::once_flag configured;  // per instantiation: the limit is a property of the function
    static hipError_t config_result = hipSuccess;
    if (kShared > 48 * 1024)
        std::call_once(configured, [&]() {
            config_result = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, kShared);
            if constexpr (NT == 1 && D != 256 && !OWN)
                if (config_result == hipSuccess)
                    config_result = hipFuncSetAttribute(reinterpret_cast<const void*>(attend_mfma_tails_kernel<D, VC, KC, K16>),
                                                        hipFuncAttributeMaxDynamicSharedMemorySize, kShared);
        });
    if (config_result != hipSuccess) return config_result;
    const dim3 grid = matrix_kernel_grid(plan);
    if (grid.y > 65535) return hipErrorInvalidConfiguration;
    if constexpr (NT == 1 && D != 256 && !OWN) {
        if (tails != nullptr) {
            launch_main_kernel(attend_mfma_tails_kernel<D, VC, KC, K16>, grid, dim3(256), kShared, s, storage, (const __half*)Q,
                               ws_ml, ws_o, plan, *tails->ptrs, tails->ml, tails->o, (uint32_t)pool_workgroups(plan));
            return hipGetLastError();
        }
    }
    launch_main_kernel(kern, grid, dim3(256), kShared, s, storage, (const __half*)Q, ws_ml, ws_o, out, plan, direct);
    return hipGetLastError();
}

// Row tiles per workgroup: two (64 rows) or one (32 rows), see matrix_kernel_block_rows().
template <int D, int VC, int KC, bool K16>
static hipError_t launch_dv(const polykv_pool* pool, const AttendPlan& plan, const void* Q, float* ws_ml, float* ws_o,
                            float* out, const TailPart* tails, hipStream_t s) {
    const uint8_t* storage = reinterpret_cast<const uint8_t*>(pool->storage);
    const int direct = matrix_kernel_direct(plan) ? 1 : 0;
    if constexpr (D != 256) {
        if (matrix_kernel_row_tiles(plan) == 2)
            return plan.own_rows ? launch_one<D, 2, VC, KC, K16, true>(storage, plan, Q, ws_ml, ws_o, out, direct, tails, s)
                                 : launch_one<D, 2, VC, KC, K16, false>(storage, plan, Q, ws_ml, ws_o, out, direct, tails, s);
    } else if (plan.own_rows) {
        return launch_one<D, 1, VC, KC, K16, true>(storage, plan, Q, ws_ml, ws_o, out, direct, tails, s);
    }
    return launch_one<D, 1, VC, KC, K16, false>(storage, plan, Q, ws_ml, ws_o, out, direct, tails, s);
}

template <int D, int KC, bool K16>
static hipError_t launch_dk(const polykv_pool* pool, const AttendPlan& plan, const void* Q, float* ws_ml, float* ws_o,
                            float* out, const TailPart* tails, hipStream_t s) {
    switch (plan.vcodec) {
        case 1: return launch_dv<D, 1, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        case 2:
            if constexpr (D == 256) return hipErrorInvalidValue;   // not built: matrix_kernel_supports() says no
            else return launch_dv<D, 2, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        case 3: return launch_dv<D, 3, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        case 4: return launch_dv<D, 4, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        case 5: return launch_dv<D, 5, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        case 6: return launch_dv<D, 6, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        default: return launch_dv<D, 0, KC, K16>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
    }
}

template <int D>
static hipError_t launch_d(const polykv_pool* pool, const AttendPlan& plan, const void* Q, float* ws_ml,
                           float* ws_o, float* out, const TailPart* tails, hipStream_t s) {
    if (plan.kcodec == POLYKV_KEYS_Q8_TENSOR) return launch_dk<D, 1, false>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
    // keys rounded to fp16 once dequantized (the precision of the dense cache the paper's read path holds): only
    // for the paper's value codec at head_dim 64 / 128, the shapes this option is meant for
    if (plan.key_fp16) {
        if constexpr (D != 256) {
            if (plan.vcodec == POLYKV_VALUES_TQ3) return launch_dv<D, 0, 0, true>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
        }
    }
    return launch_dk<D, 0, false>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
}

hipError_t launch_attend_matrix(const polykv_pool* pool, const AttendPlan& plan, const void* Q, float* ws_ml,
                                float* ws_o, float* out, const TailPart* tails, hipStream_t s) {
    if (plan.D == 128) return launch_d<128>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
    if (plan.D == 256) return launch_d<256>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
    return launch_d<64>(pool, plan, Q, ws_ml, ws_o, out, tails, s);
}

}  // namespace polykv
