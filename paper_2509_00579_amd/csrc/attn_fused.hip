// Fetch side (Section 3.3, Figure 1): one decode-attention step straight from the compressed cache.
//
// Per 2D block a single wavefront (64 lanes) stages the K record in LDS, every lane Huffman-decodes the two slices
// of one token with a lookup table -- each slice from both ends, four independent decode chains of 32 symbols per
// lane -- and accumulates q.k in registers; the wave then updates a running softmax and decodes the V record of the
// same block, every lane owning two channels (two slices, again four chains) and accumulating p.v in registers.  No
// decompressed value ever leaves the registers (Section 3.3.2): the decoded quantization codes are packed four to a
// register and handed to the matrix cores from there.
//
// What differs from the paper's kernel, and why (gfx950):
//  * lookup-table decode instead of the bit-serial tree walk of Section 3.3.1: all 64 lanes of a wave advance in
//    symbol lock-step (same trip count for every lane, no divergence), so the dequantization weight of the current
//    symbol is the same for the whole wave and the products with it fit the matrix cores: int8 codes times the signed
//    byte digits of integer weights, exact in int32 (groups of 1 and 2 query heads: "a dot product per lane"; groups of 4
//    and 8: "tile path").  The table is indexed by as many stream bits as the longest code word of the codebook, or by
//    twelve for two symbols at a time, and one 32-bit window serves several lookups with no refill test in between (DecodeMode);
//  * the dequantization is folded into the weights: q.k' = sum_c q_c min_c + sum_c (q_c step_c) code_tc, and
//    p.v'  = sum_t p_t min_t + sum_t (p_t step_t) code_tc;
//  * K and V of a block are handled by the same wave back to back with an online softmax, so scores never go to
//    memory; the next record goes from HBM straight into LDS while the last products of the previous one run;
//  * the sequence is split over workgroups; the workgroup that finishes last merges the splits (the "sum
//    reduction" of Section 3.3.2) inside the same launch.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "huff_decode.cuh"
#include "kvcomp_internal.h"
#include "split_combine.cuh"

namespace kvc {

// Only what the kernel reads, what it reads first in front: the arguments sit in memory that the scalar cache has not seen,
// and every 64-byte line of them costs a trip (about 1 us); early_args() sends for all three at once.
struct FusedArgs {
    const BlockEntry *table;
    const uint8_t *tables, *payload;
    const uint16_t *q;
    FastDiv by_splits, by_heads, by_waves;
    int n_splits, H, max_blocks, n_blocks;
    // second line
    int blocks_per_split, stage_bytes, Hq, n_bh;
    uint32_t mask[2];   // table index mask of each tensor, already scaled to the byte offset of an entry
    float bias[2];      // what the decode tables' symbols are short of: 128 with more than 128 levels, else 0
    float two_eb[2], scale;
    int k_minmax_bytes, n_res, res_head, res_tokens;
    // Append fused into this launch: the newest buffered token (number new_row of the buffer, oldest = 0) is not in the
    // buffer yet but in k_new / v_new [B][H][128]; the wave that reads it also stores it there.  new_row < 0: none.
    int new_row;
    // third line
    float *out, *partials;
    uint32_t *counters;
    const uint16_t *res, *k_new, *v_new;
    int B;
    __device__ __forceinline__ void early_args() const { asm volatile("" ::"s"(new_row), "s"(B)); }
};

// How far a score may exceed the softmax reference of groups of 1 and 2 heads before the state is rescaled.  A block's
// integer weights are scaled by that block's largest numerator, so nothing is lost below e^8 = 2981.
constexpr float kLazyMaxDot = 8.f;

constexpr int kTileMinG = 4;  // smallest query-head group on the tile path

// Symbols reach the matrix cores as int8: as they are with up to 128 levels, minus 128 (FusedArgs::bias) beyond.  Code
// words of up to 7 bits leave at most 128 levels.
template <int LB> constexpr bool kBiased = LB > 7;

// Eight query values.  The query is the caller's and may start at any fp16 element (a view into a larger tensor), so the load
// says that it is only 2-byte aligned; the hardware takes it as one 16-byte load all the same (the HSA ABI runs kernels in
// unaligned access mode).
__device__ __forceinline__ uint4 load_query(const uint16_t *p) {
    typedef uint32_t piece_t __attribute__((ext_vector_type(4), aligned(2)));
    const piece_t v = *(const __attribute__((address_space(1))) piece_t *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// softmax state of one wave for G query heads
template <int G>
struct Soft {
    float m[G], l[G], bv[G], acc[G][2];
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int g = 0; g < G; g++) { m[g] = -INFINITY; l[g] = 0.f; bv[g] = 0.f; acc[g][0] = 0.f; acc[g][1] = 0.f; }
    }
    // s: this lane's score.  Returns its softmax numerator.  The reference m is the same in all lanes and moves only when
    // a score exceeds it by more than kLazyMaxDot (m = -inf before the first block): most blocks then need no maximum
    // over the wave and no rescaling of the sums.  The test is written so that a NaN passes it: a first block whose tokens all
    // score -Inf or NaN gets its reference too.
    __device__ __forceinline__ float update(int g, float s) {
        if (__builtin_amdgcn_ballot_w64(!(s - m[g] <= kLazyMaxDot)) != 0) {
            const float mnew = fmaxf(fmaxf(m[g], wave_max(s)), kLowestRef);
            const float alpha = __expf(m[g] - mnew);
            l[g] *= alpha;
            bv[g] *= alpha;
            acc[g][0] *= alpha;
            acc[g][1] *= alpha;
            m[g] = mnew;
        }
        const float p = __expf(s - m[g]);
        l[g] += p;
        return p;
    }
};

// ---- groups of 1 and 2 query heads: a dot product per lane on the matrix cores ------------------------------------
// Every lane needs the products of ITS OWN decoded symbols with wave-uniform weights (K: token x channels, V: channel x
// tokens).  v_mfma_i32_4x4x4_16b_i8 multiplies sixteen pairs of 4 x 4 matrices, one for each block of four lanes: register i
// of lane l receives sum_k A[i][k] B[k][l % 4], where lane 4b + i holds row i of its block's A and lane l its own column of
// B, four bytes each.  So B is a lane's four packed symbols as they are, A the four digit rows of the weights of these
// four positions, and register i of every lane the dot product of digit row i with the lane's own symbols.  A must be the
// same in all sixteen blocks, and the instruction's broadcast takes it from one of them: block b of ONE register holds
// positions 4b .. 4b + 3, which is what one 4 x 4 byte transposition inside the quads of lanes leaves of a register that holds
// the digits of position l in lane l.  Word w of a slice is multiplied with block w as soon as it is packed: no lane exchange, no
// conversion, no FMA per symbol, no weights in LDS, and no word waits in a register.
//   * A weight w is scaled by a power of two (per block and head) to an integer |W| <= 2^30 and split into four signed
//     bytes, W = sum_j d_j 256^j, the four rows; the products are exact in int32 and the four sums
//     are joined in fp32.  30 bits hold every fp32 weight down to 2^-6 of the block's largest exactly and smaller ones to
//     half a unit, 2^-30 of the largest at most: less than what the rounding of a running fp32 sum over the symbols leaves.
//     Error of the output against float64 over 8 x 4 x 4 heads x 2048 tokens: 0.34 (groups of 1) and 0.40 (2) of what a
//     conversion and an FMA per symbol gave.
//   * the table holds the symbols as int8, from 128 levels on minus `bias` = 128; x' = min + step * code =
//     (min + bias * step) + step * (code - bias), so the bias only enters the constant term.
// 32 heads x 32768 tokens, 16384 block pairs: a conversion and an FMA per symbol 58.6 us a step, v_mfma_i32_16x16x64_i8 with the
// digits in LDS and three quarters of the A operand zero 50.6, this 50.8, with eight words of a half block fewer in registers:
// groups of 2 with code words of up to 10 bits spilled 22 values and took 38.1 us (3 x 8 heads x 12345 tokens), now none and
// 29.2.  The LDS pipe is what is full here (1290 of its cycles a block pair, three quarters of them table lookups).
typedef int v4i __attribute__((ext_vector_type(4)));

// power of two f = 2^up that brings the largest |weight| of the wave into [2^(BITS-1), 2^BITS); *inv = 1 / f.  All in scalar
// registers: the bit patterns of non-negative floats are ordered like the floats.
__device__ __forceinline__ uint32_t wave_max_bits(float v) {
    v = fmaxf(v, dpp_f<kDppXor1>(v));
    v = fmaxf(v, dpp_f<kDppXor2>(v));
    v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_f<kDppMirror>(v));
    const uint32_t u = __float_as_uint(v);
    const uint32_t a = __builtin_amdgcn_readlane(u, 0), b = __builtin_amdgcn_readlane(u, 16),
                   c = __builtin_amdgcn_readlane(u, 32), d = __builtin_amdgcn_readlane(u, 48);
    return max(max(a, b), max(c, d));
}
template <int BITS>
__device__ __forceinline__ float int_scale(float amax, float *inv) {
    const int e = (int)(wave_max_bits(amax) >> 23) - 126;  // amax = m * 2^e, m in [0.5, 1)
    const int up = min(BITS - e, 120);
    *inv = __uint_as_float((uint32_t)(127 - up) << 23);
    return __uint_as_float((uint32_t)(127 + up) << 23);
}
// bytes 0..3: the signed digits of W = w rounded to nearest (cut off, the weights' errors would all have one sign)
__device__ __forceinline__ uint32_t four_digits(float w) { return ((uint32_t)(int)rintf(w) + 0x00808080u) ^ 0x00808080u; }
// sums of at most 128 products of two bytes stay below 2^21, so two neighbouring digits' sums join in an int
__device__ __forceinline__ float join_four(const v4i &d) {
    return fmaf((float)(d.z + d.w * 256), 65536.f, (float)(d.x + d.y * 256));
}
// adds the products of word W of a slice with the weights of its four positions (see above) to the lane's digit sums
template <int W>
__device__ __forceinline__ void add_products(v4i &d, uint32_t digits, uint32_t word) {
    d = __builtin_amdgcn_mfma_i32_4x4x4i8((int)digits, (int)word, d, 4, W, 0);
}

// ---- K block: lane = token; its two slices are channels 0..63 and 64..127 ------------------------------------------
// hdr32: the record (LDS or global).  Leaves scale * q.k' of this lane's token in
// score[].  LB: the table width the kernel is compiled for (see DecodeMode).
template <int G, int LB, class F>
__device__ __forceinline__ void k_block(const uint32_t *hdr32, const char *lut, uint32_t mask, const float (&qreg)[G][2],
                                        float two_eb, float bias, float scale, int lane, int kmm, float (&score)[G],
                                        F &&record_done) {
    static_assert(G < kTileMinG, "groups of 4 and 8 take the tile path");
    // lane c holds the weights of channels c and c + 64.  kmm = bytes of the {min,max} pairs in the header: 512 (one pair
    // per channel) or 16 (BlockQuant: one pair for the whole block)
    const bool per_channel = kmm == kMinMaxBytesK;
    const uint32_t mm0 = hdr32[per_channel ? lane : 0], mm1 = hdr32[per_channel ? lane + 64 : 0];
    const uint32_t sb = hdr32[kmm / 4 + lane];  // bit counts of slices 2*lane and 2*lane+1
    const uint32_t start = wave_excl_scan((sb & 0xffffu) + (sb >> 16), lane);
    const Unit *units = payload_units(hdr32 + (kmm + 2 * kSlices) / 4);
    Quad<DecodeMode<LB>::J> qd;
    qd.open(units, start, sb & 0xffffu, sb >> 16);
    const float mn0 = h2f(mm0 & 0xffffu), mn1 = h2f(mm1 & 0xffffu);
    const float st0 = two_eb * (h2f(mm0 >> 16) - mn0), st1 = two_eb * (h2f(mm1 >> 16) - mn1);
    const QuadTranspose transpose(lane);
    float cst[G], inv[G];
    uint32_t digits[G][2];  // of the channels of either slice
    v4i d[G];
#pragma unroll
    for (int g = 0; g < G; g++) {
        const float w0 = qreg[g][0] * st0, w1 = qreg[g][1] * st1;
        const float f = int_scale<30>(fmaxf(fabsf(w0), fabsf(w1)), &inv[g]);
        digits[g][0] = transpose(four_digits(w0 * f));
        digits[g][1] = transpose(four_digits(w1 * f));
        // the constant part of the dot product is shared by all tokens of the block
        cst[g] = wave_sum(qreg[g][0] * fmaf(bias, st0, mn0) + qreg[g][1] * fmaf(bias, st1, mn1));
        d[g] = v4i{0, 0, 0, 0};
    }
    decode_words<LB>(qd, units, lut, mask, [&](auto slice, auto index, uint32_t word) {
#pragma unroll
        for (int g = 0; g < G; g++) add_products<decltype(index)::value>(d[g], digits[g][decltype(slice)::value], word);
    });
    wave_sync();
    record_done();
#pragma unroll
    for (int g = 0; g < G; g++) score[g] = scale * fmaf(inv[g], join_four(d[g]), cst[g]);
}

// ---- V block: lane = channels 2*lane and 2*lane+1 (its two slices) -------------------------------------------------
// p[g] = softmax numerator of token `lane`.  kLate: another wave is still computing them; they are fetched with
// numerators(p) once the whole block has been decoded, and all products follow.
template <int G, int LB, bool kLate, class F, class N>
__device__ __forceinline__ void v_block(const uint32_t *hdr32, const char *lut, uint32_t mask, float (&p)[G], float two_eb,
                                        float bias, int lane, Soft<G> &st, F &&record_done, N &&numerators) {
    static_assert(G < kTileMinG, "groups of 4 and 8 take the tile path");
    // lane t holds the folded weight p_t * step_t of token t
    const uint32_t mm = hdr32[lane];
    const uint32_t sb = hdr32[kMinMaxBytesV / 4 + lane];
    const uint32_t start = wave_excl_scan((sb & 0xffffu) + (sb >> 16), lane);
    const Unit *units = payload_units(hdr32 + kHdrBytesV / 4);
    Quad<DecodeMode<LB>::J> qd;
    qd.open(units, start, sb & 0xffffu, sb >> 16);
    const float mn = h2f(mm & 0xffffu);
    const float step = two_eb * (h2f(mm >> 16) - mn);
    const QuadTranspose transpose(lane);
    float inv[G];
    uint32_t digits[G];
    v4i d[G][2];
    auto weights = [&] {
#pragma unroll
        for (int g = 0; g < G; g++) {
            const float w = p[g] * step;
            const float f = int_scale<30>(w, &inv[g]);
            digits[g] = transpose(four_digits(w * f));
            st.bv[g] = fmaf(p[g], fmaf(bias, step, mn), st.bv[g]);
            d[g][0] = d[g][1] = v4i{0, 0, 0, 0};
        }
    };
    auto products = [&](auto slice, auto index, uint32_t word) {
#pragma unroll
        for (int g = 0; g < G; g++) add_products<decltype(index)::value>(d[g][decltype(slice)::value], digits[g], word);
    };
    if constexpr (!kLate) {
        weights();
        decode_words<LB>(qd, units, lut, mask, products);
        wave_sync();
        record_done();
    } else {
        SliceWords pw;
        decode_block<LB>(qd, units, lut, mask, pw);
        wave_sync();
        record_done();
        numerators(p);
        weights();
        static_for<0, 16>([&](auto w) {
            products(std::integral_constant<int, 0>(), w, pw.a[decltype(w)::value]);
            products(std::integral_constant<int, 1>(), w, pw.b[decltype(w)::value]);
        });
    }
#pragma unroll
    for (int g = 0; g < G; g++) {
        st.acc[g][0] = fmaf(inv[g], join_four(d[g][0]), st.acc[g][0]);
        st.acc[g][1] = fmaf(inv[g], join_four(d[g][1]), st.acc[g][1]);
    }
}

// Rare path: a record larger than the LDS staging area is decoded straight from global memory.  Kept out of line so
// that it costs the common path no registers.
template <int G, int LB>
__device__ __noinline__ void k_block_global(const uint32_t *rec, const char *lut, uint32_t mask, const float (&qreg)[G][2],
                                            float two_eb, float bias, float scale, int lane, int kmm, float (&score)[G]) {
    k_block<G, LB>(rec, lut, mask, qreg, two_eb, bias, scale, lane, kmm, score, [] {});
}
template <int G, int LB>
__device__ __noinline__ void v_block_global(const uint32_t *rec, const char *lut, uint32_t mask, const float (&p)[G],
                                            float two_eb, float bias, int lane, Soft<G> &st) {
    float pc[G];
#pragma unroll
    for (int g = 0; g < G; g++) pc[g] = p[g];
    v_block<G, LB, false>(rec, lut, mask, pc, two_eb, bias, lane, st, [] {}, [](float (&)[G]) {});
}

// ---- groups of 4 and 8 query heads, tile path ---------------------------------------------------------------------
// With several query heads per KV head the update of the accumulators is a matrix product, (heads x symbols) weights
// times the decoded block, and the decode itself is the same for all heads.  The wave therefore only packs the
// decoded symbols, four table entries to a register -- less work than one conversion and one FMA per symbol and
// head -- and multiplies them with the folded weights on v_mfma_i32_32x32x32_i8, whose result tiles (32 rows of
// weights x 32 columns) give the path its name:
//   * a register of packed symbols is an MFMA operand as it is, with no conversion; the operand wants 32 columns x 32 positions from 64 lanes that hold
//     one slice each, which one v_permlane32_swap_b32 per register arranges (step_operands);
//   * a weight w is scaled by a per-block power of two to an integer W below 2^22 and split into three signed bytes,
//     W = sum_j d_j 256^j; row 4 * head + j of the A operand holds digit j, the products are exact in int32, and the
//     digit rows of a head land in the same lane of the result, where they are recombined in fp32;
//   * the products run once the whole block is decoded: 32 registers hold it, and the result tiles take the place of the
//     stream readers.  With products after each half every digit sum was recombined twice (16 x 8 heads x 8192 tokens, groups
//     of 4: 60.4 -> 57.4 us a step, with the fourth wave per SIMD that then fits; 8 x 8 heads x 16384, groups of 8: 71.3 ->
//     65.5; code words of up to 10 bits, whose kernels of groups of 8 could hold two waves per SIMD before and hold three now,
//     8 x 8 heads x 8192: 56.0 -> 47.8);
//   * with more than 128 levels the table holds symbol - 128: sum_c W_c (s_c - 128) misses 128 * sum_c W_c, which joins
//     the constant term of the block.
// Lane l of the result tiles holds column l % 32 (token of a K block, channel of a V block) for the heads
// l / 32 + 2 i: the running softmax state lives in that layout and is converted to the per-channel layout of the
// other paths once, after the last block.
typedef int v16i __attribute__((ext_vector_type(16)));

template <int G>
struct TileSoft {
    static constexpr int HL = G / 2;  // heads per lane: l / 32 + 2 i
    float m[HL], l[HL], bv[HL], acc[HL][4];  // l, bv: this lane's share; acc[i][ct]: channel 32 ct + l % 32
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int i = 0; i < HL; i++) {
            m[i] = -INFINITY; l[i] = 0.f; bv[i] = 0.f;
#pragma unroll
            for (int c = 0; c < 4; c++) acc[i][c] = 0.f;
        }
    }
};

// maximum over the 32 lanes of this lane's half of the wave
__device__ __forceinline__ float half_max(float v, bool upper) {
    v = fmaxf(v, dpp_f<kDppXor1>(v));
    v = fmaxf(v, dpp_f<kDppXor2>(v));
    v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_f<kDppMirror>(v));
    const float lo = fmaxf(bcast(v, 0), bcast(v, 16)), hi = fmaxf(bcast(v, 32), bcast(v, 48));
    return upper ? hi : lo;
}

// The B operands of v_mfma_i32_32x32x32_i8 for one step of 32 positions (words w[8 STEP] .. of a slice) straight from
// registers.  Lane l of the operand supplies column l % 32 and positions 16 (l / 32) .. +15.  With one slice per lane and
// 64 lanes there are two column tiles: tile 0 wants words 0..3 of lanes 0..31 in its lower half and words 4..7 of the
// same lanes in its upper half, tile 1 words 0..3 of lanes 32..63 in its lower half and their words 4..7 in its upper
// half -- which is what v_permlane32_swap_b32 makes of (word i, word 4 + i).
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void step_operands(const uint32_t (&w)[16], int step, v4i &tile0, v4i &tile1) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const v2u r = __builtin_amdgcn_permlane32_swap(w[8 * step + i], w[8 * step + 4 + i], false, false);
        tile0[i] = (int)r.x;
        tile1[i] = (int)r.y;
    }
}
// v[i] summed over the 32 lanes of this lane's half of the wave, in every lane.  The values are folded together while the
// lanes are: one register is left after the steps inside a row of 16 that take as many as one value alone would.
template <int HL>
__device__ __forceinline__ void half_sums(float (&v)[HL], int lane) {
    static_assert(HL == 2 || HL == 4);
    constexpr int kRor8 = 0x128;
    float m[2];
#pragma unroll
    for (int i = 0; i < HL; i += 2) {  // lanes 0..3 and 8..11 of a row go on with v[i], the others with v[i + 1]
        const float a = v[i] + dpp_f<kDppHalfMirror>(v[i]), b = v[i + 1] + dpp_f<kDppHalfMirror>(v[i + 1]);
        m[i / 2] = (lane & 4) ? b : a;
    }
    float r = m[0] + dpp_f<kRor8>(m[0]);
    if constexpr (HL == 4) {
        const float b = m[1] + dpp_f<kRor8>(m[1]);
        r = (lane & 8) ? b : r;
    }
    r += dpp_f<kDppXor1>(r);
    r += dpp_f<kDppXor2>(r);  // lane 4 i: the row's sum of v[i]
    const v2u two = __builtin_amdgcn_permlane16_swap(__float_as_uint(r), __float_as_uint(r), false, false);
    r = __uint_as_float(two.x) + __uint_as_float(two.y);
    v[0] = dpp_f<0x150>(r);  // row_newbcast
    v[1] = dpp_f<0x154>(r);
    if constexpr (HL == 4) {
        v[2] = dpp_f<0x158>(r);
        v[3] = dpp_f<0x15c>(r);
    }
}

// Rounding to an integer inside the multiplication: for |a * b| <= 2^22, fma(a, b, 1.5 * 2^23) is rounded (to nearest,
// ties to even) at unit spacing, and its bit pattern is kMagicBits + W with W = rint(a * b), also across the binade
// boundary at W = 2^22.  One instruction instead of a product, a rounding and a conversion; W stays implicit:
//   magic_digits(bits): bytes 0..2 are the signed digits d_j of W = d2 2^16 + d1 2^8 + d0, and sums of W are sums of bit patterns minus n * kMagicBits.
constexpr float kMagic = 12582912.f;          // 1.5 * 2^23
constexpr uint32_t kMagicBits = 0x4B400000u;  // its bit pattern
__device__ __forceinline__ uint32_t magic_round(float a, float b) { return __float_as_uint(fmaf(a, b, kMagic)); }
__device__ __forceinline__ uint32_t magic_digits(uint32_t bits) { return (bits + (0x00008080u - kMagicBits)) ^ 0x00008080u; }
// words a..d (byte j = digit j of four consecutive columns) -> o[j] = digit j of the four columns, j < 3
__device__ __forceinline__ void transpose_digits(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&o)[3]) {
    const uint32_t t0 = __builtin_amdgcn_perm(b, a, 0x05010400u), t1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t t2 = __builtin_amdgcn_perm(d, c, 0x05010400u), t3 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
}
// the digit sums of one head, rows 4 i .. 4 i + 2 of a result tile, as one number (see join_four)
template <int I>
__device__ __forceinline__ float join_digits(const v16i &d) {
    return fmaf((float)d[4 * I + 2], 65536.f, (float)(d[4 * I] + d[4 * I + 1] * 256));
}
template <int HL>
__device__ __forceinline__ void join_all(const v16i &d, float (&out)[HL]) {
    out[0] = join_digits<0>(d);
    out[1] = join_digits<1>(d);
    if constexpr (HL > 2) {
        out[HL > 2 ? 2 : 0] = join_digits<2>(d);
        out[HL > 2 ? 3 : 0] = join_digits<3>(d);
    }
}
// Bytes per row of the A operand while it is laid out in the tile area: whole 16-byte reads, eight neighbouring rows in
// different banks.  Only the three digit rows of every head are
// stored: row 4 * head + digit of the operand sits at row 3 * head + digit of the area; the lanes of the operand's remaining rows
// read zeros instead.
constexpr int kARowK = kARowBytes, kARowV = kBT + 16;
// where lane l = (x, hv) of the operand reads: row x, byte 16 hv of every step of 32
template <int G, int ROW>
__device__ __forceinline__ const v4i *a_row(const uint8_t *tile, const uint8_t *zeros, int x, int hv) {
    const uint8_t *row = (x & 3) == 3 || x >= 4 * G ? zeros : tile + (3 * (x >> 2) + (x & 3)) * ROW;
    return reinterpret_cast<const v4i *>(row + 16 * hv);
}

// How far a score may exceed the softmax reference before the state is rescaled.  The numerators of a block then
// reach e^kLazyMax, and because the integer weights of all heads share one power-of-two scale per block, a head
// whose reference is behind costs the other heads that factor in weight resolution: 2 keeps the attention error
// within a factor 8 of rescaling always (measured at the 70B shape: 1e-5 instead of 4e-6; with 8 it reached 1e-3).
constexpr float kLazyMax = 2.f;

// K block.  hdr32: the record (LDS or global); tile: this wave's LDS area for laying out the A operand; qf: the query
// rows in LDS.
// Updates the softmax state and leaves the softmax numerators of tokens l%32 and 32 + l%32 in p.
// record_done() is called once the record has been read for the last time, before the last products: the place to
// request the next record, whose loads then travel while few registers are live.
template <int G, int LB, class F>
__device__ __forceinline__ void k_tile_block(const uint32_t *hdr32, const char *lut, uint32_t mask2, uint8_t *tile,
                                             const uint8_t *zeros, const float *qf, float two_eb, float bias, float scale, int lane, int kmm,
                                             TileSoft<G> &ts, float (&p)[G / 2][2], F &&record_done) {
    constexpr int HL = G / 2;
    // everything derived from the lane number is recomputed per block (a few instructions) instead of being kept in
    // registers, or spilled, across the whole decode loop
    asm volatile("" : "+v"(lane));
    const int x = lane & 31, hv = lane >> 5;
    const bool upper = hv != 0;
    const bool per_channel = kmm == kMinMaxBytesK;
    // the A operand: folded weights q_c * step_c as integers, heads l/32 + 2i, channels 4 (l%32) .. +3
    float cst[HL], inv;
    {
        float mn[4], stp[4];
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const uint32_t mm = hdr32[per_channel ? 4 * x + c : 0];
            mn[c] = h2f(mm & 0xffffu);
            stp[c] = two_eb * (h2f(mm >> 16) - mn[c]);
        }
        float qa[HL][4], amax = 0.f;
#pragma unroll
        for (int c = 0; c < 4; c++) {   // the largest |q_c step_c| of this lane: steps are not negative
            float qmax = 0.f;
#pragma unroll
            for (int i = 0; i < HL; i++) {
                qa[i][c] = qf[(hv + 2 * i) * kD + 4 * x + c];
                qmax = fmaxf(qmax, fabsf(qa[i][c]));
            }
            amax = fmaxf(amax, qmax * stp[c]);
        }
        const float f = int_scale<22>(amax, &inv);
#pragma unroll
        for (int c = 0; c < 4; c++) stp[c] *= f;   // exact: f is a power of two
#pragma unroll
        for (int i = 0; i < HL; i++) {
            uint32_t dg[4], wbits = 0;
            float qm = 0.f;
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const uint32_t bits = magic_round(qa[i][c], stp[c]);  // W = rint(q_c step_c f), |W| <= 2^22
                wbits += bits;
                qm = fmaf(qa[i][c], mn[c], qm);
                dg[c] = magic_digits(bits);
            }
            if constexpr (kBiased<LB>) qm = fmaf(bias * inv, (float)(int)(wbits - 4u * kMagicBits), qm);
            uint32_t rows[3];
            transpose_digits(dg[0], dg[1], dg[2], dg[3], rows);
            const int head = hv + 2 * i;
#pragma unroll
            for (int j = 0; j < 3; j++) *reinterpret_cast<uint32_t *>(tile + (3 * head + j) * kARowK + 4 * x) = rows[j];
            cst[i] = qm;
        }
        half_sums<HL>(cst, lane);
    }
    const uint32_t sb = hdr32[kmm / 4 + lane];  // bit counts of slices 2*lane and 2*lane+1
    const uint32_t start = wave_excl_scan((sb & 0xffffu) + (sb >> 16), lane);
    const Unit *units = payload_units(hdr32 + (kmm + 2 * kSlices) / 4);
    Quad<DecodeMode<LB>::J> qd;
    qd.open(units, start, sb & 0xffffu, sb >> 16);
    float sc[HL][2];
    {
        SliceWords pw;  // lane = token: slice a = its channels 0..63, slice b = its channels 64..127
        decode_block<LB>(qd, units, lut, mask2, pw);
        wave_sync();
        const v4i *row = a_row<G, kARowK>(tile, zeros, x, hv);  // read here: no register holds it during the decode
        v4i a[4];
#pragma unroll
        for (int ks = 0; ks < 4; ks++) a[ks] = row[2 * ks];
        record_done();
        const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        v16i d[2];  // result tiles: tokens 0..31 and 32..63
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {  // steps of 32 channels
            v4i t0, t1;
            step_operands(ks < 2 ? pw.a : pw.b, ks & 1, t0, t1);
            d[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], t0, ks ? d[0] : zero, 0, 0, 0);
            d[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], t1, ks ? d[1] : zero, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 2; t++) {
            float v[HL];
            join_all<HL>(d[t], v);
#pragma unroll
            for (int i = 0; i < HL; i++) sc[i][t] = v[i];
        }
    }
    // Online softmax with a reference value m that only moves when it has to: the state is rescaled (a maximum over
    // the tokens of every head, six multiplications per head) only when some score of the block exceeds its head's m
    // by more than kLazyMax, which after the first blocks of a sequence split is rare.  Until then the numerators are
    // at most e^kLazyMax instead of 1; the merges divide by the same m.
    const float si = scale * inv;
    float over = -INFINITY;
#pragma unroll
    for (int i = 0; i < HL; i++) {
        const float sk = scale * cst[i];
        sc[i][0] = fmaf(si, sc[i][0], sk);
        sc[i][1] = fmaf(si, sc[i][1], sk);
        // m = -inf before the first block: +inf, whatever the scores are
        over = fmaxf(over, fmaxf(fmaxf(sc[i][0], sc[i][1]), kLowestRef) - ts.m[i]);
    }
    if (__builtin_amdgcn_ballot_w64(over > kLazyMax) != 0) {
#pragma unroll
        for (int i = 0; i < HL; i++) {
            const float mnew = fmaxf(fmaxf(ts.m[i], half_max(fmaxf(sc[i][0], sc[i][1]), upper)), kLowestRef);
            const float alpha = __expf(ts.m[i] - mnew);
            ts.l[i] *= alpha;
            ts.bv[i] *= alpha;
#pragma unroll
            for (int c = 0; c < 4; c++) ts.acc[i][c] *= alpha;
            ts.m[i] = mnew;
        }
    }
#pragma unroll
    for (int i = 0; i < HL; i++) {
        p[i][0] = __expf(sc[i][0] - ts.m[i]);
        p[i][1] = __expf(sc[i][1] - ts.m[i]);
        ts.l[i] += p[i][0] + p[i][1];
    }
}

// V block.  p: softmax numerators of tokens l%32 and 32 + l%32 for this lane's heads.  kLate: see v_block.
template <int G, int LB, bool kLate, class F, class N>
__device__ __forceinline__ void v_tile_block(const uint32_t *hdr32, const char *lut, uint32_t mask2, uint8_t *tile,
                                             const uint8_t *zeros, float (&p)[G / 2][2], float two_eb, float bias, int lane,
                                             TileSoft<G> &ts, F &&record_done, N &&numerators) {
    constexpr int HL = G / 2;
    asm volatile("" : "+v"(lane));
    const int x = lane & 31, hv = lane >> 5;
    float inv;
    uint32_t minmax[2];
    if constexpr (kLate) {  // the record's staging area may be reused before the weights are made
        minmax[0] = hdr32[x];
        minmax[1] = hdr32[32 + x];
    }
    auto weights = [&] {
        float mn[2], stp[2];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            const uint32_t mm = kLate ? minmax[t] : hdr32[32 * t + x];
            mn[t] = h2f(mm & 0xffffu);
            stp[t] = two_eb * (h2f(mm >> 16) - mn[t]);
        }
        float pmax[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < HL; i++) {
            pmax[0] = fmaxf(pmax[0], p[i][0]);
            pmax[1] = fmaxf(pmax[1], p[i][1]);
        }
        const float f = int_scale<22>(fmaxf(pmax[0] * stp[0], pmax[1] * stp[1]), &inv);
        stp[0] *= f;   // exact: f is a power of two
        stp[1] *= f;
#pragma unroll
        for (int i = 0; i < HL; i++) {
            const int head = hv + 2 * i;
            uint32_t wbits = 0;
#pragma unroll
            for (int t = 0; t < 2; t++) {
                const uint32_t bits = magic_round(p[i][t], stp[t]);  // W = rint(p_t step_t f), |W| <= 2^22
                wbits += bits;
                const uint32_t dg = magic_digits(bits);
#pragma unroll
                for (int j = 0; j < 3; j++) tile[(3 * head + j) * kARowV + 32 * t + x] = (uint8_t)(dg >> (8 * j));
            }
            if constexpr (kBiased<LB>) ts.bv[i] = fmaf(bias * inv, (float)(int)(wbits - 2u * kMagicBits), ts.bv[i]);
            ts.bv[i] += fmaf(p[i][0], mn[0], p[i][1] * mn[1]);
        }
    };
    if constexpr (!kLate) weights();
    // lane = channels lane (slice a) and 64 + lane (slice b), so that a result tile of 32 channels is one slice of 32
    // neighbouring lanes; slice s starts where the bits of slices 0 .. s-1 end
    const uint16_t *bits16 = reinterpret_cast<const uint16_t *>(hdr32 + kMinMaxBytesV / 4);
    const uint32_t abits = bits16[lane], bbits = bits16[kSliceLen + lane];
    const uint32_t start_a = wave_excl_scan(abits, lane);
    const uint32_t start_b = (uint32_t)__builtin_amdgcn_readlane((int)(start_a + abits), 63) + wave_excl_scan(bbits, lane);
    const Unit *units = payload_units(hdr32 + kHdrBytesV / 4);
    Quad<DecodeMode<LB>::J> qd;
    qd.open2(units, start_a, abits, start_b, bbits);
    SliceWords pw;
    decode_block<LB>(qd, units, lut, mask2, pw);
    wave_sync();
    record_done();
    if constexpr (kLate) {
        numerators(p);
        weights();
        wave_sync();
    }
    const v4i *row = a_row<G, kARowV>(tile, zeros, x, hv);
    const v4i a[2] = {row[0], row[2]};
#pragma unroll
    for (int sl = 0; sl < 2; sl++) {  // result tiles: channels 0..31, 32..63 (slice a), 64..95, 96..127 (slice b)
        const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        v16i d[2];
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {  // steps of 32 tokens
            v4i t0, t1;
            step_operands(sl ? pw.b : pw.a, ks, t0, t1);
            d[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], t0, ks ? d[0] : zero, 0, 0, 0);
            d[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ks], t1, ks ? d[1] : zero, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 2; t++) {
            float v[HL];
            join_all<HL>(d[t], v);
#pragma unroll
            for (int i = 0; i < HL; i++) ts.acc[i][2 * sl + t] = fmaf(inv, v[i], ts.acc[i][2 * sl + t]);
        }
    }
}

// Rare path: a record larger than the LDS staging area (one that an append flushed after the host last looked at the
// record sizes) is decoded straight from global memory, out of line.
template <int G, int LB>
__device__ __noinline__ void k_tile_block_global(const uint32_t *rec, const char *lut, uint32_t mask2, uint8_t *tile,
                                                 const uint8_t *zeros, const float *qf, float two_eb, float bias, float scale, int lane, int kmm,
                                                 TileSoft<G> &ts, float (&p)[G / 2][2]) {
    k_tile_block<G, LB>(rec, lut, mask2, tile, zeros, qf, two_eb, bias, scale, lane, kmm, ts, p, [] {});
}
template <int G, int LB>
__device__ __noinline__ void v_tile_block_global(const uint32_t *rec, const char *lut, uint32_t mask2, uint8_t *tile,
                                                 const uint8_t *zeros, const float (&p)[G / 2][2], float two_eb, float bias, int lane,
                                                 TileSoft<G> &ts) {
    float pc[G / 2][2];
#pragma unroll
    for (int i = 0; i < G / 2; i++) { pc[i][0] = p[i][0]; pc[i][1] = p[i][1]; }
    v_tile_block<G, LB, false>(rec, lut, mask2, tile, zeros, pc, two_eb, bias, lane, ts, [] {}, [](float (&)[G / 2][2]) {});
}

// A wave's softmax state parked in LDS for the merge of the workgroup's waves: o[g][channel] in the wave's own staging area,
// its reference m and, summed over the lanes, l and bv (what every channel's o is short of) in ml[m, l, bv][g][wave].  The
// buffered tokens are merged into it there, and the tile path changes its layout this way.
constexpr int kMergeWaves = 16;
template <int G>
__device__ __forceinline__ float *merge_word(float *ml, int word, int g, int wave) {
    return ml + (word * G + g) * kMergeWaves + wave;
}
template <int G>
__device__ __forceinline__ void soft_to_area(const Soft<G> &st, float *area, float *ml, int wave, int lane) {
    wave_sync();
#pragma unroll
    for (int g = 0; g < G; g++) {
        *reinterpret_cast<float2 *>(area + g * kD + 2 * lane) = make_float2(st.acc[g][0], st.acc[g][1]);
        const float l = wave_sum(st.l[g]), bv = wave_sum(st.bv[g]);
        if (lane == 0) {
            *merge_word<G>(ml, 0, g, wave) = st.m[g];
            *merge_word<G>(ml, 1, g, wave) = l;
            *merge_word<G>(ml, 2, g, wave) = bv;
        }
    }
    wave_sync();
}
// the tile path's state: lane l holds column l % 32, heads l / 32 + 2 i
template <int G>
__device__ __forceinline__ void soft_to_area(const TileSoft<G> &ts, float *area, float *ml, int wave, int lane) {
    constexpr int HL = G / 2;
    const int x = lane & 31, hv = lane >> 5;
    wave_sync();
    float l[HL], bv[HL];
#pragma unroll
    for (int i = 0; i < HL; i++) {
        const int head = hv + 2 * i;
#pragma unroll
        for (int ct = 0; ct < 4; ct++) area[head * kD + 32 * ct + x] = ts.acc[i][ct];
        l[i] = ts.l[i];
        bv[i] = ts.bv[i];
    }
    half_sums<HL>(l, lane);
    half_sums<HL>(bv, lane);
#pragma unroll
    for (int i = 0; i < HL; i++) {
        if (x == 0) {
            *merge_word<G>(ml, 0, hv + 2 * i, wave) = ts.m[i];
            *merge_word<G>(ml, 1, hv + 2 * i, wave) = l[i];
            *merge_word<G>(ml, 2, hv + 2 * i, wave) = bv[i];
        }
    }
    wave_sync();
}

// The buffered fp16 tokens (Section 3.2.3: the newest vectors take part too), in units of 16 tokens; this wave takes
// units first_unit, first_unit + unit_step, ...  Token r of the buffer (oldest = 0) sits in slot
// (res_head + r) mod res_tokens; res_head is a multiple of 64, so a unit never wraps.
// A unit is read with four 16-byte loads per lane and tensor, K and V together and all in flight at once: a single wave
// has nothing else to hide the memory latency with, and small units spread the buffer over many waves.
//   scores : v_mfma_f32_16x16x32_f16, tokens x heads.  Lane l supplies K row l % 16 and query head l % 16, channels
//            32 i + 8 (l / 16) .. +7 in step i, and receives head l % 16 of the tokens 4 (l / 16) .. +3.  Each step has an
//            accumulator of its own and the four are added as a tree: a score is a fp32 sum over 128 channels, and its
//            rounding decides the error of the output (one running accumulator: half as much error again, same time
//            within 2 %).
//   p . V  : lane l holds channels 8 (l % 16) .. +7 of those same four tokens, so a numerator reaches the 16 lanes that
//            multiply with it by a broadcast inside their row of 16, which rides on the FMA.
// All heads of a group share the loads, the matrix instructions and one running softmax per unit; only the FMAs of p . V
// grow with the group.  (One head after the other on the vector ALU, with its own reductions and lane exchanges, a unit
// took 5 us for groups of 4: the waves that had one finished last.)
// When the append of the newest token is fused into the launch (new_row >= 0), its row comes from k_new / v_new
// instead of the buffer, and the lanes that read it store it into its buffer slot for the launches to come: one
// wave of the grid per (batch, head) owns that row, so there is one writer and no reader of the slot in this launch.
// The result is merged into the wave's parked state (`area` and `ml`, see soft_to_area).
// Inline: the decode loops leave room for it, and out of line it saves and restores the registers that a callee has to keep,
// through scratch memory (4 x 8 heads x 9000 tokens, 1024 of them buffered, groups of 8: 29.3 -> 27.6 us).
constexpr int kUnitTokens = 16;
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// acc + (w of lane N of this lane's row of 16) * x: the broadcast is a DPP modifier of the FMA's first operand.  w must
// not have been written by a VALU instruction in the two wait states before (row_operand()).
template <int N>
__device__ __forceinline__ float fma_row(float w, float x, float acc) {
    static_assert(N >= 0 && N < 8, "lane of the row");
#define KVC_FMA_ROW(n) if constexpr (N == n) asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:" #n " row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(w), "v"(x))
    KVC_FMA_ROW(0); KVC_FMA_ROW(1); KVC_FMA_ROW(2); KVC_FMA_ROW(3); KVC_FMA_ROW(4); KVC_FMA_ROW(5); KVC_FMA_ROW(6); KVC_FMA_ROW(7);
#undef KVC_FMA_ROW
    return acc;
}
__device__ __forceinline__ void row_operand(float &a, float &b, float &c, float &d) {
    asm volatile("s_nop 1" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
// w of lane n of this lane's row of 16
template <int N>
__device__ __forceinline__ float row_bcast(float w) { return dpp_f<0x150 + N>(w); }
template <int G, int N = 0, class F>
__device__ __forceinline__ void for_heads(F &&f) {  // f(integral constant) for the heads 0 .. G-1
    if constexpr (N < G) {
        f(std::integral_constant<int, N>());
        for_heads<G, N + 1>(f);
    }
}
// a + b over the two halves / the neighbouring rows of the wave: the first half (even rows) receives a's sum, the second
// (odd rows) b's
__device__ __forceinline__ float fold_halves(float a, float b) {
    const v2u r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
__device__ __forceinline__ float fold_rows(float a, float b) {
    const v2u r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
__device__ __forceinline__ float max_over_rows(float v) {  // over the four rows of 16, per lane of the row
    v2u r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}

template <int G>
__device__ __forceinline__ void buffered_units(const uint16_t *res, int res_tokens, int B, int H, int b, int h,
                                             int res_head, int n_res, int first_unit, int unit_step,
                                             const uint16_t *q0, float scale, int lane, const uint16_t *k_new,
                                             const uint16_t *v_new, int new_row, float *area, float *ml, int wave) {
    const size_t res_tensor = (size_t)B * res_tokens * H * kD;
    const int n_units = (n_res + kUnitTokens - 1) / kUnitTokens;
    const int col = lane & 15, grp = lane >> 4;
    uint4 qb[4];  // head `col` of the group (zeros beyond it)
#pragma unroll
    for (int i = 0; i < 4; i++)
        qb[i] = col < G ? load_query(q0 + col * kD + 32 * i + 8 * grp) : make_uint4(0, 0, 0, 0);
    float m = -INFINITY, l = 0.f;  // running maximum of head `col`; its sum, this lane's share
    float av[G][8];                // channels 8 col .. +7 of every head, this row's tokens
#pragma unroll
    for (int g = 0; g < G; g++)
#pragma unroll
        for (int k = 0; k < 8; k++) av[g][k] = 0.f;
    for (int u = first_unit; u < n_units; u += unit_step) {
        const int n_tok = min(kUnitTokens, n_res - u * kUnitTokens);
        int slot0 = res_head + u * kUnitTokens;
        if (slot0 >= res_tokens) slot0 -= res_tokens;
        const int new_tok = new_row - u * kUnitTokens;  // the appended token's number inside the unit, if it is in there
        const size_t new_off = ((size_t)b * H + h) * kD;
        const size_t buf0 = (((size_t)b * res_tokens + slot0) * H + h) * kD, row = (size_t)H * kD;
        uint4 rk[4], rv[4];
        {
            const uint16_t *src = (col == new_tok ? k_new + new_off : res + buf0 + col * row) + 8 * grp;
#pragma unroll
            for (int i = 0; i < 4; i++)
                rk[i] = col < n_tok ? *reinterpret_cast<const uint4 *>(src + 32 * i) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int t = 4 * grp + i;
            const uint16_t *src = (t == new_tok ? v_new + new_off : res + res_tensor + buf0 + t * row) + 8 * col;
            rv[i] = t < n_tok ? *reinterpret_cast<const uint4 *>(src) : make_uint4(0, 0, 0, 0);
        }
        if (new_row >= 0 && new_tok >= 0 && new_tok < kUnitTokens) {
            uint16_t *wr = const_cast<uint16_t *>(res) + buf0 + new_tok * row;
            if (col == new_tok) {
#pragma unroll
                for (int i = 0; i < 4; i++) *reinterpret_cast<uint4 *>(wr + 32 * i + 8 * grp) = rk[i];
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (4 * grp + i == new_tok) *reinterpret_cast<uint4 *>(wr + res_tensor + 8 * col) = rv[i];
        }
        v4f s[4];
#pragma unroll
        for (int i = 0; i < 4; i++)
            s[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, rk[i]), __builtin_bit_cast(v8h, qb[i]), v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        float p[4], mu = kLowestRef;
#pragma unroll
        for (int r = 0; r < 4; r++) p[r] = (s[0][r] + s[1][r]) + (s[2][r] + s[3][r]);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            p[r] = 4 * grp + r < n_tok ? scale * p[r] : -INFINITY;
            mu = fmaxf(mu, p[r]);
        }
        const float mnew = fmaxf(m, max_over_rows(mu));
        if (u != first_unit && __builtin_amdgcn_ballot_w64(mnew > m) != 0) {
            const float alpha = __expf(m - mnew);
            l *= alpha;
            for_heads<G>([&](auto gc) {
                constexpr int g = decltype(gc)::value;
                const float ag = row_bcast<g>(alpha);
#pragma unroll
                for (int k = 0; k < 8; k++) av[g][k] *= ag;
            });
        }
        m = mnew;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            p[r] = __expf(p[r] - mnew);
            l += p[r];
        }
        row_operand(p[0], p[1], p[2], p[3]);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t w[4] = {rv[i].x, rv[i].y, rv[i].z, rv[i].w};
            float x[8];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                x[2 * k] = h2f(w[k] & 0xffffu);
                x[2 * k + 1] = h2f(w[k] >> 16);
            }
            for_heads<G>([&](auto gc) {
                constexpr int g = decltype(gc)::value;
#pragma unroll
                for (int k = 0; k < 8; k++) av[g][k] = fma_row<g>(p[i], x[k], av[g][k]);
            });
        }
    }
    // merge with the parked state: head `col` in the lanes of its column
    l = fold_halves(l, l);
    l = fold_rows(l, l);
    float fa = 1.f, fb = 0.f;
    if (col < G) {
        float *pm = merge_word<G>(ml, 0, col, wave), *pl = merge_word<G>(ml, 1, col, wave), *pb = merge_word<G>(ml, 2, col, wave);
        const float ma = *pm, mx = fmaxf(ma, m);
        fa = __expf(ma - mx);  // 0 for a state that is still empty
        fb = __expf(m - mx);
        const float l1 = fmaf(*pl, fa, l * fb), bv1 = *pb * fa;
        wave_sync();
        if (grp == 0) { *pm = mx; *pl = l1; *pb = bv1; }
    }
    // fold the four rows: lane (grp, col) ends up with channels 8 col + 2 grp, +1 of all tokens
    for_heads<G>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        float w4[4];
#pragma unroll
        for (int k = 0; k < 4; k++) w4[k] = fold_halves(av[g][k], av[g][4 + k]);
        const float o0 = fold_rows(w4[0], w4[2]), o1 = fold_rows(w4[1], w4[3]);
        float2 *at = reinterpret_cast<float2 *>(area + g * kD + 8 * col + 2 * grp);
        const float2 old = *at;
        const float a = row_bcast<g>(fa), c = row_bcast<g>(fb);
        *at = make_float2(fmaf(old.x, a, o0 * c), fmaf(old.y, a, o1 * c));
    });
    wave_sync();
}

// The same out of line, for the kernels with a wave per record for code words beyond 6 bits: they have one unit or two, and the
// registers of twelve waves.  Called from kernels of sixteen waves it would have 128 registers and spill (4 x 8 heads, groups of 4,
// 1000 buffered tokens and no block: 30 us where inline takes 17).
template <int G>
__device__ __noinline__ void buffered_tokens(const uint16_t *res, int res_tokens, int B, int H, int b, int h,
                                             int res_head, int n_res, int first_unit, int unit_step,
                                             const uint16_t *q0, float scale, int lane, const uint16_t *k_new,
                                             const uint16_t *v_new, int new_row, float *area, float *ml, int wave) {
    buffered_units<G>(res, res_tokens, B, H, b, h, res_head, n_res, first_unit, unit_step, q0, scale, lane, k_new, v_new, new_row,
                      area, ml, wave);
}

// One workgroup per CU, as many waves as the registers allow per SIMD (fused_waves_per_simd): 4 (128 VGPRs) or 3 (168).  The host may launch fewer waves per workgroup (short sequences,
// large staging areas).
template <int G, int LB, bool kPaired> struct MaxWaves { static constexpr int value = fused_max_waves(G, kPaired); };

// LB = the table width the kernel is compiled for (>= longest code word of both codebooks), see DecodeMode.
//
// kPaired: a short cache leaves wave slots empty, and the time of a step is the serial chain of one wave: K record, softmax,
// V record.  The two decodes do not depend on each other, so with 2 * blocks_per_split wave slots wave w decodes the K
// record of the split's block w and wave blocks_per_split + w its V record at the same time; the softmax numerators go
// from the first to the second through the first one's record area (free by then), announced by a flag in LDS.  The waves
// behind them take the buffered tokens.  The V waves hold the state, the K waves end empty-handed.
// 1 head x 1024 tokens 9.4 -> 7.9 us a step, 96 tokens appended to 2000 (8 heads, groups of 4) 1424 -> 1134 us.
template <int G, int LB, bool kPaired>
__global__ __launch_bounds__((64 * MaxWaves<G, LB, kPaired>::value), 1) void fused_attn_kernel(FusedArgs a) {
    using M = DecodeMode<LB>;
    constexpr bool kTile = G >= kTileMinG;  // packed symbols in registers, int8 MFMA
    __shared__ __attribute__((aligned(16))) uint8_t lut_s[2][M::kTableBytes];
    __shared__ __attribute__((aligned(16))) float qf[kTile ? G * kD : 4];
    __shared__ __attribute__((aligned(16))) uint8_t zeros[kTile ? kD : 16];  // tile path: the A operand's rows without a digit
    __shared__ uint32_t ready[kPaired ? 16 : 1];  // paired: wave w's numerators are in its record area
    __shared__ float merge_ml[3 * G * kMergeWaves];  // see soft_to_area
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // per wave: staging area; tile path: + weights
    const int tid = threadIdx.x, lane = tid & 63, n_threads = blockDim.x;
    // the wave number and everything derived from it (block numbers, table entries, record addresses) are scalars
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_waves = __builtin_amdgcn_readfirstlane(n_threads >> 6);
    uint8_t *stage = smem + (size_t)wave * a.stage_bytes;
    constexpr int kWeightBytes = (int)fused_weight_bytes(G);
    // the wave's weight area (tile path): digit rows of the A operand
    uint8_t *tile = smem + (size_t)n_waves * a.stage_bytes + (size_t)wave * kWeightBytes;
    const char *lutK = reinterpret_cast<const char *>(&lut_s[0][0]);
    const char *lutV = reinterpret_cast<const char *>(&lut_s[1][0]);

    a.early_args();
    // Workgroups go to the eight XCDs round-robin by their linear number, and each XCD has its own L2.  Numbering the
    // (batch-head, split) pairs so that an XCD gets a contiguous range of them keeps the splits of one head -- whose
    // records are neighbours in memory and share cache lines at their ends, and whose partials the last of them
    // merges -- behind one L2.
    int item = blockIdx.x;
    if ((gridDim.x & (kXCDs - 1)) == 0) item = (item & (kXCDs - 1)) * (gridDim.x / kXCDs) + item / kXCDs;
    const int bh = (int)a.by_splits((uint32_t)item), split = item - bh * a.n_splits;
    const int b = (int)a.by_heads((uint32_t)bh), h = bh - b * a.H;

    const int j0 = split * a.blocks_per_split;
    const int j1 = min(j0 + a.blocks_per_split, a.n_blocks);
    const BlockEntry *tabK = a.table + (size_t)bh * a.max_blocks, *tabV = tabK + (size_t)a.n_bh * a.max_blocks;
    const uint32_t stage16 = (uint32_t)(a.stage_bytes - kStreamSlack) / 16;  // the streams' look-ahead stays inside
    const uint32_t *stage32 = reinterpret_cast<const uint32_t *>(stage);

    // Prologue: the decode tables (LDS-direct, the waves share them), the query and the Block Offsets Array entries are requested
    // together, so the workgroup starts after two trips to memory (entry, record).  The entries are loaded without a branch
    // and last: their wait is everyone's, and the barrier behind it, which is there for the tables and the query, waits for no
    // record.  Every wave then waits for its own: all records of a launch's first round are requested at once (23 MB for 32
    // heads x 32768 tokens), and the first ones arrive 2 us before the last.  (With more than 128 levels the tables are biased
    // behind that barrier, and the second barrier which that takes does wait for the records.)
    const int n_pairs = a.blocks_per_split;
    const bool is_v = kPaired && wave >= n_pairs;
    int j = j0 + wave;
    if (is_v) j = wave < 2 * n_pairs ? j - n_pairs : j1;  // the waves behind the pairs own no block
    const uint16_t *q0 = a.q + ((size_t)b * a.Hq + (size_t)h * G) * kD;
    uint4 qv[kTile ? G / 4 : 1];           // tile path: 8 query values each, of this thread and of thread + n_threads
    uint32_t qh[kTile ? 1 : G][2];         // else: q of channels lane and lane + 64
    if constexpr (kTile) {
#pragma unroll
        for (int k = 0; k < G / 4; k++)    // at least 64 threads for G * 16 pieces
            qv[k] = load_query(q0 + 8 * min(tid + k * n_threads, G * kD / 8 - 1));
    } else {
#pragma unroll
        for (int gg = 0; gg < G; gg++) { qh[gg][0] = q0[gg * kD + lane]; qh[gg][1] = q0[gg * kD + lane + 64]; }
    }
    auto stage_table = [&](const uint4 *src, int bytes, uint8_t *to) {
        for (int c = wave; 1024 * c < bytes; c += n_waves)
            if (1024 * c + 16 * lane < bytes) load_lds16(src + 64 * c + lane, to + 1024 * c);
    };
    constexpr int kTabOff = M::kPair ? kTabPairOff : kTabLutOff;
    stage_table(reinterpret_cast<const uint4 *>(a.tables + kTabOff), M::kTableBytes, &lut_s[0][0]);
    stage_table(reinterpret_cast<const uint4 *>(a.tables + kTensorTablesBytes + kTabOff), M::kTableBytes, &lut_s[1][0]);
    const uint32_t maskK = a.mask[0], maskV = a.mask[1];
    const int je = max(0, min(j, a.n_blocks - 1));  // an entry that exists for the waves that own no block, too
    BlockEntry eK = is_v ? tabV[je] : tabK[je], eV = kPaired ? eK : tabV[je];
    __builtin_amdgcn_s_waitcnt(0);
    eK.off16 = __builtin_amdgcn_readfirstlane(eK.off16);
    eK.size16 = __builtin_amdgcn_readfirstlane(eK.size16);
    const BlockEntry e0 = eK;
    if (j < j1 && e0.size16 <= stage16) stage_record(a.payload + (size_t)e0.off16 * 16, e0.size16, stage, lane);
    float qreg[kTile ? 1 : G][2];          // the tile path reads its q from LDS once per block
    if constexpr (kTile) {
#pragma unroll
        for (int k = 0; k < G / 4; k++) {
            const int i = tid + k * n_threads;
            float4 *dst = reinterpret_cast<float4 *>(qf + 8 * i);
            // An Inf in a query makes its head's output NaN, as any score with it is +-Inf or NaN; the maximum that scales the weights
            // of all heads passes over a NaN, and would leave the other heads no bits beside an Inf.
            auto value = [](uint32_t bits) { const float x = h2f(bits); return fmaf(x, 0.f, x); };
            if (i < G * kD / 8) {
                dst[0] = make_float4(value(qv[k].x & 0xffffu), value(qv[k].x >> 16), value(qv[k].y & 0xffffu), value(qv[k].y >> 16));
                dst[1] = make_float4(value(qv[k].z & 0xffffu), value(qv[k].z >> 16), value(qv[k].w & 0xffffu), value(qv[k].w >> 16));
            }
        }
        if (tid < kD / 4) reinterpret_cast<uint32_t *>(zeros)[tid] = 0;
    } else {
#pragma unroll
        for (int gg = 0; gg < G; gg++) { qreg[gg][0] = h2f(qh[gg][0]); qreg[gg][1] = h2f(qh[gg][1]); }
    }
    if constexpr (kPaired) {
        if (tid < 16) ready[tid] = 0;
    }
    // a fence would wait for the record on its way: only the LDS stores above have to be done (the tables are)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (kBiased<LB>) {
        if (a.bias[0] != 0.f || a.bias[1] != 0.f) {
            uint32_t *tk = reinterpret_cast<uint32_t *>(&lut_s[0][0]), *tv = reinterpret_cast<uint32_t *>(&lut_s[1][0]);
            if (a.bias[0] != 0.f)
                for (int i = tid; i < M::kTableBytes / 4; i += n_threads) tk[i] ^= 0x80008000u;
            if (a.bias[1] != 0.f)
                for (int i = tid; i < M::kTableBytes / 4; i += n_threads) tv[i] ^= 0x80008000u;
            __syncthreads();
        }
    }
    constexpr int kQ0 = kTile ? G / 2 : G;
    wait_record();
    wave_sync();

    Soft<G> st;
    st.init();
    TileSoft<kTile ? G : 2> ts;
    ts.init();

    if constexpr (kPaired) {
        const uint8_t *rec = a.payload + (size_t)e0.off16 * 16;
        const uint32_t *rec32 = reinterpret_cast<const uint32_t *>(rec);
        const bool staged = e0.size16 <= stage16;
        if (j < j1 && !is_v) {
            __builtin_amdgcn_s_setprio(3);  // its V wave waits for it
            float *box = reinterpret_cast<float *>(stage);
            if constexpr (kTile) {
                float p[kQ0][2];
                if (staged) {
                    k_tile_block<G, LB>(stage32, lutK, maskK, tile, zeros, qf, a.two_eb[0], a.bias[0], a.scale, lane,
                                        a.k_minmax_bytes, ts, p, [] {});
                } else {
                    TileSoft<G> ts_tmp = ts;  // copies keep the hot state in registers
                    float p_tmp[kQ0][2];
                    k_tile_block_global<G, LB>(rec32, lutK, maskK, tile, zeros, qf, a.two_eb[0], a.bias[0], a.scale, lane,
                                               a.k_minmax_bytes, ts_tmp, p_tmp);
                    ts = ts_tmp;
#pragma unroll
                    for (int i = 0; i < kQ0; i++) { p[i][0] = p_tmp[i][0]; p[i][1] = p_tmp[i][1]; }
                }
                wave_sync();
#pragma unroll
                for (int i = 0; i < kQ0; i++) {
                    box[(3 * i) * 64 + lane] = p[i][0];
                    box[(3 * i + 1) * 64 + lane] = p[i][1];
                    box[(3 * i + 2) * 64 + lane] = ts.m[i];
                }
            } else {
                float score[G];
                if (staged) {
                    k_block<G, LB>(stage32, lutK, maskK, qreg, a.two_eb[0], a.bias[0], a.scale, lane,
                                   a.k_minmax_bytes, score, [] {});
                } else {
                    float q_tmp[G][2], s_tmp[G];
#pragma unroll
                    for (int gg = 0; gg < G; gg++) { q_tmp[gg][0] = qreg[gg][0]; q_tmp[gg][1] = qreg[gg][1]; }
                    k_block_global<G, LB>(rec32, lutK, maskK, q_tmp, a.two_eb[0], a.bias[0], a.scale, lane,
                                          a.k_minmax_bytes, s_tmp);
#pragma unroll
                    for (int gg = 0; gg < G; gg++) score[gg] = s_tmp[gg];
                }
                wave_sync();
#pragma unroll
                for (int gg = 0; gg < G; gg++) {
                    box[2 * gg * 64 + lane] = st.update(gg, score[gg]);
                    box[(2 * gg + 1) * 64 + lane] = st.m[gg];
                }
            }
            if (lane == 0) __hip_atomic_store(&ready[wave], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else if (j < j1) {
            // The K wave of the pair is resident (a workgroup's waves start together) and sets its flag whatever its record
            // holds, so the wait ends.
            const int kw = wave - n_pairs;
            const float *box = reinterpret_cast<const float *>(smem + (size_t)kw * a.stage_bytes);
            auto wait_k = [&] {
                while (__hip_atomic_load(&ready[kw], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u)
                    __builtin_amdgcn_s_sleep(1);
            };
            if constexpr (kTile) {
                float p[kQ0][2];
                auto numerators = [&](float (&pp)[kQ0][2]) {
                    wait_k();
#pragma unroll
                    for (int i = 0; i < kQ0; i++) {
                        pp[i][0] = box[(3 * i) * 64 + lane];
                        pp[i][1] = box[(3 * i + 1) * 64 + lane];
                        ts.m[i] = box[(3 * i + 2) * 64 + lane];
                        ts.l[i] = pp[i][0] + pp[i][1];
                    }
                };
                if (staged) {
                    v_tile_block<G, LB, true>(stage32, lutV, maskV, tile, zeros, p, a.two_eb[1], a.bias[1], lane, ts, [] {}, numerators);
                } else {
                    numerators(p);
                    TileSoft<G> ts_tmp = ts;
                    float p_tmp[kQ0][2];
#pragma unroll
                    for (int i = 0; i < kQ0; i++) { p_tmp[i][0] = p[i][0]; p_tmp[i][1] = p[i][1]; }
                    v_tile_block_global<G, LB>(rec32, lutV, maskV, tile, zeros, p_tmp, a.two_eb[1], a.bias[1], lane, ts_tmp);
                    ts = ts_tmp;
                }
            } else {
                float p[G];
                auto numerators = [&](float (&pp)[G]) {
                    wait_k();
#pragma unroll
                    for (int gg = 0; gg < G; gg++) {
                        pp[gg] = box[2 * gg * 64 + lane];
                        st.m[gg] = box[(2 * gg + 1) * 64 + lane];
                        st.l[gg] = pp[gg];
                    }
                };
                if (staged) {
                    v_block<G, LB, true>(stage32, lutV, maskV, p, a.two_eb[1], a.bias[1], lane, st, [] {}, numerators);
                } else {
                    numerators(p);
                    Soft<G> st_tmp = st;
                    float p_tmp[G];
#pragma unroll
                    for (int gg = 0; gg < G; gg++) p_tmp[gg] = p[gg];
                    v_block_global<G, LB>(rec32, lutV, maskV, p_tmp, a.two_eb[1], a.bias[1], lane, st_tmp);
                    st = st_tmp;
                }
            }
        }
    } else {
    const auto no_numerators = [](auto &) {};
    const int total = j < j1 ? (int)a.by_waves((uint32_t)(j1 - j + n_waves - 1)) : 0;  // this wave's block pairs
    int left = total;
    __builtin_amdgcn_s_setprio(3);
    while (j < j1) {
        float score[G], p[G];
        const bool k_staged = eK.size16 <= stage16, v_staged = eV.size16 <= stage16;
        const uint8_t *recK = a.payload + (size_t)eK.off16 * 16, *recV = a.payload + (size_t)eV.off16 * 16;
        const int jn = j + n_waves;  // the next pair's Block Offsets Array entries travel with it
        BlockEntry eKn = {0, 0}, eVn = {0, 0};
        if (jn < j1) {
            eKn = tabK[jn];
            eVn = tabV[jn];
        }
        float pt[kQ0][2];  // tile path: softmax numerators in the layout of the result tiles
        // The next record is requested when the current one has been decoded: the staging area is free then, and its
        // loads travel behind the last products and the softmax.
        auto next_v = [&] { if (v_staged) stage_record(recV, eV.size16, stage, lane); };
        if constexpr (kTile) {
            if (k_staged) {
                k_tile_block<G, LB>(stage32, lutK, maskK, tile, zeros, qf, a.two_eb[0], a.bias[0], a.scale, lane, a.k_minmax_bytes,
                                     ts, pt, next_v);
            } else {
                TileSoft<G> ts_tmp = ts;
                float p_tmp[kQ0][2];
                k_tile_block_global<G, LB>(reinterpret_cast<const uint32_t *>(recK), lutK, maskK, tile, zeros, qf, a.two_eb[0],
                                            a.bias[0], a.scale, lane, a.k_minmax_bytes, ts_tmp, p_tmp);
                ts = ts_tmp;
#pragma unroll
                for (int i = 0; i < kQ0; i++) { pt[i][0] = p_tmp[i][0]; pt[i][1] = p_tmp[i][1]; }
                next_v();
            }
        } else {
        if (k_staged) {
            k_block<G, LB>(stage32, lutK, maskK, qreg, a.two_eb[0], a.bias[0], a.scale, lane, a.k_minmax_bytes, score, next_v);
        } else {  // larger than the staging area: decode from global memory (copies keep the hot state in registers)
            float q_tmp[G][2], s_tmp[G];
#pragma unroll
            for (int gg = 0; gg < G; gg++) { q_tmp[gg][0] = qreg[gg][0]; q_tmp[gg][1] = qreg[gg][1]; }
            k_block_global<G, LB>(reinterpret_cast<const uint32_t *>(recK), lutK, maskK, q_tmp, a.two_eb[0],
                                  a.bias[0], a.scale, lane, a.k_minmax_bytes, s_tmp);
#pragma unroll
            for (int gg = 0; gg < G; gg++) score[gg] = s_tmp[gg];
            next_v();
        }
        }
        if constexpr (!kTile) {
#pragma unroll
            for (int gg = 0; gg < G; gg++) p[gg] = st.update(gg, score[gg]);
        }
        wave_sync();  // every lane is done with the K record
        if (v_staged) wait_record();
        wave_sync();
        eKn.off16 = __builtin_amdgcn_readfirstlane(eKn.off16);
        eKn.size16 = __builtin_amdgcn_readfirstlane(eKn.size16);
        eVn.off16 = __builtin_amdgcn_readfirstlane(eVn.off16);
        eVn.size16 = __builtin_amdgcn_readfirstlane(eVn.size16);
        const bool next_staged = jn < j1 && eKn.size16 <= stage16;
        auto next_k = [&] { if (next_staged) stage_record(a.payload + (size_t)eKn.off16 * 16, eKn.size16, stage, lane); };
        if constexpr (kTile) {
            if (v_staged) {
                v_tile_block<G, LB, false>(stage32, lutV, maskV, tile, zeros, pt, a.two_eb[1], a.bias[1], lane, ts, next_k, no_numerators);
            } else {
                TileSoft<G> ts_tmp = ts;
                float p_tmp[kQ0][2];
#pragma unroll
                for (int i = 0; i < kQ0; i++) { p_tmp[i][0] = pt[i][0]; p_tmp[i][1] = pt[i][1]; }
                v_tile_block_global<G, LB>(reinterpret_cast<const uint32_t *>(recV), lutV, maskV, tile, zeros, p_tmp, a.two_eb[1],
                                            a.bias[1], lane, ts_tmp);
                ts = ts_tmp;
                next_k();
            }
        } else {
        if (v_staged) {
            v_block<G, LB, false>(stage32, lutV, maskV, p, a.two_eb[1], a.bias[1], lane, st, next_k, no_numerators);
        } else {
            Soft<G> st_tmp = st;
            float p_tmp[G];
#pragma unroll
            for (int gg = 0; gg < G; gg++) p_tmp[gg] = p[gg];
            v_block_global<G, LB>(reinterpret_cast<const uint32_t *>(recV), lutV, maskV, p_tmp, a.two_eb[1],
                                  a.bias[1], lane, st_tmp);
            st = st_tmp;
            next_k();
        }
        }
        wave_sync();
        if (next_staged) wait_record();
        wave_sync();
        eK = eKn;
        eV = eVn;
        j = jn;
        {   // The SIMD issues from its oldest wave first, so its resident waves finish one after the other and the
            // last one runs alone, unable to fill the VALU.  Waves that are behind get the issue slots instead:
            // the priority falls with the share of the work that is done, and the waves finish together.
            const int left4 = 4 * --left;
            if (left4 > 3 * total) __builtin_amdgcn_s_setprio(3);
            else if (left4 > 2 * total) __builtin_amdgcn_s_setprio(2);
            else if (left4 > total) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
    }
    }

    // The record area is free now: the wave's state is parked there, and the buffered tokens join it.
    if (!kPaired || is_v) {  // a K wave of a pair has no state, and its area may still be read
        float *area = reinterpret_cast<float *>(stage);
        if constexpr (kTile) soft_to_area<G>(ts, area, merge_ml, wave, lane);
        else soft_to_area<G>(st, area, merge_ml, wave, lane);
        // the buffered fp16 tokens in units of 16: unit u goes to split n_splits-1 - u % n_splits (the last split is the
        // short one), there to the waves in turn, starting after the wave that took the split's last block
        if (a.n_res > 0) {
            // 0 for the wave whose turn the next block would be; paired: for the first wave behind the pairs
            const int turn = kPaired ? wave - 2 * n_pairs : j - j1, takers = kPaired ? n_waves - 2 * n_pairs : n_waves;
            const int first = a.n_splits - 1 - split + a.n_splits * turn;
            if (turn >= 0 && first * kUnitTokens < a.n_res) {
                const int step = takers * a.n_splits;
                if constexpr (DecodeMode<LB>::kPair || !kPaired)
                    buffered_units<G>(a.res, a.res_tokens, a.B, a.H, b, h, a.res_head, a.n_res, first, step, q0, a.scale, lane,
                                      a.k_new, a.v_new, a.new_row, area, merge_ml, wave);
                else
                    buffered_tokens<G>(a.res, a.res_tokens, a.B, a.H, b, h, a.res_head, a.n_res, first, step, q0, a.scale, lane,
                                       a.k_new, a.v_new, a.new_row, area, merge_ml, wave);
            }
        }
    }
    __syncthreads();
    // Merge the waves of this workgroup into one partial (o[128], m, l) per query head, a wave per head: lane w holds wave w's
    // m, l and bv, so the weights are there after one reduction; then every lane adds up two channels.  A thread per channel
    // that read every wave's m, l and o and kept a running maximum, with the states turned into another layout before, took
    // 1.8 us for groups of 8 and 12 waves.
    const int row0 = b * a.Hq + h * G;
    // the thread number is rebuilt from the lane and the (scalar) wave number: nothing of the prologue has to stay
    // in a register, or be spilled, across the decode loop for the sake of the merge
    const int tid_m = lane + 64 * wave, nt_m = 64 * n_waves;
    for (int gg = wave; gg < G; gg += n_waves) {
        const int w0 = kPaired ? n_pairs : 0;
        float2 o[4];
        auto request = [&](int w) {  // the LDS reads of four waves' states at a time
#pragma unroll
            for (int k = 0; k < 4; k++)
                o[k] = reinterpret_cast<const float2 *>(smem + (size_t)min(w + k, n_waves - 1) * a.stage_bytes)[gg * (kD / 2) + lane];
        };
        request(w0);  // travels behind the weights
        float mw = -INFINITY, lw = 0.f, bw = 0.f;
        if (lane >= w0 && lane < n_waves) {
            mw = *merge_word<G>(merge_ml, 0, gg, lane);
            lw = *merge_word<G>(merge_ml, 1, gg, lane);
            bw = *merge_word<G>(merge_ml, 2, gg, lane);
        }
        const float M_ = wave_max(mw);
        const uint32_t live = (uint32_t)__builtin_amdgcn_ballot_w64(mw != -INFINITY);  // the others had nothing to do
        const float f = mw == -INFINITY ? 0.f : __expf(mw - M_);
        const float L = wave_sum(mw == -INFINITY ? 0.f : lw * f);
        float O0 = 0.f, O1 = 0.f;
        for (int w = w0; w < n_waves; w += 4) {
            if (w > w0) request(w);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if (!((live >> (w + k)) & 1u)) continue;  // uniform; no lane beyond the last wave is live
                // o and bv nearly cancel (min + step * code): their sum is formed before anything else is added
                const float fw = bcast(f, w + k), bv = bcast(bw, w + k);
                O0 = fmaf(fw, o[k].x + bv, O0);
                O1 = fmaf(fw, o[k].y + bv, O1);
            }
        }
        if (a.n_splits == 1) {
            a.out[(size_t)(row0 + gg) * kD + 2 * lane] = O0 / L;
            a.out[(size_t)(row0 + gg) * kD + 2 * lane + 1] = O1 / L;
        } else {
            float *dst = a.partials + ((size_t)(row0 + gg) * kMaxSplits + split) * kPartialStride;
            store_agent(dst + 2 * lane, O0);
            store_agent(dst + 2 * lane + 1, O1);
            if (lane == 0) { store_agent(dst + kD, M_); store_agent(dst + kD + 1, L); }
        }
    }
    if (a.n_splits > 1) finish_splits<G, true>(a.partials, a.counters + bh, row0, a.n_splits, a.out, tid_m, nt_m,
                                               reinterpret_cast<float *>(smem));
}

template <int G, int LB, bool kPaired>
static hipError_t launch_fused_gn(const FusedArgs &a, int n_waves, size_t lds, hipEvent_t ev0, hipEvent_t ev1,
                                  hipStream_t s) {
    static size_t attr_set = 0;
    if (lds > attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&fused_attn_kernel<G, LB, kPaired>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = lds;
    }
    if (n_waves < 1 || n_waves > MaxWaves<G, LB, kPaired>::value) return hipErrorInvalidValue;
    if (ev0) (void)hipEventRecord(ev0, s);
    hipLaunchKernelGGL((fused_attn_kernel<G, LB, kPaired>), dim3(a.n_splits * a.n_bh), dim3(64 * n_waves), lds, s, a);
    if (ev1) (void)hipEventRecord(ev1, s);
    return hipGetLastError();
}

template <int G, bool kPaired>
static hipError_t launch_fused_g(const FusedArgs &a, int longest, int n_waves, size_t lds, hipEvent_t ev0, hipEvent_t ev1,
                                 hipStream_t s) {
    switch (fused_table_bits(longest)) {
        case 6: return launch_fused_gn<G, 6, kPaired>(a, n_waves, lds, ev0, ev1, s);
        case 7: return launch_fused_gn<G, 7, kPaired>(a, n_waves, lds, ev0, ev1, s);
        case 8: return launch_fused_gn<G, 8, kPaired>(a, n_waves, lds, ev0, ev1, s);
        case 10: return launch_fused_gn<G, 10, kPaired>(a, n_waves, lds, ev0, ev1, s);
        default: return launch_fused_gn<G, 12, kPaired>(a, n_waves, lds, ev0, ev1, s);
    }
}

hipError_t launch_fused_attn(const Geo &g, const uint16_t *q, float scale, float *out, int n_blocks, int res_head,
                             int n_res, const uint16_t *k_new, const uint16_t *v_new, int n_splits, int n_waves,
                             bool paired, int stage_bytes, hipEvent_t ev0, hipEvent_t ev1, hipStream_t s) {
    FusedArgs a;
    a.k_new = k_new;
    a.v_new = v_new;
    a.new_row = k_new ? n_res - 1 : -1;  // n_res counts the token being appended
    a.table = g.table;
    a.tables = g.tables;
    a.payload = g.payload;
    a.partials = g.partials;
    a.counters = g.counters;
    a.res = g.res;
    a.res_tokens = g.res_tokens;
    a.B = g.B;
    a.H = g.H;
    a.Hq = g.Hq;
    a.n_bh = g.B * g.H;
    a.max_blocks = g.max_blocks;
    a.k_minmax_bytes = g.k_minmax_bytes;
    a.q = q;
    a.out = out;
    a.scale = scale;
    a.n_blocks = n_blocks;
    a.res_head = res_head;
    a.n_res = n_res;
    a.blocks_per_split = n_blocks > 0 ? (n_blocks + n_splits - 1) / n_splits : 0;
    a.n_splits = n_blocks > 0 ? (n_blocks + a.blocks_per_split - 1) / a.blocks_per_split : 1;
    a.stage_bytes = stage_bytes;
    a.by_splits.set((uint32_t)a.n_splits);
    a.by_heads.set((uint32_t)g.H);
    a.by_waves.set((uint32_t)n_waves);
    for (int t = 0; t < 2; t++) a.two_eb[t] = g.two_eb[t];
    for (int t = 0; t < 2; t++) a.bias[t] = g.n_sym[t] > 128 ? 128.f : 0.f;
    const int bits_k = g.lut_bits[0], bits_v = g.lut_bits[1];
    const int longest = bits_k > bits_v ? bits_k : bits_v;
    if (longest < 1 || longest > kLutBits) return hipErrorInvalidValue;
    if (fused_table_bits(longest) == 6) {  // pair tables: 12 index bits, entries of 4 bytes
        a.mask[0] = a.mask[1] = ((1u << kPairIndexBits) - 1u) << 2;
    } else {
        a.mask[0] = ((1u << bits_k) - 1u) << 1;
        a.mask[1] = ((1u << bits_v) - 1u) << 1;
    }
    const size_t lds = (size_t)n_waves * ((size_t)stage_bytes + fused_weight_bytes(g.G));
    if (paired && (2 * a.blocks_per_split + (n_res > 0) > n_waves || n_waves > 16)) return hipErrorInvalidValue;
    auto launch = [&](auto gc) {
        constexpr int G = decltype(gc)::value;
        return paired ? launch_fused_g<G, true>(a, longest, n_waves, lds, ev0, ev1, s)
                      : launch_fused_g<G, false>(a, longest, n_waves, lds, ev0, ev1, s);
    };
    switch (g.G) {
        case 1: return launch(std::integral_constant<int, 1>());
        case 2: return launch(std::integral_constant<int, 2>());
        case 4: return launch(std::integral_constant<int, 4>());
        case 8: return launch(std::integral_constant<int, 8>());
        default: return hipErrorInvalidValue;
    }
}

// ---- statistics (metrics path, not part of the hot loop) --------------------------------------------------------
// Sums record sizes and code-word bits over all blocks in use by walking the Block Offsets Array and the slice bit
// counts in the record headers.
__global__ __launch_bounds__(256) void stats_kernel(Geo g, int n_blocks) {
    const int BH = g.B * g.H;
    const long long n_items = 2ll * BH * n_blocks;
    unsigned long long bits[2] = {0, 0}, rec16[2] = {0, 0};
    const int lane = threadIdx.x & 63;
    const long long wave_id = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long long n_waves = ((long long)gridDim.x * blockDim.x) >> 6;
    for (long long i = wave_id; i < n_items; i += n_waves) {
        const int which = (int)(i / ((long long)BH * n_blocks));
        const long long rem = i - (long long)which * BH * n_blocks;
        const int bh = (int)(rem / n_blocks), j = (int)(rem - (long long)bh * n_blocks);
        const BlockEntry e = g.table[((size_t)which * BH + bh) * g.max_blocks + j];
        const uint16_t *sb = reinterpret_cast<const uint16_t *>(g.payload + (size_t)e.off16 * 16 +
                                                                (which ? kMinMaxBytesV : g.k_minmax_bytes));
        const uint32_t v = (uint32_t)sb[lane] + sb[lane + 64];
        bits[which] += v;
        if (lane == 0) rec16[which] += e.size16;
    }
    for (int w = 0; w < 2; w++) {
        unsigned long long bsum = bits[w], rsum = rec16[w];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            bsum += __shfl_xor(bsum, m);
            rsum += __shfl_xor(rsum, m);
        }
        if (lane == 0 && (bsum | rsum)) {
            atomicAdd(&g.ctrl->payload_bits[w], bsum);
            atomicAdd(&g.ctrl->record16[w], rsum);
        }
    }
}

hipError_t launch_stats(const Geo &g, int n_blocks, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(stats_kernel, dim3(128), dim3(256), 0, s, g, n_blocks);
    return hipGetLastError();
}

}  // namespace kvc
