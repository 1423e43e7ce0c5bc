// The uncompressed comparison kernel (Section 4.3 compares the fused kernel with a plain fp16 matrix-vector
// product): decode attention on the fp16 cache [B, S, H, 128], sequence split over workgroups with an online
// softmax, merged inside the kernel like the fused path.  HBM-bound: every K and V byte is read once with 16-byte
// loads.  Groups of 1 and 2 query heads run on the vector ALU; groups of 4 and 8 (one K and one V row serve several heads:
// two small matrix products) on the matrix cores.
#include <hip/hip_fp16.h>

#include <mutex>

#include "huff_decode.cuh"
#include "kvcomp_internal.h"
#include "split_combine.cuh"

namespace kvc {

__device__ __forceinline__ float bh2f(uint32_t bits) { return __half2float(__ushort_as_half((unsigned short)bits)); }

__device__ __forceinline__ void unpack8(const uint4 &v, float (&x)[8]) {
    x[0] = bh2f(v.x & 0xffffu); x[1] = bh2f(v.x >> 16);
    x[2] = bh2f(v.y & 0xffffu); x[3] = bh2f(v.y >> 16);
    x[4] = bh2f(v.z & 0xffffu); x[5] = bh2f(v.z >> 16);
    x[6] = bh2f(v.w & 0xffffu); x[7] = bh2f(v.w >> 16);
}

constexpr int kBWaves = 4;

// The waves of a workgroup have left (o[128], m, l) per query head in comb: merge them into the workgroup's partial
// and, in the last workgroup of the (batch, kv head), the splits into the output.
template <int G>
__device__ __forceinline__ void merge_waves_and_splits(float (&comb)[kBWaves][G][kPartialStride],
                                                       float *__restrict__ partials, uint32_t *__restrict__ counters,
                                                       float *__restrict__ out, int b, int h, int Hq, int split, int bh,
                                                       int tid, int split_stride) {
    for (int i = tid; i < G * kD; i += 64 * kBWaves) {
        const int g = i / kD, c = i - g * kD;
        float M = -INFINITY;
        for (int w = 0; w < kBWaves; w++) M = fmaxf(M, comb[w][g][kD]);
        float L = 0.f, O = 0.f;
        for (int w = 0; w < kBWaves; w++) {
            const float mw = comb[w][g][kD];
            const float f = mw == -INFINITY ? 0.f : __expf(mw - M);
            L += comb[w][g][kD + 1] * f;
            O += comb[w][g][c] * f;
        }
        if (gridDim.x == 1) {
            out[((size_t)b * Hq + (size_t)h * G + g) * kD + c] = O / L;
        } else {
            float *dst = partials + (((size_t)b * Hq + (size_t)h * G + g) * split_stride + split) * kPartialStride;
            store_agent(dst + c, O);
            if (c == 0) { store_agent(dst + kD, M); store_agent(dst + kD + 1, L); }
        }
    }
    if (gridDim.x > 1)
        finish_splits<G, false>(partials, counters + bh, b * Hq + h * G, (int)gridDim.x, out, tid, 64 * kBWaves, &comb[0][0][0],
                         split_stride);
}


// Lane l of a wave owns channels 8*(l%16)..+7 and the tokens 4*i + l/16 (i = 0..15) of a 64-token tile: one load
// instruction of the wave reads four whole 256-byte rows.  The loop is software-pipelined: the K rows of the next
// tile are requested as soon as the scores of the current one are formed, behind the current tile's V rows, so that
// a wave always has 16 KiB (and most of the time 32 KiB) on its way from memory; the 16-lane dot-product sums run on
// DPP row operations, not on LDS permutes.
template <int G>
__global__ __launch_bounds__(64 * kBWaves, 2) void baseline_attn_kernel(int B, int H, int Hq, const uint16_t *__restrict__ K,
                                                                         const uint16_t *__restrict__ V, int seq,
                                                                         const uint16_t *__restrict__ q, float scale,
                                                                         float *__restrict__ partials,
                                                                         uint32_t *__restrict__ counters,
                                                                         float *__restrict__ out, int tokens_per_split, int split_stride) {
    __shared__ float comb[kBWaves][G][kPartialStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int split = blockIdx.x, bh = blockIdx.y, b = bh / H, h = bh - b * H;
    const int cc = (lane & 15) * 8, sub = lane >> 4;
    float qr[G][8];
#pragma unroll
    for (int g = 0; g < G; g++) {
        const uint4 v = *reinterpret_cast<const uint4 *>(q + ((size_t)b * Hq + (size_t)h * G + g) * kD + cc);
        unpack8(v, qr[g]);
    }
    float m[G], lsum[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; g++) {
        m[g] = -INFINITY;
        lsum[g] = 0.f;
#pragma unroll
        for (int k = 0; k < 8; k++) acc[g][k] = 0.f;
    }
    const int t_begin = split * tokens_per_split;
    const int t_end = min(t_begin + tokens_per_split, seq);
    const size_t row = (size_t)H * kD;  // elements between consecutive tokens
    const uint16_t *Kb = K + ((size_t)b * seq * H + h) * kD + cc;
    const uint16_t *Vb = V + ((size_t)b * seq * H + h) * kD + cc;

    uint4 kv[16];
    auto load_k = [&](int t0) {
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int t = t0 + 4 * i + sub;
            kv[i] = t < t_end ? *reinterpret_cast<const uint4 *>(Kb + (size_t)t * row) : make_uint4(0, 0, 0, 0);
        }
    };
    int t0 = t_begin + wave * 64;
    if (t0 < t_end) load_k(t0);
    for (; t0 < t_end; t0 += 64 * kBWaves) {
        float s[G][16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            float x[8];
            unpack8(kv[i], x);
            const bool valid = t0 + 4 * i + sub < t_end;
#pragma unroll
            for (int g = 0; g < G; g++) {
                float d = 0.f;
#pragma unroll
                for (int k = 0; k < 8; k++) d = fmaf(qr[g][k], x[k], d);
                d += dpp_f<kDppXor1>(d);
                d += dpp_f<kDppXor2>(d);
                d += dpp_f<kDppHalfMirror>(d);
                d += dpp_f<kDppMirror>(d);  // the row's 16 lanes all hold its dot product
                s[g][i] = valid ? scale * d : -INFINITY;
            }
        }
        uint4 vv[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int t = t0 + 4 * i + sub;
            vv[i] = t < t_end ? *reinterpret_cast<const uint4 *>(Vb + (size_t)t * row) : make_uint4(0, 0, 0, 0);
        }
        if (t0 + 64 * kBWaves < t_end) load_k(t0 + 64 * kBWaves);  // behind the V rows: they are waited for first
        float p[G][16];
#pragma unroll
        for (int g = 0; g < G; g++) {
            float ml = s[g][0];
#pragma unroll
            for (int i = 1; i < 16; i++) ml = fmaxf(ml, s[g][i]);
            ml = fmaxf(ml, __shfl_xor(ml, 16));
            ml = fmaxf(ml, __shfl_xor(ml, 32));
            const float mnew = fmaxf(fmaxf(m[g], ml), kLowestRef);
            const float alpha = __expf(m[g] - mnew);
            m[g] = mnew;
            float ps = 0.f;
#pragma unroll
            for (int i = 0; i < 16; i++) {
                p[g][i] = __expf(s[g][i] - mnew);
                ps += p[g][i];
            }
            lsum[g] = lsum[g] * alpha + ps;
#pragma unroll
            for (int k = 0; k < 8; k++) acc[g][k] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < 16; i++) {
            float x[8];
            unpack8(vv[i], x);
#pragma unroll
            for (int g = 0; g < G; g++)
#pragma unroll
                for (int k = 0; k < 8; k++) acc[g][k] = fmaf(p[g][i], x[k], acc[g][k]);
        }
    }
    // reduce the four token sub-groups of the wave, then the waves of the workgroup
#pragma unroll
    for (int g = 0; g < G; g++) {
        lsum[g] += __shfl_xor(lsum[g], 16);
        lsum[g] += __shfl_xor(lsum[g], 32);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            acc[g][k] += __shfl_xor(acc[g][k], 16);
            acc[g][k] += __shfl_xor(acc[g][k], 32);
        }
        if (sub == 0) {
#pragma unroll
            for (int k = 0; k < 8; k++) comb[wave][g][cc + k] = acc[g][k];
        }
        if (lane == 0) {
            comb[wave][g][kD] = m[g];
            comb[wave][g][kD + 1] = lsum[g];
        }
    }
    __syncthreads();
    merge_waves_and_splits<G>(comb, partials, counters, out, b, h, Hq, split, bh, tid, split_stride);
}

// ---- groups of 4 and 8 query heads --------------------------------------------------------------------------------
// Both products run on v_mfma_f32_16x16x32_f16 with every operand straight from the registers it was loaded or computed in:
//   A: lane l holds row l % 16, eight reduction slots of slot group l / 16;  B: column l % 16, the same slots;
//   D: lane l holds column l % 16, rows 4 (l / 16) .. + 3.
// Which index a slot stands for is free as long as A and B agree.
//   scores: S^T = K Q^T, rows = 16 tokens, columns = query heads (repeated: column j is head j % G).  Step i maps slot
//           (l / 16, r) to channel 8 (l / 16 + 4 i) + r: a lane's operand is one 16-byte load of its K row.
//   p . V : O = P V, rows = heads, 32 tokens at a time.  A lane's eight scores of two tiles, tokens 16 tt + 4 (l / 16) + r,
//           are the eight slots of its group, so the numerators are the A operand without leaving the lane.  V is loaded for
//           those tokens, 8 channels of one token per load; the 8 x 8 halves of a lane are transposed in its registers (one
//           v_perm_b32 per pair) into one B operand per channel: column l % 16 of tile ct is channel 8 (l % 16) + ct.
//   A numerator is a fp32 number, an fp16 operand holds eleven bits of it above 2^-14 and fewer below: it goes in as four
//   parts, each what the ones before left of it times 2^11 (truncated, so that the rest is exact and positive).  Three parts
//   hold fp32's 24 bits of a numerator near 1, four hold them down to 2^-34.  The parts are the A rows G apart (the copies of
//   the score columns are there for that) and are added at the end; groups of 8 have rows for two, and the other two take
//   a second product per operand.  With two parts only, a numerator of e^-14 had 16 bits and one of e^-24 none.
// The loop keeps a tile of 64 V rows and the next tile of K rows on their way (16 to 32 KiB a wave; registers for two waves
// per SIMD, the host starts one unless there are more heads than CUs).
// With p . V on the vector ALU, 8 FMAs per value for groups of 8, and the numerators through LDS, it was bound by the ALU:
// 8 x 8 heads x 16384 tokens, groups of 8: 121 us (4.4 TB/s) -> 104 us (5.2 TB/s; a plain read reaches 6.0); groups of 4,
// 16 x 8 heads x 8192: 103 -> 99 us.  Four parts instead of two cost nothing there (107.6 and 107.5 us in one run).
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr float kNextPart = 2048.f;    // scale of a numerator's part against the one before it
constexpr float kLazyMaxFp16 = 8.f;    // how far a score may exceed the softmax reference before the state is rescaled

// v + f * (v of the lane DIST further), valid in the lanes of the lower half (DIST 32) or of the even rows of 16 (DIST 16)
template <int DIST>
__device__ __forceinline__ float add_next(float v, float f) {
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    const uint32_t u = __float_as_uint(v);
    const v2u r = DIST == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaf(__uint_as_float(r.y), f, __uint_as_float(r.x));
}

template <int G>
__global__ __launch_bounds__(64 * kBWaves, 2) void baseline_attn_gqa_kernel(
    int B, int H, int Hq, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V, int seq,
    const uint16_t *__restrict__ q, float scale, float *__restrict__ partials, uint32_t *__restrict__ counters,
    float *__restrict__ out, int tokens_per_split, int split_stride) {
    static_assert(G == 4 || G == 8, "group size");
    __shared__ float comb[kBWaves][G][kPartialStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int split = blockIdx.x, bh = blockIdx.y, b = bh / H, h = bh - b * H;
    const int j = lane & 15, gq = lane >> 4, part = j / G;
    v8h qb[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
        qb[i] = *reinterpret_cast<const v8h *>(q + ((size_t)b * Hq + (size_t)h * G + j % G) * kD + 8 * (gq + 4 * i));
    float m = -INFINITY, lsum = 0.f;  // reference and sum of head j % G (this lane's tokens)
    v4f acc[8];                       // channel 8 j + ct of rows 4 gq .. + 3
#pragma unroll
    for (int ct = 0; ct < 8; ct++) acc[ct] = v4f{0.f, 0.f, 0.f, 0.f};
    const int t_begin = split * tokens_per_split;
    const int t_end = min(t_begin + tokens_per_split, seq);
    const size_t row = (size_t)H * kD;
    const uint16_t *Kb = K + ((size_t)b * seq * H + h) * kD + 8 * gq;
    const uint16_t *Vb = V + ((size_t)b * seq * H + h) * kD + 8 * j;

    uint4 kv[16], vv[16];
    auto load_k16 = [&](int t16, uint4 (&k4)[4]) {  // 16 tokens
        const int t = t16 + j;
#pragma unroll
        for (int i = 0; i < 4; i++)
            k4[i] = t < t_end ? *reinterpret_cast<const uint4 *>(Kb + (size_t)t * row + 32 * i) : make_uint4(0, 0, 0, 0);
    };
    auto load_k = [&](int t0) {
#pragma unroll
        for (int tt = 0; tt < 4; tt++) {
            uint4 k4[4];
            load_k16(t0 + 16 * tt, k4);
#pragma unroll
            for (int i = 0; i < 4; i++) kv[tt * 4 + i] = k4[i];
        }
    };
    auto scores = [&](const uint4 (&k4)[4]) {
        v4f d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; i++)
            d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, k4[i]), qb[i], d, 0, 0, 0);
        return d;
    };
    auto load_v = [&](int t0) {
#pragma unroll
        for (int tt = 0; tt < 4; tt++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int t = t0 + 16 * tt + 4 * gq + r;
                vv[tt * 4 + r] = t < t_end ? *reinterpret_cast<const uint4 *>(Vb + (size_t)t * row) : make_uint4(0, 0, 0, 0);
            }
    };
    int t0 = t_begin + wave * 64;
    if (t0 < t_end) load_k(t0);
    for (; t0 < t_end; t0 += 64 * kBWaves) {
        load_v(t0);
        float s[16], ml = kLowestRef;
#pragma unroll
        for (int tt = 0; tt < 4; tt++) {
            const uint4 k4[4] = {kv[tt * 4], kv[tt * 4 + 1], kv[tt * 4 + 2], kv[tt * 4 + 3]};
            const v4f d = scores(k4);
#pragma unroll
            for (int r = 0; r < 4; r++) s[tt * 4 + r] = scale * d[r];  // token t0 + 16 tt + 4 gq + r
        }
        if (t0 + 64 * kBWaves < t_end) load_k(t0 + 64 * kBWaves);
        if (t0 + 64 > t_end) {  // the last tile of the split
#pragma unroll
            for (int n = 0; n < 16; n++)
                if (t0 + 16 * (n >> 2) + 4 * gq + (n & 3) >= t_end) s[n] = -INFINITY;
        }
#pragma unroll
        for (int n = 0; n < 16; n++) ml = fmaxf(ml, s[n]);
        // The reference moves only when some score exceeds it by more than kLazyMaxFp16 (it is -inf at first: always then).
        if (__builtin_amdgcn_ballot_w64(ml - m > kLazyMaxFp16) != 0) {
            ml = fmaxf(ml, __shfl_xor(ml, 16));
            ml = fmaxf(ml, __shfl_xor(ml, 32));
            const float mnew = fmaxf(m, ml);  // not -inf
            const float alpha = __expf(m - mnew);
            m = mnew;
            lsum *= alpha;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const float ar = __shfl(alpha, 4 * gq + r);  // of row 4 gq + r, head (4 gq + r) % G
#pragma unroll
                for (int ct = 0; ct < 8; ct++) acc[ct][r] *= ar;
            }
        }
        float ps = 0.f;
#pragma unroll
        for (int n = 0; n < 16; n++) {
            s[n] = __expf(s[n] - m);
            ps += s[n];
        }
        lsum += ps;
        union { v8h v; uint32_t w[4]; } pa[2], pb[2];  // tokens 0..31 and 32..63 of the tile; pb: groups of 8
#pragma unroll
        for (int k = 0; k < 8; k++) {
            float p0 = s[2 * k], p1 = s[2 * k + 1];
            uint32_t w[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const v2h h = __builtin_bit_cast(v2h, __builtin_amdgcn_cvt_pkrtz(p0, p1));
                w[i] = __builtin_bit_cast(uint32_t, h);
                p0 = fmaf((float)h[0], -kNextPart, p0 * kNextPart);  // exact
                p1 = fmaf((float)h[1], -kNextPart, p1 * kNextPart);
            }
            if constexpr (G == 8) {
                pa[k >> 2].w[k & 3] = part == 0 ? w[0] : w[1];
                pb[k >> 2].w[k & 3] = part == 0 ? w[2] : w[3];
            } else {
                pa[k >> 2].w[k & 3] = part == 0 ? w[0] : part == 1 ? w[1] : part == 2 ? w[2] : w[3];
            }
        }
#pragma unroll
        for (int ct = 0; ct < 8; ct++) {
            v4f low = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int hh = 0; hh < 2; hh++) {
                union { v8h v; uint32_t w[4]; } vb;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const uint4 &r0 = vv[8 * hh + 2 * k], &r1 = vv[8 * hh + 2 * k + 1];
                    const uint32_t a = ct < 2 ? r0.x : ct < 4 ? r0.y : ct < 6 ? r0.z : r0.w;
                    const uint32_t c = ct < 2 ? r1.x : ct < 4 ? r1.y : ct < 6 ? r1.z : r1.w;
                    vb.w[k] = __builtin_amdgcn_perm(c, a, (ct & 1) ? 0x07060302u : 0x05040100u);
                }
                acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(pa[hh].v, vb.v, acc[ct], 0, 0, 0);
                if constexpr (G == 8) low = __builtin_amdgcn_mfma_f32_16x16x32_f16(pb[hh].v, vb.v, low, 0, 0, 0);
            }
            if constexpr (G == 8) {
#pragma unroll
                for (int r = 0; r < 4; r++) acc[ct][r] = fmaf(low[r], 1.f / (kNextPart * kNextPart), acc[ct][r]);
            }
        }
    }
    // An Inf in V times a numerator is Inf, but times the numerator's parts it is NaN wherever one of them is zero (or
    // Inf - Inf where they differ in sign).  No finite V overflows the sums, so a sum that is not finite sends the wave over
    // its tokens once more, with p . V in fp32 on the vector ALU against the final reference.
    v4f all = acc[0];
#pragma unroll
    for (int ct = 1; ct < 8; ct++) all += acc[ct];
    if (__builtin_amdgcn_ballot_w64(!(fabsf((all[0] + all[1]) + (all[2] + all[3])) < INFINITY)) != 0) {
#pragma unroll
        for (int ct = 0; ct < 8; ct++) acc[ct] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int u0 = t_begin + wave * 64; u0 < t_end; u0 += (u0 & 48) == 48 ? 64 * kBWaves - 48 : 16) {  // 16 tokens at a time
            uint4 k4[4];
            load_k16(u0, k4);
            v4f p = scores(k4);
#pragma unroll
            for (int r = 0; r < 4; r++) p[r] = __expf(scale * p[r] - m);  // token u0 + 4 gq + r
            const int n = min(t_end - u0, 16);
#pragma unroll 1
            for (int t = 0; t < n; t++) {
                float x[8];
                unpack8(*reinterpret_cast<const uint4 *>(Vb + (size_t)(u0 + t) * row), x);
                const float pt = (t & 2) ? (t & 1) ? p[3] : p[2] : (t & 1) ? p[1] : p[0];
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float pr = __shfl(pt, 16 * (t >> 2) + 4 * gq + r);  // of row 4 gq + r
#pragma unroll
                    for (int ct = 0; ct < 8; ct++)
                        if (4 * gq + r < G) acc[ct][r] = fmaf(pr, x[ct], acc[ct][r]);  // the rows of later parts stay zero
                }
            }
        }
    }
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
    if (gq == 0 && j < G) {
        comb[wave][j][kD] = m;
        comb[wave][j][kD + 1] = lsum;
    }
    // the next part of row 4 gq + r sits G rows further, in lane group gq + G / 4
#pragma unroll
    for (int ct = 0; ct < 8; ct++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            float v = acc[ct][r];
            if constexpr (G == 4) v = add_next<16>(v, 1.f / kNextPart);
            v = add_next<32>(v, G == 4 ? 1.f / (kNextPart * kNextPart) : 1.f / kNextPart);
            if (4 * gq + r < G) comb[wave][4 * gq + r][8 * j + ct] = v;
        }
    __syncthreads();
    merge_waves_and_splits<G>(comb, partials, counters, out, b, h, Hq, split, bh, tid, split_stride);
}

// ---- a plain streaming read: the bound for any kernel that has to read the fp16 cache ---------------------------------
// Every workgroup reads one contiguous chunk with 16-byte loads, eight in flight per lane, and folds the words;
// the fold is stored only if it equals a value the caller's data does not produce (the loads must not be optimised
// away), so normally nothing is written.
constexpr int kStreamLoads = 8;
__global__ __launch_bounds__(256) void read_stream_kernel(const uint4 *__restrict__ src, size_t per_wg16,
                                                          uint32_t *__restrict__ sink) {
    const uint4 *p = src + (size_t)blockIdx.x * per_wg16 + threadIdx.x;
    uint32_t acc = 0;
    for (size_t i = 0; i < per_wg16; i += 256 * kStreamLoads) {
        uint4 v[kStreamLoads];
#pragma unroll
        for (int u = 0; u < kStreamLoads; u++) v[u] = p[i + (size_t)u * 256];
#pragma unroll
        for (int u = 0; u < kStreamLoads; u++) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    if (acc == 0x9e3779b9u && threadIdx.x == 1023) sink[0] = acc;  // never: blockDim.x is 256
}

// Up to 2048 workgroups, each reading a whole number of 32 KiB pieces (256 lanes x 8 loads x 16 bytes); *bytes_read
// receives what is read in total (the largest such amount that fits into `bytes`).
hipError_t launch_read_stream(const void *src, size_t bytes, uint32_t *sink, size_t *bytes_read, hipStream_t s) {
    const size_t piece = (size_t)256 * kStreamLoads * 16;
    const size_t grid = bytes / piece < 2048 ? bytes / piece : 2048;
    *bytes_read = 0;
    if (grid == 0) return hipSuccess;
    const size_t per_wg = bytes / grid / piece * piece;
    *bytes_read = per_wg * grid;
    hipLaunchKernelGGL(read_stream_kernel, dim3((unsigned)grid), dim3(256), 0, s, static_cast<const uint4 *>(src),
                       per_wg / 16, sink);
    return hipGetLastError();
}

// ---- scratch of the entry point that allocates nothing ---------------------------------------------------------
// kvcomp_baseline_fp16_attn_noalloc keeps the split tickets and the split partials in this array instead of a
// caller's workspace.  Every GPU holds its own copy at its own address until the process ends.  Layout: tickets (one
// per (batch, kv head), zero between launches: the merging workgroup resets its ticket) in the first
// kStaticTicketBytes, the partials [batch * q heads][splits used][130] fp32 behind them.
constexpr size_t kStaticTicketBytes = 64 * 1024;    // 16384 (batch, kv head) pairs
constexpr size_t kStaticScratchBytes = 4u << 20;    // tickets + partials
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device (the array's name is a host-side stand-in, not an address that a
// kernel may be given), looked up once per device.
hipError_t baseline_static_scratch(uint32_t **tickets, float **partials, size_t *max_tickets, size_t *partial_bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static unsigned char *per_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    unsigned char *ptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!per_device[dev]) {
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            per_device[dev] = static_cast<unsigned char *>(p);
        }
        ptr = per_device[dev];
    }
    *tickets = reinterpret_cast<uint32_t *>(ptr);
    *partials = reinterpret_cast<float *>(ptr + kStaticTicketBytes);
    *max_tickets = kStaticTicketBytes / sizeof(uint32_t);
    *partial_bytes = kStaticScratchBytes - kStaticTicketBytes;
    return hipSuccess;
}

// Sequence splits that a launch really uses for `seq` tokens when n_splits are asked for (whole 64-token tiles).
int baseline_splits(int seq, int n_splits) {
    int tps = (seq + n_splits - 1) / n_splits;
    tps = (tps + 63) / 64 * 64;
    return (seq + tps - 1) / tps;
}

// split_stride: splits per query head that the layout of `partials` has room for (>= the splits used)
hipError_t launch_baseline_attn(int B, int H, int Hq, const uint16_t *K, const uint16_t *V, int seq, const uint16_t *q,
                                float scale, float *out, float *partials, uint32_t *counters, int n_splits,
                                int split_stride, hipStream_t s) {
    const int G = Hq / H;
    int tps = (seq + n_splits - 1) / n_splits;
    tps = (tps + 63) / 64 * 64;
    n_splits = (seq + tps - 1) / tps;
    if (n_splits > split_stride) return hipErrorInvalidValue;
    const dim3 grid(n_splits, B * H), block(64 * kBWaves);
    switch (G) {
        case 1: hipLaunchKernelGGL(baseline_attn_kernel<1>, grid, block, 0, s, B, H, Hq, K, V, seq, q, scale, partials, counters, out, tps, split_stride); break;
        case 2: hipLaunchKernelGGL(baseline_attn_kernel<2>, grid, block, 0, s, B, H, Hq, K, V, seq, q, scale, partials, counters, out, tps, split_stride); break;
        case 4: hipLaunchKernelGGL(baseline_attn_gqa_kernel<4>, grid, block, 0, s, B, H, Hq, K, V, seq, q, scale, partials, counters, out, tps, split_stride); break;
        case 8: hipLaunchKernelGGL(baseline_attn_gqa_kernel<8>, grid, block, 0, s, B, H, Hq, K, V, seq, q, scale, partials, counters, out, tps, split_stride); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kvc
