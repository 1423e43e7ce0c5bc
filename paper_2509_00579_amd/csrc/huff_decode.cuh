// Wave-level Huffman decode machinery shared by the fused decode-attention kernel and the stand-alone decompressor:
// wave reductions on DPP, the stream readers of a slice (two chains per slice, read from both ends), and the
// lookup-table decode of several symbols per 32-bit window (Section 3.3.1 replaced by a table decode, see
// attn_fused.hip for the reasons).
#pragma once

#include <hip/hip_fp16.h>

#include "kvcomp_internal.h"

namespace kvc {

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float h2f(uint32_t bits) { return __half2float(__ushort_as_half((unsigned short)bits)); }

// value of `v` in lane `lane_idx` (wave-uniform index), delivered in a scalar register
__device__ __forceinline__ float bcast(float v, int lane_idx) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane_idx));
}

// Wave-wide reductions and the prefix sum run on DPP row operations and v_readlane, not on ds_bpermute: the LDS pipe
// is the busiest unit of this kernel and a butterfly of six dependent LDS round trips costs far more latency.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {  // lanes without a source read 0
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;              // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kDppHalfMirror = 0x141, kDppMirror = 0x140;    // lane i <-> 7 - i (within 8) and i <-> 15 - i (within 16)
constexpr int kDppRowShr = 0x110;                            // + n: lane i reads lane i - n of its row of 16

// the same value in every lane
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f<kDppXor1>(v);
    v += dpp_f<kDppXor2>(v);
    v += dpp_f<kDppHalfMirror>(v);
    v += dpp_f<kDppMirror>(v);  // every lane: sum of its row of 16
    return (bcast(v, 0) + bcast(v, 16)) + (bcast(v, 32) + bcast(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_f<kDppXor1>(v));
    v = fmaxf(v, dpp_f<kDppXor2>(v));
    v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_f<kDppMirror>(v));
    return fmaxf(fmaxf(bcast(v, 0), bcast(v, 16)), fmaxf(bcast(v, 32), bcast(v, 48)));
}
// exclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, int lane) {
    uint32_t inc = v;
    inc += dpp_u<kDppRowShr + 1>(inc);
    inc += dpp_u<kDppRowShr + 2>(inc);
    inc += dpp_u<kDppRowShr + 4>(inc);
    inc += dpp_u<kDppRowShr + 8>(inc);  // inclusive within each row of 16
    const uint32_t t0 = __builtin_amdgcn_readlane(inc, 15), t1 = __builtin_amdgcn_readlane(inc, 31),
                   t2 = __builtin_amdgcn_readlane(inc, 47);
    const int row = lane >> 4;
    const uint32_t before = row == 0 ? 0u : row == 1 ? t0 : row == 2 ? t0 + t1 : t0 + t1 + t2;
    return inc + before - v;
}

// A slice holds two decode chains (see the record layout): symbols 0..31 are read upwards from the slice start,
// symbols 63..32 downwards from the slice end.
//   wm1   payload words, pointer moved back by one word: payload bit x is bit x + 32 of wm1
// A window is 32 bits whose lowest J bits are don't-cares and whose bits J.. are the next unread stream bits in
// reading order, i.e. the stream already scaled to the byte offset of a table entry of 2^J bytes (J = 1: 16-bit
// entries, one symbol each; J = 2: 32-bit entries that deliver two symbols).
// (Unaligned 4-byte LDS reads at byte granularity, and re-reading both words of every window, were tried: slower.)
//
// Readers keep a 64-bit piece {hi,lo} of the stream in registers plus the next word in reading direction, fetched
// one window ahead: one 4-byte LDS read per window, off the critical path (only table lookups depend on each other).
template <int J>
struct UpReader {
    uint32_t P, idx, lo, hi, nx;  // P = (next unread payload bit) + 32 - J = window start in wm1 bit coordinates
    __device__ __forceinline__ void open(const uint32_t *wm1, uint32_t first_bit) {
        P = first_bit + (uint32_t)(32 - J);
        idx = P >> 5;
        lo = wm1[idx];
        hi = wm1[idx + 1];
        nx = wm1[idx + 2];
    }
    __device__ __forceinline__ uint32_t window(const uint32_t *) const { return __builtin_amdgcn_alignbit(hi, lo, P); }
    __device__ __forceinline__ void advance(const uint32_t *wm1, uint32_t used) {  // used <= 32 - J
        P += used;
        const uint32_t nidx = P >> 5;
        const bool adv = nidx != idx;
        lo = adv ? hi : lo;
        hi = adv ? nx : hi;
        idx = nidx;
        nx = wm1[nidx + 2];
    }
};
template <int J>
struct DownReader {
    uint32_t P, idx, lo, hi, pv;  // P = (one past the next unread payload bit) + J: the window [P, P+32) of wm1 ends J
                                  // bits above the next unread bit; bit-reversed it reads downwards
    __device__ __forceinline__ void open(const uint32_t *wm1, uint32_t end_bit) {
        P = end_bit + (uint32_t)J;
        idx = P >> 5;
        lo = wm1[idx];
        hi = wm1[idx + 1];
        pv = wm1[(int)idx - 1];
    }
    __device__ __forceinline__ uint32_t window(const uint32_t *) const {
        return __builtin_bitreverse32(__builtin_amdgcn_alignbit(hi, lo, P));
    }
    __device__ __forceinline__ void advance(const uint32_t *wm1, uint32_t used) {  // used <= 32 - J
        P -= used;
        const uint32_t nidx = P >> 5;
        const bool adv = nidx != idx;
        hi = adv ? lo : hi;
        lo = adv ? pv : lo;
        idx = nidx;
        pv = wm1[(int)nidx - 1];
    }
};

// A table entry.  J = 1: 16-bit entries (symbol << 8) | code length, indexed by the next `bits` stream bits,
// mask = ((1 << bits) - 1) << 1.  J = 2: 32-bit entries of the pair table, indexed by the next 12 stream bits
// (mask = 0xfff << 2): byte 0 = length of two consecutive code words together, byte 1 = first symbol, byte 2 = second
// symbol.  Lookups per window * index width <= 31 - J from four lookups on, else <= 32 - J, is the caller's promise.
// The four chains of one lane (two slices x two directions) advance together, CNT lookups each.  The four lookups of a
// round are issued back to back before any of their results is used: a wave then waits for the LDS once per round, not
// once per lookup.  (Left to itself the compiler runs the chains of some blocks one after the other.)
template <int J>
struct Quad {
    UpReader<J> au, bu;
    DownReader<J> ad, bd;
    // a = [a0, a0 + abits), b follows it
    __device__ __forceinline__ void open(const uint32_t *wm1, uint32_t a0, uint32_t abits, uint32_t bbits) {
        au.open(wm1, a0);
        ad.open(wm1, a0 + abits);
        bu.open(wm1, a0 + abits);
        bd.open(wm1, a0 + abits + bbits);
    }
    // the same for two slices that do not follow each other in the record
    __device__ __forceinline__ void open2(const uint32_t *wm1, uint32_t a0, uint32_t abits, uint32_t b0, uint32_t bbits) {
        au.open(wm1, a0);
        ad.open(wm1, a0 + abits);
        bu.open(wm1, b0);
        bd.open(wm1, b0 + bbits);
    }
    __device__ __forceinline__ static uint32_t entry(const char *lut, uint32_t at) {
        if constexpr (J == 1) return *reinterpret_cast<const uint16_t *>(lut + at);
        else return *reinterpret_cast<const uint32_t *>(lut + at);
    }
    template <int CNT>
    __device__ __forceinline__ void step(const uint32_t *wm1, const char *lut, uint32_t mask, uint32_t (&fau)[CNT],
                                         uint32_t (&fad)[CNT], uint32_t (&fbu)[CNT], uint32_t (&fbd)[CNT]) {
        // From four lookups on the bits used are counted by a one in bit 31 of the window that the shifts move down (CNT
        // code words leave it untouched); for fewer it is cheaper to add up the entries' length bytes.
        constexpr bool kSentinel = CNT >= 4;
        uint32_t w[4] = {au.window(wm1), ad.window(wm1), bu.window(wm1), bd.window(wm1)}, tot[4] = {0, 0, 0, 0};
        if constexpr (kSentinel) {
#pragma unroll
            for (int c = 0; c < 4; c++) w[c] |= 0x80000000u;
        }
#pragma unroll
        for (int k = 0; k < CNT; k++) {
            uint32_t at[4], e[4];
#pragma unroll
            for (int c = 0; c < 4; c++) at[c] = w[c] & mask;
#pragma unroll
            for (int c = 0; c < 4; c++) e[c] = entry(lut, at[c]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < 4; c++) {
                if (kSentinel || k + 1 < CNT) w[c] >>= (e[c] & 31u);
                if (!kSentinel) tot[c] += e[c];
            }
            fau[k] = e[0]; fad[k] = e[1]; fbu[k] = e[2]; fbd[k] = e[3];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) tot[c] = kSentinel ? (uint32_t)__builtin_clz(w[c]) : tot[c] & 0xffu;
        au.advance(wm1, tot[0]);
        ad.advance(wm1, tot[1]);
        bu.advance(wm1, tot[2]);
        bd.advance(wm1, tot[3]);
    }
};

constexpr int kHalf = kSliceLen / 2;  // symbols per chain
constexpr int kPairIndexBits = 12;    // index width of the pair table: two code words of up to 6 bits
constexpr int kPairLongest = kPairIndexBits / 2;

// How a kernel compiled for code words of up to LB bits decodes.  LB <= 6: the pair table (every lookup delivers two
// symbols, so a chain of 32 symbols is 16 dependent lookups).  Otherwise the single-symbol table of 2^LB 16-bit
// entries.
template <int LB>
struct DecodeMode {
    static constexpr bool kPair = LB <= kPairLongest;
    static constexpr int J = kPair ? 2 : 1;                               // log2 of the entry size in bytes
    static constexpr int kIndexBits = kPair ? kPairIndexBits : LB;
    static constexpr int kSymsPerLookup = kPair ? 2 : 1;
    static constexpr int kLookupsPerWindow = (32 - J) / kIndexBits;       // pair table: 2; 7, 8, 10, 12 bits: 4, 3, 3, 2
    static constexpr int kSymsPerWindow = kSymsPerLookup * kLookupsPerWindow;
    static constexpr int kLookupsPerChain = kHalf / kSymsPerLookup;
    static constexpr int kTableBytes = (kPair ? 4 : 2) << kIndexBits;     // per tensor
};

// bytes 1 of four table entries (the symbols) as one word, first entry in the lowest byte
__device__ __forceinline__ uint32_t pack_syms(uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e3) {
    const uint32_t lo = __builtin_amdgcn_perm(e1, e0, 0x0c0c0501u), hi = __builtin_amdgcn_perm(e3, e2, 0x0c0c0501u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
// the same from two entries of the pair table (bytes 1 and 2 of each are two consecutive symbols): e0's symbols in
// the two lowest bytes; and with the four symbols in the opposite order (a chain that was read downwards)
__device__ __forceinline__ uint32_t pack_pairs(uint32_t e0, uint32_t e1) { return __builtin_amdgcn_perm(e1, e0, 0x06050201u); }
__device__ __forceinline__ uint32_t pack_pairs_rev(uint32_t e0, uint32_t e1) { return __builtin_amdgcn_perm(e1, e0, 0x01020506u); }

// The table entries of a lane's four chains while they wait to be packed (fully unrolled code: an entry lives in a
// register from its lookup to the packing of its word).  NE entries per chain: 32 one-symbol or 16 two-symbol ones.
template <int NE>
struct ChainSyms {
    uint32_t au[NE], ad[NE], bu[NE], bd[NE];
};
// The decoded symbols of the lane's two slices, four per word, in ascending position inside the slice:
// word j of a slice holds positions 4j .. 4j+3.  The up chain delivers words 0, 1, .. and the down chain 15, 14, ..
struct SliceWords {
    uint32_t a[16], b[16];
};
// Decodes symbols S0 .. S1-1 of this lane's four chains (whole windows from S0 on; the last window of a chain may be
// short) and packs every word whose four symbols are there.
template <int LB, int S0, int S1>
__device__ __forceinline__ void decode_span(Quad<DecodeMode<LB>::J> &qd, const uint32_t *wm1, const char *lut, uint32_t mask,
                                            ChainSyms<DecodeMode<LB>::kLookupsPerChain> &e, SliceWords &p) {
    using M = DecodeMode<LB>;
    constexpr int SP = M::kSymsPerLookup, NL = M::kLookupsPerWindow, NS = M::kSymsPerWindow;
    static_assert(S0 % NS == 0 && S0 < S1 && S1 <= kHalf && (S1 % NS == 0 || S1 == kHalf), "whole windows");
    auto pack_words = [&](int w0, int w1) {
#pragma unroll
        for (int w = w0; w < w1; w++) {
            if constexpr (SP == 1) {
                p.a[w] = pack_syms(e.au[4 * w], e.au[4 * w + 1], e.au[4 * w + 2], e.au[4 * w + 3]);
                p.a[15 - w] = pack_syms(e.ad[4 * w + 3], e.ad[4 * w + 2], e.ad[4 * w + 1], e.ad[4 * w]);
                p.b[w] = pack_syms(e.bu[4 * w], e.bu[4 * w + 1], e.bu[4 * w + 2], e.bu[4 * w + 3]);
                p.b[15 - w] = pack_syms(e.bd[4 * w + 3], e.bd[4 * w + 2], e.bd[4 * w + 1], e.bd[4 * w]);
            } else {
                p.a[w] = pack_pairs(e.au[2 * w], e.au[2 * w + 1]);
                p.a[15 - w] = pack_pairs_rev(e.ad[2 * w], e.ad[2 * w + 1]);
                p.b[w] = pack_pairs(e.bu[2 * w], e.bu[2 * w + 1]);
                p.b[15 - w] = pack_pairs_rev(e.bd[2 * w], e.bd[2 * w + 1]);
            }
        }
    };
    constexpr int kFull = (S1 - S0) / NS, kTailSyms = (S1 - S0) - kFull * NS, kTail = kTailSyms / SP;
    static_assert(kTailSyms % SP == 0, "a span ends on a whole table entry");
#pragma unroll
    for (int r = 0; r < kFull; r++) {
        uint32_t fau[NL], fad[NL], fbu[NL], fbd[NL];
        qd.template step<NL>(wm1, lut, mask, fau, fad, fbu, fbd);
        const int s = S0 + r * NS;
#pragma unroll
        for (int k = 0; k < NL; k++) {
            e.au[s / SP + k] = fau[k]; e.ad[s / SP + k] = fad[k]; e.bu[s / SP + k] = fbu[k]; e.bd[s / SP + k] = fbd[k];
        }
        pack_words(s / 4, (s + NS) / 4);
    }
    if constexpr (kTail > 0) {
        uint32_t fau[kTail ? kTail : 1], fad[kTail ? kTail : 1], fbu[kTail ? kTail : 1], fbd[kTail ? kTail : 1];
        qd.template step<(kTail ? kTail : 1)>(wm1, lut, mask, fau, fad, fbu, fbd);
        constexpr int s = S0 + kFull * NS;
#pragma unroll
        for (int k = 0; k < kTail; k++) {
            e.au[s / SP + k] = fau[k]; e.ad[s / SP + k] = fad[k]; e.bu[s / SP + k] = fbu[k]; e.bd[s / SP + k] = fbd[k];
        }
        pack_words(s / 4, (s + kTailSyms) / 4);
    }
}
// the 4 x 4 bytes of a quad of lanes transposed: lane q of the result holds byte q of the four lanes' words, lane 0's in
// the lowest byte
struct QuadTranspose {
    uint32_t sel1, sel2;
    __device__ __forceinline__ explicit QuadTranspose(int lane)
        : sel1((lane & 1) ? 0x03070105u : 0x06020400u), sel2((lane & 2) ? 0x03020706u : 0x05040100u) {}
    __device__ __forceinline__ uint32_t operator()(uint32_t u) const {
        const uint32_t v = __builtin_amdgcn_perm(dpp_u<kDppXor1>(u), u, sel1);
        return __builtin_amdgcn_perm(dpp_u<kDppXor2>(v), v, sel2);
    }
};
// A record goes from global memory straight into the wave's staging area with LDS-direct loads (lane l of load i delivers
// its 16 bytes to byte 1024 i + 16 l; in the last one the lanes beyond the record are masked out), issued when the
// previous record has been decoded: no register holds it on the way.
__device__ __forceinline__ void load_lds16(const uint4 *src, uint8_t *dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}
__device__ __forceinline__ void stage_record(const uint8_t *rec, uint32_t size16, uint8_t *stage, int lane) {
    const uint4 *src = reinterpret_cast<const uint4 *>(rec);
    const uint32_t n_full = size16 >> 6, rest = size16 & 63u;
    for (uint32_t i = 0; i < n_full; i++) load_lds16(src + 64 * i + lane, stage + 1024 * i);
    if ((uint32_t)lane < rest) load_lds16(src + 64 * n_full + lane, stage + 1024 * n_full);
}
__device__ __forceinline__ void wait_record() { __builtin_amdgcn_s_waitcnt(0); }  // vmcnt(0): the loads have written the LDS

}  // namespace kvc
