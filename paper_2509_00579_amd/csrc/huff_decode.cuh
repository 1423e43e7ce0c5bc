// Wave-level Huffman decode machinery shared by the fused decode-attention kernel and the stand-alone decompressor:
// wave reductions on DPP, the stream readers of a slice (two chains per slice, read from both ends), and the
// lookup-table decode of several symbols per 32-bit window (Section 3.3.1 replaced by a table decode, see
// attn_fused.hip for the reasons).
#pragma once

#include <hip/hip_fp16.h>

#include <type_traits>

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

template <int A, int B, class F>
__device__ __forceinline__ void static_for(F &&f) {  // f(integral constant) for A .. B-1
    if constexpr (A < B) {
        f(std::integral_constant<int, A>());
        static_for<A + 1, B>(f);
    }
}

// A slice holds two decode chains (see the record layout): symbols 0..31 are read upwards from the slice start,
// symbols 63..32 downwards from the slice end.
//   units   the payload as 8-byte units, pointer moved back by one unit: payload bit x is bit x + 64 of units
// A window is 32 bits whose lowest J bits are don't-cares and whose bits J.. are the next unread stream bits in
// reading order, i.e. the stream already scaled to the byte offset of a table entry of 2^J bytes (J = 1: 16-bit
// entries, one symbol each; J = 2: 32-bit entries that deliver two symbols).
//
// A reader gives 64 bits at a time, two windows: the second one starts where the first one's code words end, which one
// funnel shift arranges, so positions and registers move on once per two windows.  It keeps the unit that holds its position,
// the one behind it in reading direction for the bits that reach over, and a third one on its way: one aligned 8-byte LDS
// read per two windows, off the critical path (only table lookups depend on each other).
// The LDS pipe is the busiest unit of the decoders and the streams were a third of its work: a 4-byte gather of 64 lanes from
// a record costs the pipe of a CU 2.5 ns, an aligned 8-byte one 2.2, two 4-byte halves in one ds_read2_b32 4.9, an 8-byte
// one at an odd word 27 (lane by lane), and a chain of 32 symbols takes five aligned ones where it took nine of 4 bytes (with
// the pair table and tables of 7 bits; tables of 8 and 10 bits seven for twelve, of 12 bits nine for seventeen).
struct __attribute__((aligned(8))) Unit { uint32_t lo, hi; };
// payload: first word behind a record's header, 16-byte aligned.  The readers look at up to 16 bytes in front of it and, for
// lookups that are never made, up to kStreamSlack bytes behind the record.
__device__ __forceinline__ const Unit *payload_units(const uint32_t *payload) { return reinterpret_cast<const Unit *>(payload) - 1; }
// From word `odd` of a and b on: words 0, 1 and words 1, 2 shifted by the position's low five bits
__device__ __forceinline__ void unit_bits(const Unit &a, const Unit &b, uint32_t P, uint32_t &lo, uint32_t &hi) {
    const bool odd = (P & 32u) != 0;
    const uint32_t x0 = odd ? a.hi : a.lo, x1 = odd ? b.lo : a.hi, x2 = odd ? b.hi : b.lo;
    lo = __builtin_amdgcn_alignbit(x1, x0, P);
    hi = __builtin_amdgcn_alignbit(x2, x1, P);
}
template <int J>
struct UpReader {
    uint32_t P;       // (next unread payload bit) + 64 - J = start of the 64 bits in unit coordinates
    Unit a, b, next;  // units P / 64, P / 64 + 1, P / 64 + 2
    __device__ __forceinline__ void open(const Unit *units, uint32_t first_bit) {
        P = first_bit + (uint32_t)(64 - J);
        const Unit *u = units + (P >> 6);
        a = u[0];
        b = u[1];
        next = u[2];
    }
    // window at the position, and the 32 stream bits behind it
    __device__ __forceinline__ void bits(uint32_t &first, uint32_t &second) const { unit_bits(a, b, P, first, second); }
    __device__ __forceinline__ void advance(const Unit *units, uint32_t used) {  // used < 64
        const uint32_t old = P >> 6;
        P += used;
        const uint32_t now = P >> 6;
        const bool adv = now != old;
        a.lo = adv ? b.lo : a.lo;
        a.hi = adv ? b.hi : a.hi;
        b.lo = adv ? next.lo : b.lo;
        b.hi = adv ? next.hi : b.hi;
        next = units[now + 2];
    }
};
template <int J>
struct DownReader {
    uint32_t P;       // (one past the next unread payload bit) + J: the 64 bits [P, P + 64) of units end J bits above the
                      // next unread bit; bit-reversed they read downwards
    Unit a, b, next;  // units P / 64, P / 64 + 1, P / 64 - 1
    __device__ __forceinline__ void open(const Unit *units, uint32_t end_bit) {
        P = end_bit + (uint32_t)J;
        const Unit *u = units + (P >> 6);
        a = u[0];
        b = u[1];
        next = u[-1];
    }
    __device__ __forceinline__ void bits(uint32_t &first, uint32_t &second) const {
        uint32_t lo, hi;
        unit_bits(a, b, P, lo, hi);
        first = __builtin_bitreverse32(hi);
        second = __builtin_bitreverse32(lo);
    }
    __device__ __forceinline__ void advance(const Unit *units, uint32_t used) {  // used < 64
        const uint32_t old = P >> 6;
        P -= used;
        const uint32_t now = P >> 6;
        const bool adv = now != old;
        b.lo = adv ? a.lo : b.lo;
        b.hi = adv ? a.hi : b.hi;
        a.lo = adv ? next.lo : a.lo;
        a.hi = adv ? next.hi : a.hi;
        next = units[(int)now - 1];
    }
};

// A table entry.  J = 1: 16-bit entries (symbol << 8) | code length, indexed by the next `bits` stream bits,
// mask = ((1 << bits) - 1) << 1.  J = 2: 32-bit entries of the pair table, indexed by the next 12 stream bits
// (mask = 0xfff << 2): byte 0 = length of two consecutive code words together, byte 1 = first symbol, byte 2 = second
// symbol.  Lookups per window * index width <= 31 - J from four lookups on, else <= 32 - J, is the caller's promise.
// The four chains of one lane (two slices x two directions) advance together.  The four lookups of a
// round are issued back to back before any of their results is used: a wave then waits for the LDS once per round, not
// once per lookup.  (Left to itself the compiler runs the chains of some blocks one after the other.)
template <int J>
struct Quad {
    UpReader<J> au, bu;
    DownReader<J> ad, bd;
    // a = [a0, a0 + abits), b follows it
    __device__ __forceinline__ void open(const Unit *units, uint32_t a0, uint32_t abits, uint32_t bbits) {
        au.open(units, a0);
        ad.open(units, a0 + abits);
        bu.open(units, a0 + abits);
        bd.open(units, a0 + abits + bbits);
    }
    // the same for two slices that do not follow each other in the record
    __device__ __forceinline__ void open2(const Unit *units, uint32_t a0, uint32_t abits, uint32_t b0, uint32_t bbits) {
        au.open(units, a0);
        ad.open(units, a0 + abits);
        bu.open(units, b0);
        bd.open(units, b0 + bbits);
    }
    __device__ __forceinline__ static uint32_t entry(const char *lut, uint32_t at) {
        if constexpr (J == 1) return *reinterpret_cast<const uint16_t *>(lut + at);
        else return *reinterpret_cast<const uint32_t *>(lut + at);
    }
    // CNT lookups of every chain in its window w; tot: what of it they used, only its low five bits are to be looked at
    // (without the sentinel the symbols are above them).  got(K0 + k, entries) as soon as lookup k is there.
    template <int CNT, int K0, class F>
    __device__ __forceinline__ static void window(const char *lut, uint32_t mask, uint32_t (&w)[4], uint32_t (&tot)[4], F &&got) {
        // From four lookups on the bits used are counted by a one in bit 31 of the window that the shifts move down (CNT
        // code words leave it untouched); for fewer it is cheaper to add up the entries' length bytes.
        constexpr bool kSentinel = CNT >= 4;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            tot[c] = 0;
            if constexpr (kSentinel) w[c] |= 0x80000000u;
        }
        static_for<0, CNT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
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
            got(std::integral_constant<int, K0 + k>(), e);
        });
        if constexpr (kSentinel) {
#pragma unroll
            for (int c = 0; c < 4; c++) tot[c] = (uint32_t)__builtin_clz(w[c]);
        }
    }
    // C1 lookups of every chain in the first window and C2 (0: none) in the second; got(k, entries of au, ad, bu, bd)
    template <int C1, int C2, class F>
    __device__ __forceinline__ void step(const Unit *units, const char *lut, uint32_t mask, F &&got) {
        uint32_t w[4], first[4], rest[4], tot[4];
        au.bits(first[0], rest[0]);
        __builtin_amdgcn_sched_barrier(0);
        ad.bits(first[1], rest[1]);
        __builtin_amdgcn_sched_barrier(0);
        bu.bits(first[2], rest[2]);
        __builtin_amdgcn_sched_barrier(0);
        bd.bits(first[3], rest[3]);
#pragma unroll
        for (int c = 0; c < 4; c++) w[c] = first[c];
        window<C1, 0>(lut, mask, w, tot, got);
        if constexpr (C2 > 0) {
            uint32_t tot2[4];
#pragma unroll
            for (int c = 0; c < 4; c++) w[c] = __builtin_amdgcn_alignbit(rest[c], first[c], tot[c]);
            window<C2, C1>(lut, mask, w, tot2, got);
#pragma unroll
            for (int c = 0; c < 4; c++) tot[c] += tot2[c];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) tot[c] &= 0xffu;
        // one chain after the other: the selects then all take their condition from VCC, where an instruction is one issue slot
        // and not two
        __builtin_amdgcn_sched_barrier(0);
        au.advance(units, tot[0]);
        __builtin_amdgcn_sched_barrier(0);
        ad.advance(units, tot[1]);
        __builtin_amdgcn_sched_barrier(0);
        bu.advance(units, tot[2]);
        __builtin_amdgcn_sched_barrier(0);
        bd.advance(units, tot[3]);
        __builtin_amdgcn_sched_barrier(0);
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
    static constexpr int kTableBytes = (kPair ? 4 : 2) << kIndexBits;     // per tensor
};

// A word of four consecutive symbols of a chain grows by one table entry at a time.  AT: number of the entry's first symbol
// inside the word; kDown: the chain is read downwards, so that its first symbol belongs into the highest byte.
template <int SYMS, int AT, bool kDown>
__device__ __forceinline__ uint32_t add_syms(uint32_t word, uint32_t e) {
    if constexpr (AT == 0) return e;  // as it came: its symbols are in bytes 1 (and 2)
    if constexpr (SYMS == 2) return __builtin_amdgcn_perm(e, word, kDown ? 0x01020506u : 0x06050201u);
    // one symbol an entry: word holds AT of them, the first still in byte 1 for AT = 1
    if constexpr (AT == 1) return __builtin_amdgcn_perm(e, word, kDown ? 0x0c0c0105u : 0x0c0c0501u);
    if constexpr (AT == 2) return __builtin_amdgcn_perm(e, word, kDown ? 0x0c010005u : 0x0c050100u);
    return __builtin_amdgcn_perm(e, word, kDown ? 0x02010005u : 0x05020100u);
}

// The decoded symbols of the lane's two slices, four per word, in ascending position inside the slice:
// word j of a slice holds positions 4j .. 4j+3.  The up chain delivers words 0, 1, .. and the down chain 15, 14, ..
struct SliceWords {
    uint32_t a[16], b[16];
};
// Decodes this lane's four chains and packs every word as soon as its four symbols are there: word(slice, index, value), the
// first two as integral constants.
template <int LB, class F>
__device__ __forceinline__ void decode_words(Quad<DecodeMode<LB>::J> &qd, const Unit *units, const char *lut, uint32_t mask,
                                             F &&word) {
    using M = DecodeMode<LB>;
    using std::integral_constant;
    constexpr int SP = M::kSymsPerLookup, NL = M::kLookupsPerWindow, kLookups = kHalf / SP;
    uint32_t part[4];
    // C1 + C2 lookups from number K on
    auto take = [&](auto kc, auto c1, auto c2) {
        constexpr int K = decltype(kc)::value, C1 = decltype(c1)::value, C2 = decltype(c2)::value;
        qd.template step<C1, C2>(units, lut, mask, [&](auto lc, const uint32_t (&e)[4]) {
            constexpr int first = (K + decltype(lc)::value) * SP, at = first % 4, w = first / 4;
#pragma unroll
            for (int c = 0; c < 4; c++)
                part[c] = c & 1 ? add_syms<SP, at, true>(part[c], e[c]) : add_syms<SP, at, false>(part[c], e[c]);
            // packed here and now: left to itself the compiler packs after the last lookup and keeps every entry until then
            if constexpr (at > 0 && (at + SP) % 2 == 0) asm volatile("" : "+v"(part[0]), "+v"(part[1]), "+v"(part[2]), "+v"(part[3]));
            if constexpr (at + SP == 4) {
                constexpr integral_constant<int, 0> a;
                constexpr integral_constant<int, 1> b;
                constexpr integral_constant<int, w> up;
                constexpr integral_constant<int, 15 - w> down;
                word(a, up, part[0]);
                word(a, down, part[1]);
                word(b, up, part[2]);
                word(b, down, part[3]);
            }
        });
    };
    constexpr int kSteps = (kLookups + 2 * NL - 1) / (2 * NL);  // two windows each; the last one may be short
    static_for<0, kSteps>([&](auto r) {
        constexpr int K = decltype(r)::value * 2 * NL, n = kLookups - K < 2 * NL ? kLookups - K : 2 * NL;
        constexpr int C1 = n < NL ? n : NL;
        take(integral_constant<int, K>(), integral_constant<int, C1>(), integral_constant<int, n - C1>());
    });
}
// the same into registers
template <int LB>
__device__ __forceinline__ void decode_block(Quad<DecodeMode<LB>::J> &qd, const Unit *units, const char *lut, uint32_t mask,
                                             SliceWords &p) {
    decode_words<LB>(qd, units, lut, mask, [&](auto slice, auto index, uint32_t v) {
        if constexpr (decltype(slice)::value == 0) p.a[decltype(index)::value] = v;
        else p.b[decltype(index)::value] = v;
    });
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
