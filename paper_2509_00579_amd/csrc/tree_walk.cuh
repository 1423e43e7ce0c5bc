// The bit-serial decoder of Section 3.3.1, for the A/B against the table decoder: one stream bit per step, node =
// tree[node][bit], a symbol is emitted and the walk restarts at the root when a leaf is reached; no branch depends on the data.
#pragma once

#include "huff_decode.cuh"

namespace kvc {

struct TreeWalk {
    int node, count;  // current inner node, symbols emitted so far
    __device__ __forceinline__ void init() { node = 0; count = 0; }
    // returns the symbol (>= 0) if this bit completed a code word of a chain that still has symbols to give, else -1
    __device__ __forceinline__ int step(const int16_t *tree, uint32_t bit) {
        const int next = tree[node * 2 + (int)bit];
        const bool leaf = next < 0, live = count < kHalf;
        node = leaf ? 0 : next;
        const int sym = (leaf && live) ? ~next : -1;
        count += (leaf && live) ? 1 : 0;
        return sym;
    }
};

// All four chains of the lane walk one bit per step; a window gives 31 bits, then every reader whose chain goes on moves on by
// 31 (all 31 were that chain's, so it stays inside its slice; one whose chain has ended stays where it is, while other
// lanes go on).  A chain stops emitting after its 32 symbols; the wave runs until every chain of every lane is done.
// emit(chain, symbol or -1, its number in the chain); any: whether its argument is true in any lane of the wave.
template <class E, class A>
__device__ __forceinline__ void walk_chains(const Unit *units, const int16_t *tree, uint32_t start, uint32_t abits, uint32_t bbits,
                                            E &&emit, A &&any) {
    constexpr int kWindowBits = 31;
    Quad<1> qd;
    qd.open(units, start, abits, bbits);
    TreeWalk tw[4];
#pragma unroll
    for (int c = 0; c < 4; c++) tw[c].init();
    // 32 symbols of at most 12 bits need at most 13 windows of 31 bits: the bound also ends the loop on a
    // damaged table
    bool more = true;
    for (int round = 0; round < 16 && more; round++) {
        uint32_t w0, w1, w2, w3, behind;
        qd.au.bits(w0, behind);
        qd.ad.bits(w1, behind);
        qd.bu.bits(w2, behind);
        qd.bd.bits(w3, behind);
        w0 >>= 1; w1 >>= 1; w2 >>= 1; w3 >>= 1;
#pragma unroll 1
        for (int k = 0; k < kWindowBits; k++) {
            const int i0 = tw[0].count, i1 = tw[1].count, i2 = tw[2].count, i3 = tw[3].count;
            emit(0, tw[0].step(tree, w0 & 1u), i0);
            emit(1, tw[1].step(tree, w1 & 1u), i1);
            emit(2, tw[2].step(tree, w2 & 1u), i2);
            emit(3, tw[3].step(tree, w3 & 1u), i3);
            w0 >>= 1; w1 >>= 1; w2 >>= 1; w3 >>= 1;
        }
        const bool g0 = tw[0].count < kHalf, g1 = tw[1].count < kHalf, g2 = tw[2].count < kHalf, g3 = tw[3].count < kHalf;
        qd.au.advance(units, g0 ? kWindowBits : 0);
        qd.ad.advance(units, g1 ? kWindowBits : 0);
        qd.bu.advance(units, g2 ? kWindowBits : 0);
        qd.bd.advance(units, g3 ? kWindowBits : 0);
        more = any(g0 || g1 || g2 || g3);
    }
}

}  // namespace kvc
