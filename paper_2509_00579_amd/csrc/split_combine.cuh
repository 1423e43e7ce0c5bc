// Merging the sequence splits of a decode-attention launch inside the same kernel (the "sum reduction" that ends
// the V path in Section 3.3.2).  Every workgroup writes one partial (o[128], m, l) per query head; the workgroup
// that arrives last at a per-(batch, kv head) ticket counter merges all splits and writes the output.  The counter
// is left at zero for the next launch.
//
// gfx950 has one L2 per XCD, and the workgroups of one launch are spread over all XCDs.  A device-scope fence would
// write back / invalidate a whole L2 on every workgroup, which costs far more than the merge itself.  Instead the
// few words that cross workgroups -- the partials and the ticket -- are written and read with device-scope (agent)
// atomic accesses, which go through to the memory-side coherence point, and each wave waits for its own partial
// stores to complete before the workgroup takes its ticket.
#pragma once

#include "huff_decode.cuh"
#include "kvcomp_internal.h"

namespace kvc {

// The lowest reference of a softmax state that has met a token.  A maximum over tokens that all score -Inf or NaN is -Inf (fmaxf
// passes a NaN over), and against a reference of -Inf the numerators of the former would be NaN, while a state with the latter
// would look like one that has met nothing.  Against this one they are 0 and NaN.  So a reference of -Inf says that a state holds
// nothing, to every merge, and a NaN score makes its head's output NaN whatever wave or split it is in.
constexpr float kLowestRef = -3.402823466e38f;

__device__ __forceinline__ void store_agent(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_agent(const float *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by all threads of the workgroup after they have written this workgroup's partials with store_agent() to
// partials[(row0 + g) * split_stride + split].  nt = threads per workgroup (whole waves); scratch: kPartialStride floats of
// LDS per wave, free behind the caller's last barrier.
//
// The merge is the tail of the launch: one workgroup, bound by the latency of loads that pass the L2.  A wave merges one
// head over a range of splits, with as many ranges as there are waves to a head: lane s holds {m, l} of the range's split
// s (two splits when the range is that long), so the weight of every split is known after one reduction, and the two
// accumulator words per lane and split are requested 16 splits at a time before anything is waited for.  Before, a
// thread ran over all splits of one channel with a running maximum, three loads a split, and half or more of the threads
// of a small workgroup ran over several channels one after the other.
// Few heads over a long cache have the most splits.  us a step, before -> now: 1 head x 32768 tokens (128 splits) groups
// of 1 18.0 -> 10.7, of 8 34.4 -> 22.8; 8 heads x 16384 (32) 16.0 -> 15.0 and 24.1 -> 21.5; 8 heads x 2048 (8) 8.6 -> 8.5
// and 13.5 -> 12.1; fp16 kernel, groups of 8, 2 heads x 16384 (64) 30.9 -> 20.3, 8 x 8 heads x 16384 (4) 105.4 -> 103.3.
// kPairs: the partials are 8-byte aligned, and a lane takes two neighbouring channels with one load.
template <int G, bool kPairs>
__device__ __forceinline__ void finish_splits(float *partials, uint32_t *counter, int row0, int n_splits, float *out,
                                              int tid, int nt, float *scratch, int split_stride = kMaxSplits) {
    static_assert(kMaxSplits <= 128, "a lane holds the state of two splits");
    __shared__ uint32_t s_last;
    // every wave: all of its (write-through) partial stores have completed before the barrier is passed
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);  // vmcnt(0) expcnt(0) lgkmcnt(0)
    __syncthreads();
    if (tid == 0) {
        const uint32_t ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = ticket == (uint32_t)(n_splits - 1);
    }
    __syncthreads();
    if (!s_last) return;
    constexpr int kBatch = 16;  // ranges shorter than this only add their own merge
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = nt >> 6;
    const int c0 = kPairs ? 2 * lane : lane, c1 = kPairs ? c0 + 1 : lane + 64;  // this lane's channels
    const int ranges = min(max(n_waves / G, 1), (n_splits + kBatch - 1) / kBatch);
    const int per = (n_splits + ranges - 1) / ranges;
    for (int item = wave; item < G * ranges; item += n_waves) {  // one round, unless there are fewer waves than heads
        const int r = item / G, g = item - r * G, s0 = r * per, n = min(per, n_splits - s0);  // n < 1: an empty range
        const float *p = partials + ((size_t)(row0 + g) * split_stride + s0) * kPartialStride;
        float m0 = -INFINITY, m1 = -INFINITY, l0 = 0.f, l1 = 0.f;
        if (lane < n) {
            m0 = load_agent(p + lane * kPartialStride + kD);
            l0 = load_agent(p + lane * kPartialStride + kD + 1);
        }
        if (lane + 64 < n) {
            m1 = load_agent(p + (lane + 64) * kPartialStride + kD);
            l1 = load_agent(p + (lane + 64) * kPartialStride + kD + 1);
        }
        float o[kBatch][2];
        auto request = [&](int s) {
#pragma unroll
            for (int k = 0; k < kBatch; k++) {
                o[k][0] = o[k][1] = 0.f;
                if (s + k >= n) continue;
                if constexpr (kPairs) {
                    const unsigned long long two = __hip_atomic_load(
                        reinterpret_cast<const unsigned long long *>(p + (s + k) * kPartialStride + 2 * lane), __ATOMIC_RELAXED,
                        __HIP_MEMORY_SCOPE_AGENT);
                    o[k][0] = __uint_as_float((uint32_t)two);
                    o[k][1] = __uint_as_float((uint32_t)(two >> 32));
                } else {
                    o[k][0] = load_agent(p + (s + k) * kPartialStride + lane);
                    o[k][1] = load_agent(p + (s + k) * kPartialStride + lane + 64);
                }
            }
        };
        request(0);
        float mx = fmaxf(m0, m1);
        mx = wave_max(mx);
        // a split that had nothing to do (m = -inf) takes no part, whatever its words are
        if (m0 == -INFINITY) l0 = 0.f;
        if (m1 == -INFINITY) l1 = 0.f;
        const unsigned long long live0 = __builtin_amdgcn_ballot_w64(m0 != -INFINITY),
                                 live1 = __builtin_amdgcn_ballot_w64(m1 != -INFINITY);
        const float f0 = m0 == -INFINITY ? 0.f : __expf(m0 - mx), f1 = m1 == -INFINITY ? 0.f : __expf(m1 - mx);
        const float L = wave_sum(l0 * f0 + l1 * f1);
        float O0 = 0.f, O1 = 0.f;
        for (int s = 0; s < n; s += kBatch) {
            if (s) request(s);
#pragma unroll
            for (int k = 0; k < kBatch; k++) {  // without branches: the loads are waited for once
                const int at = (s + k) & 63;
                const float w0 = bcast(f0, at), w1 = bcast(f1, at);
                const float w = s + k < 64 ? w0 : w1;
                const bool live = ((s + k < 64 ? live0 : live1) >> at) & 1;
                O0 = fmaf(w, live ? o[k][0] : 0.f, O0);
                O1 = fmaf(w, live ? o[k][1] : 0.f, O1);
            }
        }
        if (ranges == 1) {
            out[(size_t)(row0 + g) * kD + c0] = O0 / L;
            out[(size_t)(row0 + g) * kD + c1] = O1 / L;
        } else {
            float *c = scratch + item * kPartialStride;  // item = wave here
            c[c0] = O0;
            c[c1] = O1;
            if (lane == 0) { c[kD] = mx; c[kD + 1] = L; }
        }
    }
    if (ranges > 1) {
        __syncthreads();
        for (int i = tid; i < G * kD; i += nt) {
            const int g = i / kD, c = i - g * kD;
            float mx = -INFINITY, L = 0.f, O = 0.f;
            for (int r = 0; r < ranges; r++) mx = fmaxf(mx, scratch[(r * G + g) * kPartialStride + kD]);
            for (int r = 0; r < ranges; r++) {
                const float *cr = scratch + (r * G + g) * kPartialStride;
                const float f = cr[kD] == -INFINITY ? 0.f : __expf(cr[kD] - mx);
                L = fmaf(cr[kD + 1], f, L);
                O = fmaf(cr[c], f, O);
            }
            out[(size_t)(row0 + g) * kD + c] = O / L;
        }
    }
    if (tid == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace kvc
