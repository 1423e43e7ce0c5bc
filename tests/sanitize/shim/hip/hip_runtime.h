// Stands in for the HIP runtime header where device code is compiled for the CPU: what the decoders' headers use of it, for
// one lane.  The AMD builtins are written out from their documented results.
#pragma once

#include <stddef.h>
#include <stdint.h>

#define __host__
#define __device__
#define __forceinline__ inline

typedef int hipError_t;
typedef void *hipStream_t, *hipEvent_t;

inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline uint32_t shim_alignbit(uint32_t hi, uint32_t lo, uint32_t sh) { return (uint32_t)((((uint64_t)hi << 32) | lo) >> (sh & 31u)); }
inline uint32_t shim_bitreverse32(uint32_t v) {
    uint32_t r = 0;
    for (int i = 0; i < 32; i++) r |= ((v >> i) & 1u) << (31 - i);
    return r;
}
inline uint32_t shim_perm(uint32_t a, uint32_t b, uint32_t sel) {  // selectors 0..7 and 0x0c are all that is used
    const uint64_t both = ((uint64_t)a << 32) | b;
    uint32_t r = 0;
    for (int i = 0; i < 4; i++) {
        const uint32_t s = (sel >> (8 * i)) & 0xffu;
        if (s < 8) r |= (uint32_t)((both >> (8 * s)) & 0xffu) << (8 * i);
    }
    return r;
}
#define __builtin_amdgcn_alignbit shim_alignbit
#define __builtin_bitreverse32 shim_bitreverse32
#define __builtin_amdgcn_perm shim_perm
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
// exchanges between lanes: never called here
#define __builtin_amdgcn_readlane(v, l) (v)
#define __builtin_amdgcn_update_dpp(old, v, ...) (v)
#define __builtin_bit_cast(T, v) shim_bit_cast<T>(v)
template <class T, class F>
inline T shim_bit_cast(const F &f) {
    static_assert(sizeof(T) == sizeof(F), "same size");
    T t;
    __builtin_memcpy(&t, &f, sizeof(t));
    return t;
}
inline int __float_as_int(float f) { return shim_bit_cast<int>(f); }
inline float __int_as_float(int i) { return shim_bit_cast<float>(i); }
template <class P>
inline void shim_load_lds(P, void *, int, int, int) { __builtin_trap(); }
#define __builtin_amdgcn_global_load_lds(src, dst, n, off, aux) shim_load_lds(src, (void *)(dst), n, off, aux)
