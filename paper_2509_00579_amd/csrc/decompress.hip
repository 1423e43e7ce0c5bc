// Stand-alone decompression: the first stage of the multi-kernel pipeline that Section 4.3 compares the fused kernel
// with (decode -> dequantize -> write the cache back in its own precision; a separate matrix-vector kernel then reads
// it).  One wave per 2D block: the record is staged in LDS, decoded with the same table decoder as the fused kernel
// (four chains per lane) into packed codes in registers, and written out as fp16 rows,
//     x' = fp16( min + float(code) * width ),   binary32 multiply, binary32 add, one rounding.
#include "huff_decode.cuh"
#include "kvcomp_internal.h"
#include "tree_walk.cuh"

namespace kvc {

constexpr int kDecWaves = 4;

struct DecompArgs {
    Geo g;
    uint16_t *out;
    int which, n_blocks, seq_stride, area_bytes, stage_bytes;
    int res_head, n_res;
    uint32_t *host_refused;  // pinned host memory
    uint32_t mask2;
    FastDiv by_seq, by_heads;  // items of a sequence (heads * blocks), heads
};

// codes k and k + 1 of a word as fp16 values
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t fp16_pair(uint32_t w, int k, float mn0, float st0, float mn1, float st1) {
    const float p0 = (float)((w >> (8 * k)) & 0xffu) * st0, p1 = (float)((w >> (8 * k + 8)) & 0xffu) * st1;
    const v2h v = {(_Float16)(mn0 + p0), (_Float16)(mn1 + p1)};  // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}

// the buffered fp16 tokens follow the blocks: token r of the buffer (oldest first) sits in slot
// (res_head + r) mod res_tokens of the ring.  `part` of `parts` workgroups copies its share.
__device__ __forceinline__ void copy_buffered(const DecompArgs &a, int part, int parts) {
    const Geo &g = a.g;
    const size_t res_tensor = (size_t)g.B * g.res_tokens * g.H * kD;
    const size_t per_tok = (size_t)g.H * kD / 8;  // 16-byte units
    const size_t per_b = (size_t)a.n_res * per_tok;
    const size_t n16 = (size_t)g.B * per_b;
    for (size_t i = (size_t)part * blockDim.x + threadIdx.x; i < n16; i += (size_t)parts * blockDim.x) {
        const size_t b = i / per_b, rem = i - b * per_b;  // rem indexes [r][h][c/8]
        const size_t r = rem / per_tok, in_tok = rem - r * per_tok;
        size_t slot = (size_t)a.res_head + r;
        if (slot >= (size_t)g.res_tokens) slot -= (size_t)g.res_tokens;
        const uint4 v = reinterpret_cast<const uint4 *>(g.res + a.which * res_tensor +
                                                        (b * g.res_tokens + slot) * g.H * kD)[in_tok];
        reinterpret_cast<uint4 *>(a.out + ((size_t)b * a.seq_stride + (size_t)a.n_blocks * kBT) * g.H * kD)[rem] = v;
    }
}

// What a wave needs of its block: decided once per wave, false if there is nothing to do.
struct BlockOfWave {
    uint16_t *dst;       // first element of the block's first row in the output
    const uint8_t *rec;
    uint32_t size16;
    __device__ __forceinline__ bool find(const DecompArgs &a, int wave, int lane) {
        const Geo &g = a.g;
        const uint32_t item = blockIdx.x * kDecWaves + wave, per_b = (uint32_t)(g.H * a.n_blocks);
        if (item >= (uint32_t)g.B * per_b) return false;
        // items are numbered (batch, block, head), head fastest: the rows that neighbouring waves write are neighbours in
        // memory (a token's row holds all heads)
        const uint32_t b = a.by_seq(item), rest = item - b * per_b;
        const uint32_t j = a.by_heads(rest), h = rest - j * g.H;
        const BlockEntry e = g.table[((size_t)a.which * g.B * g.H + (size_t)b * g.H + h) * g.max_blocks + j];
        size16 = __builtin_amdgcn_readfirstlane(e.size16);
        rec = g.payload + (size_t)(uint32_t)__builtin_amdgcn_readfirstlane(e.off16) * 16;
        dst = a.out + (((size_t)b * a.seq_stride + (size_t)j * kBT) * g.H + h) * kD;
        // A record larger than the staging area (the host sizes it from the largest record, so only a corrupted table gets
        // here) is not decoded: its block is NaN, so that it cannot pass for data, and the next synchronising call, or the
        // next decompression that is queued once this one has run, fails.
        if (size16 > (uint32_t)(a.stage_bytes - kStreamSlack) / 16) {  // stage_bytes is at least kStreamSlack
            if (lane == 0) {
                atomicOr(&g.ctrl->fault, kFaultStageSmall);
                __hip_atomic_store(a.host_refused, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            for (int t = lane >> 4; t < kBT; t += 4)
                *reinterpret_cast<uint4 *>(dst + (size_t)t * g.H * kD + 8 * (lane & 15)) = make_uint4(~0u, ~0u, ~0u, ~0u);
            return false;
        }
        return true;
    }
};

// Table decoder compiled for code words of up to LB bits (LB >= 7; shorter ones take the 7-bit build).  The whole block's
// codes wait in 32 registers of a lane, four to a register, and then go through LDS -- over the record, which is not
// needed any more -- as rows of a token's 128 codes, to be stored as four whole 256-byte rows per instruction.  K: a lane
// decodes a token's row; V: two channels, whose words of four tokens become words of four channels of a token by a 4 x 4 byte
// transposition inside each quad of lanes.  (V stored from there, 128-byte pieces of 8 bytes a lane: 50 instead of 40 us.)
// Sixteen waves of four-wave workgroups fit a CU; with a code tile beside the record, which the decoder filled byte by
// byte, eight did: 32 heads x 15000 tokens, 48 MB in and 123 MB out, 61 -> 38 us (K) and
// 40 us (V): 4.5 and 4.3 TB/s, 92 and 88 % of what a large copy reaches.
constexpr int kDecRow = kD + 16;  // row of the code tile: 16-byte accesses of neighbouring rows start in different banks
template <int WHICH, int LB>
__global__ __launch_bounds__(64 * kDecWaves, 4) void decompress_kernel(DecompArgs a) {
    using M = DecodeMode<LB>;
    static_assert(!M::kPair, "single-symbol table");
    __shared__ __attribute__((aligned(16))) uint8_t lut_s[M::kTableBytes];
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // per wave: the record, then the code tile
    const Geo &g = a.g;
    const int n_wg = (g.B * g.H * a.n_blocks + kDecWaves - 1) / kDecWaves;
    if ((int)blockIdx.x >= n_wg) {  // the workgroups behind the blocks' copy the buffered tokens
        copy_buffered(a, (int)blockIdx.x - n_wg, (int)gridDim.x - n_wg);
        return;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    uint8_t *stage = smem + (size_t)wave * a.area_bytes;
    BlockOfWave blk;
    const bool busy = blk.find(a, wave, lane);
    for (int c = wave; 1024 * c < M::kTableBytes; c += kDecWaves)
        if (1024 * c + 16 * lane < M::kTableBytes)
            load_lds16(reinterpret_cast<const uint4 *>(lut_of(g, WHICH)) + 64 * c + lane, lut_s + 1024 * c);
    if (busy) stage_record(blk.rec, blk.size16, stage, lane);
    wait_record();
    __syncthreads();
    if (!busy) return;
    const uint32_t *hdr32 = reinterpret_cast<const uint32_t *>(stage);
    const char *lut = reinterpret_cast<const char *>(lut_s);
    SliceWords pw;
    Quad<M::J> qd;
    const float two_eb = g.two_eb[WHICH];
    // stores: instruction i covers tokens 4 i + lane / 16, channels 8 (lane % 16) .. + 7 (four rows)
    const int c0 = (lane & 15) * 8, sub = lane >> 4;
    uint32_t mm[WHICH == 0 ? 8 : 16];  // K: {min,max} of the lane's channels; V: of its tokens
    if constexpr (WHICH == 0) {
#pragma unroll
        for (int k = 0; k < 8; k++) mm[k] = hdr32[g.k_units == 1 ? 0 : c0 + k];
        const uint32_t sb = hdr32[g.k_minmax_bytes / 4 + lane];
        const uint32_t start = wave_excl_scan((sb & 0xffffu) + (sb >> 16), lane);
        const Unit *units = payload_units(hdr32 + (g.k_minmax_bytes + 2 * kSlices) / 4);
        qd.open(units, start, sb & 0xffffu, sb >> 16);
        decode_block<LB>(qd, units, lut, a.mask2, pw);
        wave_sync();  // every lane is done with the record
        uint4 *mine = reinterpret_cast<uint4 *>(stage + lane * kDecRow);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            mine[i] = make_uint4(pw.a[4 * i], pw.a[4 * i + 1], pw.a[4 * i + 2], pw.a[4 * i + 3]);
            mine[4 + i] = make_uint4(pw.b[4 * i], pw.b[4 * i + 1], pw.b[4 * i + 2], pw.b[4 * i + 3]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; i++) mm[i] = hdr32[4 * i + sub];
        const uint16_t *bits16 = reinterpret_cast<const uint16_t *>(hdr32 + kMinMaxBytesV / 4);
        const uint32_t abits = bits16[lane], bbits = bits16[kSliceLen + lane];  // slices: channels lane and 64 + lane
        const uint32_t start_a = wave_excl_scan(abits, lane);
        const uint32_t start_b = (uint32_t)__builtin_amdgcn_readlane((int)(start_a + abits), 63) + wave_excl_scan(bbits, lane);
        const Unit *units = payload_units(hdr32 + kHdrBytesV / 4);
        qd.open2(units, start_a, abits, start_b, bbits);
        decode_block<LB>(qd, units, lut, a.mask2, pw);
        wave_sync();
        const QuadTranspose transpose(lane);
        uint8_t *mine = stage + (lane & 3) * kDecRow + (lane & ~3);
#pragma unroll
        for (int w = 0; w < 16; w++) {  // token 4 w + lane % 4, channels 4 (lane / 4) .. +3 and the same plus 64
            *reinterpret_cast<uint32_t *>(mine + 4 * w * kDecRow) = transpose(pw.a[w]);
            *reinterpret_cast<uint32_t *>(mine + 4 * w * kDecRow + kSliceLen) = transpose(pw.b[w]);
        }
    }
    wave_sync();
    float mn[8], st[8];
    auto range = [&](int k, uint32_t v) {
        mn[k] = h2f(v & 0xffffu);
        st[k] = two_eb * (h2f(v >> 16) - mn[k]);
    };
    if constexpr (WHICH == 0) {
#pragma unroll
        for (int k = 0; k < 8; k++) range(k, mm[k]);
    }
    const uint32_t row_bytes = (uint32_t)g.H * kD * 2, at = (uint32_t)sub * row_bytes + 2 * c0;  // uniform base + lane offset
    char *dst = reinterpret_cast<char *>(blk.dst);
#pragma unroll
    for (int i = 0; i < 16; i++) {
        if constexpr (WHICH == 1) {
            range(0, mm[i]);
#pragma unroll
            for (int k = 1; k < 8; k++) { mn[k] = mn[0]; st[k] = st[0]; }
        }
        const int t = 4 * i + sub;
        const uint2 w = *reinterpret_cast<const uint2 *>(stage + t * kDecRow + c0);
        uint4 o;
        o.x = fp16_pair(w.x, 0, mn[0], st[0], mn[1], st[1]);
        o.y = fp16_pair(w.x, 2, mn[2], st[2], mn[3], st[3]);
        o.z = fp16_pair(w.y, 0, mn[4], st[4], mn[5], st[5]);
        o.w = fp16_pair(w.y, 2, mn[6], st[6], mn[7], st[7]);
        *reinterpret_cast<uint4 *>(dst + (size_t)(4 * i) * row_bytes + at) = o;
    }
}

// ---- the paper's bit-serial decoder, kept for an A/B on this hardware ----------------------------------------------
constexpr int kTreeRow = kD + 8;  // padded row of the code tile (bytes; keeps 8-byte reads aligned)
__global__ __launch_bounds__(64 * kDecWaves) void tree_walk_kernel(DecompArgs a) {
    __shared__ __attribute__((aligned(16))) uint16_t tree_s[512];
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];  // per wave: the record, then the code tile
    const Geo &g = a.g;
    const int n_wg = (g.B * g.H * a.n_blocks + kDecWaves - 1) / kDecWaves;
    if ((int)blockIdx.x >= n_wg) {
        copy_buffered(a, (int)blockIdx.x - n_wg, (int)gridDim.x - n_wg);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), which = a.which;
    {  // the tree of this tensor: 256 nodes x 2 children, 16 bits each
        const uint4 *src = reinterpret_cast<const uint4 *>(tree_of(g, which));
        for (int i = tid; i < 64; i += 64 * kDecWaves) reinterpret_cast<uint4 *>(tree_s)[i] = src[i];
    }
    uint8_t *stage = smem + (size_t)wave * a.area_bytes, *tile = stage + a.stage_bytes;
    BlockOfWave blk;
    const bool busy = blk.find(a, wave, lane);
    if (busy) stage_record(blk.rec, blk.size16, stage, lane);
    wait_record();
    __syncthreads();
    if (!busy) return;
    const uint32_t *hdr32 = reinterpret_cast<const uint32_t *>(stage);
    const int mmb = which == 0 ? g.k_minmax_bytes : kMinMaxBytesV;
    const uint32_t sb = hdr32[mmb / 4 + lane];
    const uint32_t start = wave_excl_scan((sb & 0xffffu) + (sb >> 16), lane);
    const Unit *units = payload_units(hdr32 + (mmb + 2 * kSlices) / 4);
    // K: lane = token, chains 0 and 1 = channels 0..63 (up / down), 2 and 3 = channels 64..127
    // V: lane = channels 2*lane (chains 0 and 1) and 2*lane+1, symbol index = token
    walk_chains(units, reinterpret_cast<const int16_t *>(tree_s), start, sb & 0xffffu, sb >> 16,
                [&](int c, int sym, int idx) {  // chain c emitted its idx-th symbol
                    if (sym < 0) return;
                    const int pos = (c & 1) ? kSliceLen - 1 - idx : idx;  // chains 1 and 3 read downwards
                    if (which == 0) tile[lane * kTreeRow + (c >> 1) * kSliceLen + pos] = (uint8_t)sym;
                    else tile[pos * kTreeRow + 2 * lane + (c >> 1)] = (uint8_t)sym;
                },
                [](bool mine) { return __any(mine) != 0; });
    wave_sync();
    // dequantize and write: instruction i covers tokens 4 i + lane / 16, channels 8 (lane % 16) .. + 7 (four rows)
    const int c0 = (lane & 15) * 8, sub = lane >> 4;
    const float two_eb = g.two_eb[which];
#pragma unroll 1
    for (int i = 0; i < 16; i++) {
        const int t = 4 * i + sub;
        const uint2 w = *reinterpret_cast<const uint2 *>(tile + t * kTreeRow + c0);
        float mn[8], st[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t mm = hdr32[which == 1 ? t : g.k_units == 1 ? 0 : c0 + k];
            mn[k] = h2f(mm & 0xffffu);
            st[k] = two_eb * (h2f(mm >> 16) - mn[k]);
        }
        uint4 o;
        o.x = fp16_pair(w.x, 0, mn[0], st[0], mn[1], st[1]);
        o.y = fp16_pair(w.x, 2, mn[2], st[2], mn[3], st[3]);
        o.z = fp16_pair(w.y, 0, mn[4], st[4], mn[5], st[5]);
        o.w = fp16_pair(w.y, 2, mn[6], st[6], mn[7], st[7]);
        *reinterpret_cast<uint4 *>(blk.dst + (size_t)t * g.H * kD + c0) = o;
    }
}

static hipError_t launch_dec(void (*kernel)(DecompArgs), size_t &attr_set, const DecompArgs &a, size_t lds, int grid, hipStream_t s) {
    if (lds > attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = lds;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * kDecWaves), lds, s, a);
    return hipGetLastError();
}
template <int LB>
static hipError_t launch_dec_lb(const DecompArgs &a, size_t lds, int grid, hipStream_t s) {
    static size_t attr_set[2] = {0, 0};
    return a.which == 0 ? launch_dec(decompress_kernel<0, LB>, attr_set[0], a, lds, grid, s)
                        : launch_dec(decompress_kernel<1, LB>, attr_set[1], a, lds, grid, s);
}

hipError_t launch_decompress(const Geo &g, int which, uint16_t *out, int n_blocks, int res_head, int n_res, int seq_stride,
                             int stage_bytes, int tree_walk, uint32_t *host_refused, hipStream_t s) {
    DecompArgs a;
    a.g = g;
    a.out = out;
    a.which = which;
    a.n_blocks = n_blocks;
    a.seq_stride = seq_stride;
    a.stage_bytes = stage_bytes;
    a.res_head = res_head;
    a.n_res = n_res;
    a.host_refused = host_refused;
    const int bits = g.lut_bits[which];
    if (bits < 1 || bits > kLutBits) return hipErrorInvalidValue;
    a.mask2 = ((1u << bits) - 1u) << 1;
    a.area_bytes = tree_walk ? stage_bytes + kBT * kTreeRow : stage_bytes < kBT * kDecRow ? kBT * kDecRow : stage_bytes;
    const size_t lds = (size_t)kDecWaves * a.area_bytes;
    const long long items = (long long)g.B * g.H * n_blocks;  // at most 2^28 (checked when the context is created)
    a.by_seq.set((uint32_t)(g.H * (n_blocks > 0 ? n_blocks : 1)));
    a.by_heads.set((uint32_t)g.H);
    // the buffered tokens: one workgroup for every 4 KiB, at most 64
    const long long tail16 = (long long)g.B * n_res * g.H * (kD / 8);
    const long long tail = tail16 / 256 > 63 ? 64 : (tail16 + 255) / 256;
    const int grid = (int)((items + kDecWaves - 1) / kDecWaves + tail);
    if (grid == 0) return hipSuccess;
    static size_t tree_attr = 0;
    if (tree_walk) return launch_dec(tree_walk_kernel, tree_attr, a, lds, grid, s);
    switch (fused_table_bits(bits)) {
        case 6:
        case 7: return launch_dec_lb<7>(a, lds, grid, s);
        case 8: return launch_dec_lb<8>(a, lds, grid, s);
        case 10: return launch_dec_lb<10>(a, lds, grid, s);
        default: return launch_dec_lb<12>(a, lds, grid, s);
    }
}

}  // namespace kvc
