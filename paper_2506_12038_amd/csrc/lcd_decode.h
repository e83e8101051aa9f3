// What the two decode kernels (lcd_gemv.hip, lcd_tokens.hip) and their launcher share.
#pragma once
#include <hip/hip_runtime.h>
#include "lcd_internal.h"
#include "lcd_device.h"

namespace lcd {

// Cache policy of the packed-index loads: non-temporal.  Every index byte is read exactly once per
// launch, and without the hint the stream pushes the small reused data (activations, smoothing
// factors, codebook tables) out of the caches: measured +4 % (7B set, 3 bits) to +8 % (70B MLP, 2
// bits) on the single-token kernel, +3.5 % on the tokens kernel.  (Bit 1 of the buffer
// instructions' cache-policy operand is "nt" on gfx950.)
constexpr int kStreamPolicy = 2;

// Buffer resources give branch-free predication: a lane whose offset is past the end of the
// buffer reads zeros and touches no memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
constexpr uint32_t kOob = 0xFFFFFFF0u;

constexpr int kBW = 8;            // waves per workgroup

struct BucketProblem {
    const uint8_t *packed;
    const float *lutA;
    const uint16_t *x;
    const float *s;
    uint16_t *y;
    int nt, kc;
    int tiles_base, tiles_extra;  // workgroup i of this layer owns tiles_base (+1 if i < tiles_extra) row tiles
    float act_scale;              // 0: fp16 activations x/s; s_q > 0: INT8 codes of Sec. 4.1, output scaled by s_q
    int x_ready;                  // tokens kernel: x already holds the smoothed activations / the codes (transform_kernel)
    int wg_first;                 // first workgroup of this layer
};
// The table of first workgroups (wg_begin[1..16], 16 bits each) also travels as eight leading scalar
// kernel arguments: those are preloaded into scalar registers when a wave starts, so a workgroup
// knows its layer without a load and the problem record is the only load between the kernel's
// entry and its first index loads.  Number of table entries <= b, for b < 2^15 - 1:
struct WgTable { uint32_t t[kMaxGroup / 2]; };
__device__ __forceinline__ int layer_of_workgroup(uint32_t b, uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3,
                                                  uint32_t t4, uint32_t t5, uint32_t t6, uint32_t t7)
{
    // per 16-bit field f: bit 15 of (0x8000 + f) - (b + 1) is clear exactly when f <= b (no borrow crosses a field)
    const uint32_t bb = (b + 1u) * 0x00010001u, top = 0x80008000u;
    const uint32_t t[8] = {t0, t1, t2, t3, t4, t5, t6, t7};
    int n = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) n += __builtin_popcount(~((t[i] | top) - bb) & top);
    return n;
}
struct BucketBatch {
    BucketProblem p[kMaxGroup];
    int count;
};

// ---- tokens kernel (lcd_tokens.hip) ---------------------------------------------------------------
constexpr int kTokenBlock = 16;      // tokens per block of the tokens kernel (the columns of one matrix instruction)
constexpr int kMaxTokenBlocks = 2;   // blocks it holds in registers: up to 32 tokens

// A variant for `blocks` token blocks that holds up to `tiles` row tiles at a time, or the one that holds
// the most if none holds that many.
struct TokensVariant {
    const void *fn;
    int tiles;          // row tiles it holds at a time
    int waves;          // waves of its workgroups
    size_t lds_bytes;
    int id;             // 0 .. kTokensVariants - 1
};
constexpr int kTokensVariants = 3 * kMaxTokenBlocks * 4;
TokensVariant tokens_variant(int bits, int blocks, int tiles);

}  // namespace lcd
