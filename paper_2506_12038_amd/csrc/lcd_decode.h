// What the two decode kernels (lcd_bucket.hip, lcd_tokens.h) and their launcher share.
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
    int wg_first;                 // first workgroup of this layer
};
// What a workgroup needs first travels as leading kernel arguments: those are preloaded into scalar registers when a wave
// starts, while a read of the argument segment takes 0.6 us (measured from a wave's entry).  The first eight words are the
// table of first workgroups (wg_begin[1..16], 16 bits each), from which a workgroup finds its layer, or, in a launch of
// a single layer, the layer itself (see part_of).  Then x, s and DecodeHead::word for layers that all read one input
// (q, k, v or gate, up of a decoder block, and every single layer): the activations, which start the longest chain, are asked for
// without waiting for the layer's record.
// Measured, 7B blocks: 2 bits, 16 tokens 39.4 -> 38.4 us; 4 tokens of INT8 codes 32.4 -> 31.5; 3 bits, one token 34.6 -> 33.9.
struct DecodeHead {
    const uint16_t *x;   // input of all layers (shared)
    const float *s;
    uint32_t word;       // bits 0..21 K / 256, 22..27 tokens, then the flags
};
constexpr uint32_t kHeadShared = 1u << 28, kHeadSingle = 1u << 29;
__device__ __forceinline__ int head_kc(uint32_t word) { return (int)(word & 0x3fffffu); }
__device__ __forceinline__ int head_tokens(uint32_t word) { return (int)((word >> 22) & 63u); }

// The narrow kernel has more tokens and narrower inputs: its word holds K / 256 in bits 0..18 and the tokens in bits 19..27.
constexpr uint32_t kNarrowTokensShift = 19, kNarrowTokensMask = 0x1ff;

// Number of table entries <= b, for b < 2^15 - 1:
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
};
// A launch of one layer: the argument segment is written across the bus, 1.4 us of host time per KiB.
struct SingleBatch {
    BucketProblem p[1];
};

// The input a workgroup's layer reads: from the leading arguments if the layers share it, else from the record.  (The
// empty assembly statements keep the branches: as selects they would wait for the record on every path.)
template <class BATCH>
__device__ __forceinline__ void input_of(const BATCH &batch, int pi, uint32_t word, const uint16_t *&x, const float *&s, int &kc)
{
    kc = head_kc(word);
    if (!(word & kHeadShared)) {
        x = batch.p[pi].x;
        s = batch.p[pi].s;
        kc = batch.p[pi].kc;
        asm volatile("" : "+s"(x), "+s"(s), "+s"(kc));
    }
}
// The rest of the layer: row tiles [ta, tb) are the workgroup's.
struct LayerPart { const uint8_t *packed; const float *lut; int nt, ta, tb; };
template <class BATCH>
__device__ __forceinline__ LayerPart part_of(const BATCH &batch, int pi, uint32_t word, uint32_t b, uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3,
                                             uint32_t t4, uint32_t t5, uint32_t t6)
{
    LayerPart l;
    int li, base, extra;
    if (word & kHeadSingle) {
        l.packed = reinterpret_cast<const uint8_t *>((uint64_t)t1 << 32 | t0);
        l.lut = reinterpret_cast<const float *>((uint64_t)t3 << 32 | t2);
        l.nt = (int)t4; base = (int)t5; extra = (int)t6; li = (int)b;
        asm volatile("" : "+s"(l.packed), "+s"(l.lut), "+s"(l.nt), "+s"(base), "+s"(extra));
    } else {
        l.packed = batch.p[pi].packed; l.lut = batch.p[pi].lutA;
        l.nt = batch.p[pi].nt; base = batch.p[pi].tiles_base; extra = batch.p[pi].tiles_extra; li = (int)b - batch.p[pi].wg_first;
        asm volatile("" : "+s"(l.packed), "+s"(l.lut), "+s"(l.nt), "+s"(base), "+s"(extra), "+s"(li));
    }
    l.ta = li * base + min(li, extra);
    l.tb = l.ta + base + (li < extra ? 1 : 0);
    return l;
}

// ---- bucket kernel (lcd_bucket.hip) ---------------------------------------------------------------
struct BucketVariant {
    const void *fn, *single;   // kernels for a group and for one layer (SingleBatch)
    int tiles;          // row tiles it holds at a time
    int waves;          // waves of its workgroups
    size_t lds_bytes;
    int id;             // 0 .. kBucketVariants - 1, of the two kernels 2 id and 2 id + 1
};
constexpr int kBucketVariants = 72;
// tokens: 1 (2 and 3 bits), 2 (2 bits), 3 and 4 (2 bits, INT8 codes)
// pass: place in kBucketPass; tiles: most row tiles of a workgroup; kc: chunks of the widest layer
BucketVariant bucket_variant(int bits, int tokens, bool int8_codes, int pass, int tiles, int kc);

// Partial tiles in LDS (tokens and narrow kernel): where row quad q of token j of a tile stands, in floats; r: the tile's row tile in the pass.
// 16 lanes that write (one q, all j) and 16 that read (the quads of one token, row tile after row tile) each cover all banks; in
// plain [token][row] order both met in a quarter of them.  7B block, 3 bits, 40 tokens 58.9 -> 58.1 us; blocks of mixed widths, six tokens
// 214.5 -> 211.7 (four blocks).
__device__ __forceinline__ int partial_quad(int r, int q, int j) { return 4 * ((4 * j + (q ^ (j >> 2))) ^ ((r & 3) << 2)); }

// What a lane of the tokens and the narrow kernel holds of a (tile, chunk) and of a row.
template <int BITS>
struct PackedTile {
    uint4v lo;
    uint2v hi;     // 3 bits: the third-bit words
    uint4v hi4;    // 4 bits: the second plane
};
template <int BITS> struct TablesOf { typedef RowTables type; };
template <> struct TablesOf<4> { typedef RowTables4 type; };
template <int BITS> constexpr int row_table_bytes() { return BITS == 2 ? 8 : BITS == 3 ? 16 : 32; }

// ---- tokens kernel (lcd_tokens.h) ---------------------------------------------------------------
constexpr int kTokenBlock = 16;      // tokens per block of the tokens kernel (the columns of one matrix instruction)
constexpr int kMaxTokenBlocks = 2;   // blocks it holds in registers: up to 32 tokens

// A variant for `tokens` tokens that holds up to `tiles` row tiles at a time, or the one that holds
// the most if none holds that many.
struct TokensVariant {
    const void *fn;
    int tiles;          // row tiles it holds at a time
    int waves;          // waves of its workgroups
    size_t lds_bytes;
    int id;             // 0 .. kTokensVariants - 1
};
constexpr int kTokensVariants = 3 * kMaxTokenBlocks * 4 * 10;
// ready: x holds the transformed activations in operand order (transform_kernel)
TokensVariant tokens_variant(int bits, int tokens, int tiles, int kc, bool ready);
// the narrow kernel (lcd_narrow.hip), 17 .. 16 kNarrowBlocks tokens; ids of their own
constexpr int kNarrowBlocks = 6;
constexpr int kNarrowVariants = 3 * kNarrowBlocks * 4;
TokensVariant narrow_variant(int bits, int tokens, int tiles);
// for layers of several widths, up to 16 tokens (lcd_tokens_mixed.hip); ids of their own
constexpr int kMixedTokensVariants = 15;
TokensVariant tokens_mixed_variant(int tokens, int tiles, int kc);

}  // namespace lcd
