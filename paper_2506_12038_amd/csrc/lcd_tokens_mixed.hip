// The tokens kernel (lcd_tokens.h) for a group of layers with index widths of their own, up to 16 tokens: a workgroup runs the
// code of its layer's width.  One launch instead of one per width: each has its start-up, its gap in front and a tail in which most
// compute units wait for a few.  q, k, v (5120 x 5120, widths 3, 3, 2), six tokens 17.7 -> 11.9 us in a graph; gate, up (13824 x 5120, 2, 3) 20.8 -> 16.2.
// The layers are in descending order of their widths, so that two numbers in the leading (preloaded) arguments tell a workgroup its width.
#include <hip/hip_runtime.h>
#include "lcd_tokens.h"

namespace lcd {

template <int R> constexpr int tiles_of_width(int bits) { return R == 6 && bits == 4 ? 4 : R; }   // (6: as many as leave room for their words of a chunk)

template <int R, int WAVES, int PAIRS, bool RESIDENT>
__global__ void __launch_bounds__(WAVES * 64, 1) gemv_tokens_mixed_kernel(const uint32_t t0, const uint32_t t1, const uint32_t t2, const uint32_t t3,
                                                                         const uint32_t t4, const uint32_t t5, const uint32_t t6, const uint32_t t7,
                                                                         const uint16_t *head_x, const float *head_s, const uint32_t head_word,
                                                                         const uint32_t widths, const BucketBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const uint32_t b = blockIdx.x;       // widths: first workgroup of the 3-bit layers, and (upper half) of the 2-bit layers
    if (b < (widths & 0xffffu)) tokens_workgroup<4, 1, tiles_of_width<R>(4), WAVES, PAIRS, false, RESIDENT>(t0, t1, t2, t3, t4, t5, t6, t7, head_x, head_s, head_word, batch, smem);
    else if (b < widths >> 16) tokens_workgroup<3, 1, R, WAVES, PAIRS, false, RESIDENT>(t0, t1, t2, t3, t4, t5, t6, t7, head_x, head_s, head_word, batch, smem);
    else tokens_workgroup<2, 1, R, WAVES, PAIRS, false, RESIDENT>(t0, t1, t2, t3, t4, t5, t6, t7, head_x, head_s, head_word, batch, smem);
}

template <int R, int WAVES, int PAIRS, bool RESIDENT = false>
static TokensVariant variant_of(int slot)
{
    return TokensVariant{(const void *)gemv_tokens_mixed_kernel<R, WAVES, PAIRS, RESIDENT>, R, WAVES, tokens_lds_bytes<4, 1, R, WAVES, PAIRS, false>(),
                         slot * 3 + (PAIRS == 2 ? 0 : PAIRS == 4 ? 1 : 2)};
}

template <int PAIRS>
static TokensVariant pick(int tiles, int kc)
{
    if (tiles <= 1) return variant_of<1, 2 * kBW, PAIRS>(0);
    // (9 to 16 tokens: the 4-bit part spills 12 registers, which costs less than 8 waves do the others: 4096 rows of 3 and of 2 bits, K = 13824,
    // 9 tokens 15.8 us, with 8 waves 17.0; 6144 rows of 4 and 2048 of 3 bits the same with either, K = 5120 11.0, 13824 24.4)
    if (tiles <= 2) return variant_of<2, 2 * kBW, PAIRS>(1);
    if (kc <= 2 * kBW) return variant_of<3, 2 * kBW, PAIRS, true>(2);
    return tiles <= whole_chunk_tiles<3, 1>() ? variant_of<whole_chunk_tiles<3, 1>(), kBW, PAIRS>(3) : variant_of<kManyTiles, kBW, PAIRS>(4);
}

TokensVariant tokens_mixed_variant(int tokens, int tiles, int kc)
{
    return tokens <= 4 ? pick<2>(tiles, kc) : tokens <= 8 ? pick<4>(tiles, kc) : pick<8>(tiles, kc);
}

}  // namespace lcd
