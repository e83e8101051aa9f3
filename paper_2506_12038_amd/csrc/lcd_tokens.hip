// The tokens kernel (lcd_tokens.h) for layers of one index width.
#include <hip/hip_runtime.h>
#include "lcd_tokens.h"

namespace lcd {

template <int BITS, int TB, int R, int WAVES, int PAIRS, bool READY, bool RESIDENT>
__global__ void __launch_bounds__(WAVES * 64, 1) gemv_tokens_kernel(const uint32_t t0, const uint32_t t1, const uint32_t t2, const uint32_t t3,
                                                                   const uint32_t t4, const uint32_t t5, const uint32_t t6, const uint32_t t7,
                                                                   const uint16_t *head_x, const float *head_s, const uint32_t head_word, const BucketBatch batch)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    tokens_workgroup<BITS, TB, R, WAVES, PAIRS, READY, RESIDENT>(t0, t1, t2, t3, t4, t5, t6, t7, head_x, head_s, head_word, batch, smem);
}

constexpr int kAnyTiles = 1 << 24;     // (more than any layer has)
template <int BITS, int TB, int R, int WAVES, int PAIRS, bool READY, bool RESIDENT = false>
static TokensVariant variant_of(int slot)
{
    return TokensVariant{(const void *)gemv_tokens_kernel<BITS, TB, R, WAVES, PAIRS, READY, RESIDENT>, RESIDENT ? kAnyTiles : R, WAVES, tokens_lds_bytes<BITS, TB, R, WAVES, PAIRS, READY>(),
                         (((BITS - 2) * kMaxTokenBlocks + (TB - 1)) * 4 + (READY ? 3 : PAIRS == 2 ? 0 : PAIRS == 4 ? 1 : 2)) * 10 + slot};
}

template <int BITS, int TB, int PAIRS, bool READY>
static TokensVariant pick_tiles(int tiles, int kc)   // (of 16 waves those that do not spill)
{
    if (tiles <= 1) return variant_of<BITS, TB, 1, 2 * kBW, PAIRS, READY>(0);
    // Two row tiles of 4 bits, 9 to 16 tokens made in the kernel: 8 waves, or the resident form where most of 16 waves have a chunk.
    // 8192 rows, 16 waves (spilled) / 8 / resident, 9 and 16 tokens, us: K = 2048 7.2 6.6 7.2, 7.5 6.9 7.7; 3072 8.5 7.7 7.9, 8.9 7.9 8.4;
    // 4096 9.8 9.5 8.7, 10.3 10.1 9.3; 5120 11.0 10.5, 11.8 11.0; 7936 15.3 15.2, 16.4 16.2.
    constexpr bool spills = BITS == 4 && TB == 1 && PAIRS == 8 && !READY;
    if (tiles <= 2 && !(spills && kc > 12 && kc <= 2 * kBW)) return variant_of<BITS, TB, 2, TB == 1 && !spills ? 2 * kBW : kBW, PAIRS, READY>(1);
    if constexpr (TB == 1) {
        if (kc <= 2 * kBW) return variant_of<BITS, 1, 3, 2 * kBW, PAIRS, READY, true>(5);
        if constexpr (BITS == 2 || (BITS == 3 && (READY || PAIRS < 8))) if (tiles == 3) return variant_of<BITS, 1, 3, 2 * kBW, PAIRS, READY>(2);
    }
    if (tiles <= 3) return variant_of<BITS, TB, 3, kBW, PAIRS, READY>(6);
    constexpr int whole = whole_chunk_tiles<BITS, TB>();
    if constexpr (BITS == 2 && TB == 1 && PAIRS == 8 && !READY) {
        if (tiles == 4) return variant_of<BITS, 1, 4, kBW, PAIRS, READY>(8);
        if (tiles == 5) return variant_of<BITS, 1, 5, kBW, PAIRS, READY>(9);
    }
    if (TB > 1 || tiles <= whole) return variant_of<BITS, TB, whole, kBW, PAIRS, READY>(3);
    if constexpr (BITS == 2 && PAIRS == 8 && !READY) if ((tiles + 11) / 12 == (tiles + 13) / 14) return variant_of<BITS, 1, 12, kBW, PAIRS, READY>(7);
    return variant_of<BITS, 1, kManyTiles, kBW, PAIRS, READY>(4);
}

template <int BITS>
static TokensVariant pick(int tokens, int tiles, int kc, bool ready)
{
    if (tokens > kTokenBlock) return ready ? pick_tiles<BITS, 2, 8, true>(tiles, kc) : pick_tiles<BITS, 2, 8, false>(tiles, kc);
    if (ready) return pick_tiles<BITS, 1, 8, true>(tiles, kc);
    return tokens <= 4 ? pick_tiles<BITS, 1, 2, false>(tiles, kc) : tokens <= 8 ? pick_tiles<BITS, 1, 4, false>(tiles, kc) : pick_tiles<BITS, 1, 8, false>(tiles, kc);
}

TokensVariant tokens_variant(int bits, int tokens, int tiles, int kc, bool ready)
{
    return bits == 2 ? pick<2>(tokens, tiles, kc, ready) : bits == 3 ? pick<3>(tokens, tiles, kc, ready) : pick<4>(tokens, tiles, kc, ready);
}

}  // namespace lcd
