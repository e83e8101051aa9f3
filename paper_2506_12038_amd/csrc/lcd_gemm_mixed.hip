// Prefill of a group whose layers take different kernels (gfx950): the large tiles and the split kernel's tiles in ONE
// launch.  Both kinds have workgroups of 512 threads that fill a compute unit; every XCD's queue holds the large tiles
// first (the longest), so that the compute units their last round leaves idle start on the others.  One launch after the other, each
// leaves its own last round behind: q 4096, k and v 1024 rows, K = 4096, 3 bits, 1100 tokens (144 large tiles on 256 compute units,
// then 288 split ones): 95 us, in one launch 72.  q 8192, k and v 1024 rows, K = 8192: 700 tokens 147 -> 128, 1100 tokens 235 -> 196.
// The tiles are those of the two kernels, so a layer's bits do not depend on its neighbours.
#include <hip/hip_runtime.h>
#include "lcd_gemm_large.h"
#include "lcd_gemm_split.h"

namespace lcd {

template <int BITS, int TBLK>
__global__ void __launch_bounds__(kGemmWaves * 64, 1) gemm_mixed_kernel(const GemmBatch large, const GemmBatch split, const uint32_t large_blocks)
{
    static_assert(kGemmWaves == kSplitWaves, "one workgroup size");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    if (blockIdx.x < large_blocks) gemm_workgroup<BITS>(large, blockIdx.x, lds);      // (large_blocks is a multiple of the XCDs)
    else split_workgroup<BITS, 2, TBLK>(split, blockIdx.x - large_blocks, lds);
}

template <int BITS, int TBLK>
static SplitVariant variant_of()
{
    constexpr size_t split = split_lds_bytes<2, TBLK>(), large = 2 * kStageBytes;
    return SplitVariant{(const void *)gemm_mixed_kernel<BITS, TBLK>, split > large ? split : large, (BITS - 2) * 2 + TBLK - 3};
}

SplitVariant mixed_variant(int bits, int blocks)
{
    if (blocks <= 3) return bits == 2 ? variant_of<2, 3>() : bits == 3 ? variant_of<3, 3>() : variant_of<4, 3>();
    return bits == 2 ? variant_of<2, 4>() : bits == 3 ? variant_of<3, 4>() : variant_of<4, 4>();
}

}  // namespace lcd
