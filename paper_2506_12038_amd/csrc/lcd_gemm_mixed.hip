// Prefill of a group whose layers take different kernels (gfx950): the wide kernel's tiles (in halves) and the split kernel's in ONE
// launch.  Both kinds have workgroups of 512 threads that fill a compute unit; every XCD's queue holds the wide tiles
// first (the longest), so that the compute units their last round leaves idle start on the others.  One launch after the other, each
// leaves its own last round behind: q 4096, k and v 1024 rows, K = 4096, 3 bits, 1100 tokens 76.8 us, in one launch 67.3; q 8192, k and v 1024 rows,
// K = 8192, 3 bits, 700 tokens 125.4, in one launch 115.2.  When calls take it: plan_launches in lcd_gemm_plan.h.
// The tiles are those of the two kernels, so a layer's bits do not depend on its neighbours.
#include <hip/hip_runtime.h>
#include "lcd_gemm_wide.h"
#include "lcd_gemm_split.h"

namespace lcd {

template <int BITS, int TBLK, int B, int PAIRS>
__global__ void __launch_bounds__(kSplitWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) gemm_mixed_kernel(const GemmBatch wide, const GemmBatch split, const uint32_t wide_blocks)
{
    static_assert(kSplitWaves == 8, "one workgroup size");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    if (blockIdx.x < wide_blocks) wide_workgroup<BITS, B, 2, PAIRS>(wide, blockIdx.x, lds);      // (wide_blocks is a multiple of the XCDs)
    else split_workgroup<BITS, 2, TBLK>(split, blockIdx.x - wide_blocks, lds);
}

template <int BITS, int TBLK, int B, int PAIRS>
static WideVariant variant_of()
{
    constexpr size_t split = split_lds_bytes<2, TBLK>(), wide = wide_lds_bytes<B, 2, PAIRS>();
    return WideVariant{(const void *)gemm_mixed_kernel<BITS, TBLK, B, PAIRS>, split > wide ? split : wide, kSplitWaves * 64, (((BITS - 2) * 2 + TBLK - 3) * 2 + B - 3) * 2 + PAIRS - 1};
}
template <int BITS, int TBLK>
static WideVariant pick(const WideTiles &t)
{
    if (t.form == kHalves128) return t.blocks == 3 ? variant_of<BITS, TBLK, 3, 1>() : variant_of<BITS, TBLK, 4, 1>();
    return t.blocks == 3 ? variant_of<BITS, TBLK, 3, 2>() : variant_of<BITS, TBLK, 4, 2>();
}

template <int BITS>
WideVariant mixed_variant(const WideTiles &t, int blocks)
{
    return blocks <= 3 ? pick<BITS, 3>(t) : pick<BITS, 4>(t);
}
template WideVariant mixed_variant<LCD_GEMM_BITS>(const WideTiles &, int);

}  // namespace lcd
