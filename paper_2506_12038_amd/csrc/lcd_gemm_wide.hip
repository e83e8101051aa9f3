// The wide prefill kernel (lcd_gemm_wide.h) for every tile shape of one index width (LCD_GEMM_BITS, given by the build: the widths compile side by side).
#include <hip/hip_runtime.h>
#include "lcd_gemm_wide.h"

namespace lcd {

// K in halves (SPLIT 2: 8 waves), or whole (4 waves)
template <int BITS, int B, int SPLIT, int PAIRS>
__global__ void __launch_bounds__(SPLIT * 256) __attribute__((amdgpu_waves_per_eu(SPLIT, SPLIT))) gemm_wide_kernel(const GemmBatch batch)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    wide_workgroup<BITS, B, SPLIT, PAIRS>(batch, blockIdx.x, lds);
}

template <int BITS, int B, int SPLIT, int PAIRS>
static WideVariant variant_of()
{
    return WideVariant{(const void *)gemm_wide_kernel<BITS, B, SPLIT, PAIRS>, wide_lds_bytes<B, SPLIT, PAIRS>(), SPLIT * 256, (BITS - 2) * 12 + (SPLIT == 1 ? 8 + B - 5 : (PAIRS - 1) * 4 + B - 1)};
}

template <int BITS>
WideVariant wide_variant(const WideTiles &t)
{
    if (t.form == kWhole256) return t.blocks == 5 ? variant_of<BITS, 5, 1, 2>() : t.blocks == 6 ? variant_of<BITS, 6, 1, 2>() : t.blocks == 7 ? variant_of<BITS, 7, 1, 2>() : variant_of<BITS, 8, 1, 2>();
    if (t.form == kHalves256) return t.blocks == 1 ? variant_of<BITS, 1, 2, 2>() : t.blocks == 2 ? variant_of<BITS, 2, 2, 2>() : t.blocks == 3 ? variant_of<BITS, 3, 2, 2>() : variant_of<BITS, 4, 2, 2>();
    return t.blocks == 1 ? variant_of<BITS, 1, 2, 1>() : t.blocks == 2 ? variant_of<BITS, 2, 2, 1>() : t.blocks == 3 ? variant_of<BITS, 3, 2, 1>() : variant_of<BITS, 4, 2, 1>();
}
template WideVariant wide_variant<LCD_GEMM_BITS>(const WideTiles &);

}  // namespace lcd
