// The split prefill kernel (lcd_gemm_split.h) for every tile shape.
#include <hip/hip_runtime.h>
#include "lcd_gemm_split.h"

namespace lcd {

template <int BITS, int PAIRS, int TBLK>
__global__ void __launch_bounds__(kSplitWaves * 64, 1) gemm_split_kernel(const GemmBatch batch)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    split_workgroup<BITS, PAIRS, TBLK>(batch, blockIdx.x, lds);
}

template <int BITS, int PAIRS, int TBLK>
static SplitVariant variant_of()
{
    return SplitVariant{(const void *)gemm_split_kernel<BITS, PAIRS, TBLK>, split_lds_bytes<PAIRS, TBLK>(), (BITS - 2) * 6 + (PAIRS - 1) * 2 + TBLK - 1};
}

template <int BITS>
static SplitVariant pick(int pairs, int blocks)
{
    if (pairs == 1) return blocks == 1 ? variant_of<BITS, 1, 1>() : variant_of<BITS, 1, 2>();
    return blocks == 1 ? variant_of<BITS, 2, 1>() : blocks == 2 ? variant_of<BITS, 2, 2>() : blocks == 3 ? variant_of<BITS, 2, 3>() : variant_of<BITS, 2, 4>();
}

SplitVariant split_variant(int bits, int pairs, int blocks)
{
    return bits == 2 ? pick<2>(pairs, blocks) : bits == 3 ? pick<3>(pairs, blocks) : pick<4>(pairs, blocks);
}

}  // namespace lcd
