// What the wide and the split prefill kernel (lcd_gemm_wide.h, lcd_gemm_split.h) share: accumulators in fixed registers,
// codebook tables, packed words, LDS helpers.
#pragma once
#include <hip/hip_runtime.h>
#include "lcd_internal.h"
#include "lcd_device.h"
#include "lcd_gemm_plan.h"

namespace lcd {

// packed weights are read by every token block of the layer: default cache policy (the non-temporal
// hint of the decode kernels costs 2 % here)
constexpr int kGemmWeightPolicy = 0;

typedef __attribute__((address_space(3))) uint32_t lds_u32;

// ---- accumulators in fixed accumulation registers ------------------------------------------------
// The accumulators of a wave (up to 16 of 16 registers each) live in a[0:255] and are touched only by the
// inline assembly below, so the compiler never copies them (as loop-carried values it would move
// all 128 registers to VGPRs and back in every iteration).  The files that include this are compiled
// with AGPR spilling disabled and use no MFMA builtins, which leaves the compiler one use for an AGPR: a value that it keeps across the
// loop when a kernel has no vector register left.  It does not know the accumulators to be live between their instructions, so no
// kernel may come to that: tests/test_prefill_registers.py reads it from the built code, and the distances below as well.
// The compiler does not look inside the assembly text, so it cannot keep the distance the hardware
// requires between a vector instruction that writes a register and a matrix instruction that reads it
// as an operand (it is free to place the last instruction of an operand's dequantisation directly in
// front of the matrix instruction, and does so depending on unrelated details of the source): every
// matrix instruction therefore brings its own two wait states (APART), but for those of the wide kernel, which pins the last instruction of every
// operand at least one matrix instruction ahead of the one that reads it.
template <int IDX, bool APART = true> __device__ __forceinline__ void mfma_acc(uint4v a, uint4v b);
template <int IDX> __device__ __forceinline__ float16v read_acc();
template <int IDX> __device__ __forceinline__ void zero_acc();
// Register names cannot be computed inside assembly text, so each accumulator lists its 16 registers once.
#define LCD_ACC_CLOBBERS(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                   \
    "a" #r0, "a" #r1, "a" #r2, "a" #r3, "a" #r4, "a" #r5, "a" #r6, "a" #r7, "a" #r8, "a" #r9, "a" #r10, "a" #r11, "a" #r12,      \
        "a" #r13, "a" #r14, "a" #r15
#define LCD_ACC_READ(n, r) "v_accvgpr_read_b32 %" #n ", a" #r
#define LCD_ACC_ZERO(r) "v_accvgpr_write_b32 a" #r ", 0"
#define LCD_ACCUMULATOR(IDX, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                                \
    template <> __device__ __forceinline__ void mfma_acc<IDX, false>(uint4v a, uint4v b)                                          \
    {                                                                                                                              \
        asm volatile("v_mfma_f32_32x32x16_f16 a[" #r0 ":" #r15 "], %0, %1, a[" #r0 ":" #r15 "]"                                  \
                     :                                                                                                             \
                     : "v"(a), "v"(b)                                                                                              \
                     : LCD_ACC_CLOBBERS(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));                    \
    }                                                                                                                              \
    template <> __device__ __forceinline__ void mfma_acc<IDX, true>(uint4v a, uint4v b)                                           \
    {                                                                                                                              \
        asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_f16 a[" #r0 ":" #r15 "], %0, %1, a[" #r0 ":" #r15 "]"                     \
                     :                                                                                                             \
                     : "v"(a), "v"(b)                                                                                              \
                     : LCD_ACC_CLOBBERS(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));                    \
    }                                                                                                                              \
    template <> __device__ __forceinline__ float16v read_acc<IDX>()                                                                \
    {                                                                                                                              \
        float t[16];                                                                                                               \
        asm volatile(LCD_ACC_READ(0, r0) "\n\t" LCD_ACC_READ(1, r1) "\n\t" LCD_ACC_READ(2, r2) "\n\t" LCD_ACC_READ(3, r3) "\n\t"   \
                     LCD_ACC_READ(4, r4) "\n\t" LCD_ACC_READ(5, r5) "\n\t" LCD_ACC_READ(6, r6) "\n\t" LCD_ACC_READ(7, r7) "\n\t"   \
                     LCD_ACC_READ(8, r8) "\n\t" LCD_ACC_READ(9, r9) "\n\t" LCD_ACC_READ(10, r10) "\n\t" LCD_ACC_READ(11, r11)      \
                     "\n\t" LCD_ACC_READ(12, r12) "\n\t" LCD_ACC_READ(13, r13) "\n\t" LCD_ACC_READ(14, r14) "\n\t"                 \
                     LCD_ACC_READ(15, r15)                                                                                         \
                     : "=v"(t[0]), "=v"(t[1]), "=v"(t[2]), "=v"(t[3]), "=v"(t[4]), "=v"(t[5]), "=v"(t[6]), "=v"(t[7]),             \
                       "=v"(t[8]), "=v"(t[9]), "=v"(t[10]), "=v"(t[11]), "=v"(t[12]), "=v"(t[13]), "=v"(t[14]), "=v"(t[15]));      \
        float16v v;                                                                                                                \
        for (int i = 0; i < 16; ++i) v[i] = t[i];                                                                                  \
        return v;                                                                                                                  \
    }                                                                                                                              \
    template <> __device__ __forceinline__ void zero_acc<IDX>()                                                                    \
    {                                                                                                                              \
        asm volatile(LCD_ACC_ZERO(r0) "\n\t" LCD_ACC_ZERO(r1) "\n\t" LCD_ACC_ZERO(r2) "\n\t" LCD_ACC_ZERO(r3) "\n\t"               \
                     LCD_ACC_ZERO(r4) "\n\t" LCD_ACC_ZERO(r5) "\n\t" LCD_ACC_ZERO(r6) "\n\t" LCD_ACC_ZERO(r7) "\n\t"               \
                     LCD_ACC_ZERO(r8) "\n\t" LCD_ACC_ZERO(r9) "\n\t" LCD_ACC_ZERO(r10) "\n\t" LCD_ACC_ZERO(r11) "\n\t"             \
                     LCD_ACC_ZERO(r12) "\n\t" LCD_ACC_ZERO(r13) "\n\t" LCD_ACC_ZERO(r14) "\n\t" LCD_ACC_ZERO(r15)                  \
                     :                                                                                                             \
                     :                                                                                                             \
                     : LCD_ACC_CLOBBERS(r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15));                    \
    }
LCD_ACCUMULATOR(0, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15)
LCD_ACCUMULATOR(1, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31)
LCD_ACCUMULATOR(2, 32, 33, 34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47)
LCD_ACCUMULATOR(3, 48, 49, 50, 51, 52, 53, 54, 55, 56, 57, 58, 59, 60, 61, 62, 63)
LCD_ACCUMULATOR(4, 64, 65, 66, 67, 68, 69, 70, 71, 72, 73, 74, 75, 76, 77, 78, 79)
LCD_ACCUMULATOR(5, 80, 81, 82, 83, 84, 85, 86, 87, 88, 89, 90, 91, 92, 93, 94, 95)
LCD_ACCUMULATOR(6, 96, 97, 98, 99, 100, 101, 102, 103, 104, 105, 106, 107, 108, 109, 110, 111)
LCD_ACCUMULATOR(7, 112, 113, 114, 115, 116, 117, 118, 119, 120, 121, 122, 123, 124, 125, 126, 127)
LCD_ACCUMULATOR(8, 128, 129, 130, 131, 132, 133, 134, 135, 136, 137, 138, 139, 140, 141, 142, 143)
LCD_ACCUMULATOR(9, 144, 145, 146, 147, 148, 149, 150, 151, 152, 153, 154, 155, 156, 157, 158, 159)
LCD_ACCUMULATOR(10, 160, 161, 162, 163, 164, 165, 166, 167, 168, 169, 170, 171, 172, 173, 174, 175)
LCD_ACCUMULATOR(11, 176, 177, 178, 179, 180, 181, 182, 183, 184, 185, 186, 187, 188, 189, 190, 191)
LCD_ACCUMULATOR(12, 192, 193, 194, 195, 196, 197, 198, 199, 200, 201, 202, 203, 204, 205, 206, 207)
LCD_ACCUMULATOR(13, 208, 209, 210, 211, 212, 213, 214, 215, 216, 217, 218, 219, 220, 221, 222, 223)
LCD_ACCUMULATOR(14, 224, 225, 226, 227, 228, 229, 230, 231, 232, 233, 234, 235, 236, 237, 238, 239)
LCD_ACCUMULATOR(15, 240, 241, 242, 243, 244, 245, 246, 247, 248, 249, 250, 251, 252, 253, 254, 255)
#undef LCD_ACCUMULATOR
#undef LCD_ACC_ZERO
#undef LCD_ACC_READ
#undef LCD_ACC_CLOBBERS

// byte-split codebook of a lane's row: two words of each kind up to 3 bits, four with 4 bits
template <int BITS> struct GemmTables { typedef RowTables type; };
template <> struct GemmTables<4> { typedef RowTables4 type; };

template <int N>
__device__ __forceinline__ void lds_wait()
{
    asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory");
}
template <int N>
__device__ __forceinline__ void vmem_wait()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// 16 bytes per lane from LDS, not waited for
template <int OFFSET>
__device__ __forceinline__ uint4v lds_read(uint32_t base)
{
    uint4v v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(base), "n"(OFFSET) : "memory");
    return v;
}
__device__ __forceinline__ uint32_t lds_address(const uint8_t *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}

// One lane's packed words of a chunk half: per pair, the lane's row and the 64 columns
// [64*(2*half + L>>5), +64) of the chunk.
template <int BITS, int PAIRS>
struct GemmTileRegs {
    uint4v lo[PAIRS];
    uint2v hi[PAIRS];    // 3 bits: the third-bit words
    uint4v hi4[PAIRS];   // 4 bits: the second plane
};

// Where a lane's packed words of each pair stand: its row and slot never change (rows past the layer out of range: zeros), the 128-column half
// travels as the scalar offset.
template <int PAIRS> struct GemmRows { uint32_t at[PAIRS], slot; };
template <int BITS, int PAIRS>
__device__ __forceinline__ GemmRows<PAIRS> gemm_rows(int t0, int nt, int kc, int lane)
{
    constexpr uint32_t TB = kTileRows * kTileCols * BITS / 8;
    GemmRows<PAIRS> rows;
    rows.slot = 16 * (lane >> 5) + (lane & 15);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        const uint32_t tile = t0 + 2 * p + ((lane >> 4) & 1);
        rows.at[p] = tile < (uint32_t)nt ? tile * (uint32_t)kc * TB + 16 * rows.slot : 0xFFFFFFF0u;
    }
    return rows;
}
// half h of chunk c
template <int BITS, int PAIRS>
__device__ __forceinline__ void load_gemm_words(GemmTileRegs<BITS, PAIRS> &r, __amdgpu_buffer_rsrc_t packed, const GemmRows<PAIRS> &rows, uint32_t c, uint32_t h)
{
    const uint32_t o = c * (kTileRows * kTileCols * BITS / 8);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        r.lo[p] = __builtin_amdgcn_raw_buffer_load_b128(packed, rows.at[p], o + h * 512, kGemmWeightPolicy);
        if (BITS == 3) r.hi[p] = __builtin_amdgcn_raw_buffer_load_b64(packed, rows.at[p] < 0xFFFFFFF0u ? rows.at[p] - 8 * rows.slot : 0xFFFFFFF0u, o + h * 256 + 1024, kGemmWeightPolicy);
        if (BITS == 4) r.hi4[p] = __builtin_amdgcn_raw_buffer_load_b128(packed, rows.at[p], o + h * 512 + 1024, kGemmWeightPolicy);
    }
}

// a lane's row in each pair, and its byte-split codebook
template <int BITS, int PAIRS>
__device__ __forceinline__ void load_gemm_tables(typename GemmTables<BITS>::type (&tb)[PAIRS], const uint8_t *__restrict__ lutB, int t0, int nt, int lane)
{
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        const int tile = min(t0 + 2 * p + ((lane >> 4) & 1), nt - 1);
        const int row = tile * kTileRows + (lane & 15);
        if constexpr (BITS == 2) {
            const uint2v v = *reinterpret_cast<const uint2v *>(lutB + (size_t)row * 8);
            tb[p].lo[0] = v[0]; tb[p].hi[0] = v[1]; tb[p].lo[1] = 0; tb[p].hi[1] = 0;
        } else if constexpr (BITS == 3) {
            const uint4v v = *reinterpret_cast<const uint4v *>(lutB + (size_t)row * 16);
            tb[p].lo[0] = v[0]; tb[p].lo[1] = v[1]; tb[p].hi[0] = v[2]; tb[p].hi[1] = v[3];
        } else {
            const uint4v v = *reinterpret_cast<const uint4v *>(lutB + (size_t)row * 32);
            const uint4v w = *reinterpret_cast<const uint4v *>(lutB + (size_t)row * 32 + 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) { tb[p].lo[u] = v[u]; tb[p].hi[u] = w[u]; }
        }
    }
}

// The dequantiser's first two stages for quarter T of word DN of pair P, for any width: the selector
// (4 bits: and the pool word), then the table lookups.
template <int BITS, int DN, int T, int PAIRS>
__device__ __forceinline__ void gemm_select(const GemmTileRegs<BITS, PAIRS> &r, int p, const HighBits &hb, uint32_t &sel, uint32_t &pool)
{
    if constexpr (BITS == 4) decode_select4<T>(r.lo[p][DN], r.hi4[p][DN], sel, pool);
    else sel = decode_select<BITS, DN, T>(r.lo[p][DN], hb);
}
template <int BITS>
__device__ __forceinline__ void gemm_lookup(uint32_t sel, uint32_t pool, const typename GemmTables<BITS>::type &tb, uint32_t &lo, uint32_t &hi)
{
    if constexpr (BITS == 4) decode_lookup4(sel, pool, tb, lo, hi);
    else decode_lookup<BITS>(sel, tb, lo, hi);
}

// ---- a launch: the layers and their places in the XCDs' queues of workgroups --------------------------
struct GemmProblem {
    const uint8_t *packed, *lutB, *xs;
    uint16_t *y;
    int N, K, grid_rows;
    float out_scale;        // 1, or the layer's activation quantisation step
    uint32_t tiles[2];      // wide kernel: in the columns of the most blocks, and of one block less
    int tiles_per_xcd, queue_begin;   // split kernel: position of this layer's first tile in an XCD's queue
};
struct GemmBatch {
    GemmProblem p[kMaxGroup];
    int count, M, Mpad;
    WideTiles tiles;        // wide kernel
};

// A variant of the split kernel (lcd_gemm_split.hip): 32 * pairs rows x 32 * blocks tokens per workgroup; pairs 1 with
// blocks 1 or 2, pairs 2 with blocks 1..4.
struct SplitVariant {
    const void *fn;
    size_t lds_bytes;
    int id;             // 0 .. kSplitVariants - 1
};
constexpr int kSplitVariants = 3 * 6;
SplitVariant split_variant(int bits, int pairs, int blocks);
// A variant of the wide kernel (lcd_gemm_wide.hip), and of the kernel that takes wide tiles (in halves, 3 or 4 blocks) and split tiles of 64 rows x
// 32 * blocks tokens, blocks 3 or 4 (lcd_gemm_mixed.hip).
struct WideVariant {
    const void *fn;
    size_t lds_bytes;
    int threads;
    int id;             // 0 .. kWideVariants - 1, 0 .. kMixedVariants - 1
};
constexpr int kWideVariants = 3 * 12, kMixedVariants = 3 * 8;
template <int BITS> WideVariant wide_variant(const WideTiles &t);
template <int BITS> WideVariant mixed_variant(const WideTiles &t, int blocks);

}  // namespace lcd
