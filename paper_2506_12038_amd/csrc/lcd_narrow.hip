// Prefill of few tokens (17 and more) of the smoothed table-lookup product, gfx950: the narrow kernel.
//
// The packed indices are dequantised in registers (as in the tokens kernel) into the A operand of v_mfma_f32_16x16x32_f16; the
// activations have been transformed into operand order (transform_kernel), so that a B operand is one load of 16 bytes per lane,
// straight from the L2 into registers: no LDS, no barrier inside K, tokens padded to blocks of 16 only.
//
// Work split.  A workgroup owns a contiguous run of row tiles (16 rows) of ONE layer and takes them R at a time, with all tokens; its 8 waves
// split K, wave w takes the 256-column chunks w, w + 8, ...  A packed word (16 weights per lane) is two k-steps: it is decoded for each of the R row
// tiles and multiplied with the two steps' TB blocks of tokens, which wait in a window of four steps.  At the end the 8 partial
// tiles are added through LDS in the order of the waves, rounded once and stored: the order of the additions of one output depends on K alone.
//
// What bounds it: the activations' way into the registers (every compute unit reads all of them per pass: 114 GB/s of its 134 at 64 bytes a cycle),
// then the dequantiser and the matrix instructions, which hardly overlap: a workgroup of t row tiles and TB blocks takes about 2.4 us
// + rounds of 8 chunks * (0.37 TB per pass + t * (0.6 + 0.155 TB)), 3 bits.  40 tokens, 3 bits, matrix launch alone: 4096 x 4096 6.6 us, three of
// them 10.6, two of 11008 x 4096 16.8 (0.43 PFLOP/s).  More waves (16) with shorter windows, windows of 8 steps and matrix and vector instructions
// interleaved by hand changed nothing.  Against the split kernel (64-row tiles whose activations go through LDS, tokens padded to 32 or 64): see
// narrow_takes, which also says where the line lies.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "lcd_decode.h"

namespace lcd {

template <int TB, int R> constexpr size_t narrow_lds_bytes() { return (size_t)kBW * R * TB * 1024; }
constexpr int WINDOW = 4;     // k-steps whose B operands are held or under way

template <int BITS, int TB, int R>
__global__ void __launch_bounds__(kBW * 64, 1) gemm_narrow_kernel(const uint32_t t0, const uint32_t t1, const uint32_t t2, const uint32_t t3,
                                                                  const uint32_t t4, const uint32_t t5, const uint32_t t6, const uint32_t t7,
                                                                  const uint16_t *head_x, const float *head_s, const uint32_t head_word, const BucketBatch batch)
{
    constexpr uint32_t TBYTES = kTileRows * kTileCols * BITS / 8;
    constexpr uint32_t ROW_TABLE = row_table_bytes<BITS>();
    constexpr int NC = BITS == 2 ? 4 : 8;
    typedef typename TablesOf<BITS>::type Tables;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // partial tiles [wave][tile][block][partial_quad]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keeps addresses scalar
    const int q = lane >> 4, j = lane & 15;

    int pi = (head_word & kHeadSingle) ? 0 : layer_of_workgroup(blockIdx.x, t0, t1, t2, t3, t4, t5, t6, t7);
    const uint16_t *x = head_x;
    const float *s = head_s;
    int kc;
    input_of(batch, pi, head_word & ~(kNarrowTokensMask << kNarrowTokensShift), x, s, kc);
    const int M = (int)((head_word >> kNarrowTokensShift) & kNarrowTokensMask);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(x, (uint32_t)M * (uint32_t)kc * (kTileCols * 2));

    // B operands: lane (q, j) of block t holds columns 64 q + 8 g .. of token 16 t + j, at ((chunk * 8 + g) * 4 + q) * M + token, 16 bytes each.
    // Everything but the lane's part is wave-uniform and travels as the scalar offset; lanes past the last token read zeros.
    const uint32_t x_lane = (uint32_t)(q * M + j) * 16;
    const uint32_t x_last = 16 * (TB - 1) + j < M ? x_lane : kOob;
    uint4v B[WINDOW][TB];
    auto load_step = [&](uint4v (&b)[TB], int chunk, int g) __attribute__((always_inline)) {
        uint32_t o = __builtin_amdgcn_readfirstlane((uint32_t)(chunk * 8 + g) * 4 * (uint32_t)M * 16);
        asm volatile("" : "+s"(o));
#pragma unroll
        for (int t = 0; t < TB; ++t)
            b[t] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, t == TB - 1 ? x_last : x_lane, o + t * 256, 0);
    };
    if (wave < kc) {
        unrolled<WINDOW>([&](auto g) __attribute__((always_inline)) { load_step(B[g], wave, decltype(g)::value); });
    }
    asm volatile("" ::: "memory");
    const LayerPart l = part_of(batch, pi, head_word, blockIdx.x, t0, t1, t2, t3, t4, t5, t6);
    const int ta = l.ta, tb_end = l.tb, N = l.nt * kTileRows;
    asm volatile("" : "+s"(pi) : : "memory");   // what is needed last is asked for last
    uint16_t *const y = batch.p[pi].y;
    const float act_scale = batch.p[pi].act_scale, out_scale = act_scale != 0.0f ? act_scale : 1.0f;
    const __amdgpu_buffer_rsrc_t rs_packed = make_rsrc(l.packed, (uint32_t)l.nt * (uint32_t)kc * TBYTES);
    // byte-split tables: behind the bucket multipliers (2 and 3 bits), the whole table (4 bits)
    const __amdgpu_buffer_rsrc_t rs_tb = make_rsrc(reinterpret_cast<const uint8_t *>(l.lut) + (BITS == 4 ? 0 : (size_t)N * NC * 4), (uint32_t)N * ROW_TABLE);
    auto load_tile = [&](PackedTile<BITS> &p, int tile, int chunk) __attribute__((always_inline)) {
        const bool v = tile < tb_end && chunk < kc;
        const uint32_t o = v ? ((uint32_t)tile * (uint32_t)kc + (uint32_t)chunk) * TBYTES : 0u;
        p.lo = __builtin_amdgcn_raw_buffer_load_b128(rs_packed, v ? 16 * lane : kOob, o, kStreamPolicy);
        if (BITS == 3) p.hi = __builtin_amdgcn_raw_buffer_load_b64(rs_packed, v ? 8 * lane : kOob, o + 1024, kStreamPolicy);
        if (BITS == 4) p.hi4 = __builtin_amdgcn_raw_buffer_load_b128(rs_packed, v ? 16 * lane : kOob, o + 1024, kStreamPolicy);
    };
    Tables tab[R];
    PackedTile<BITS> P[R];
    float4v acc[R][TB];

    for (int v0 = ta; v0 < tb_end; v0 += R) {
        const int n = min(R, tb_end - v0);
        if (v0 > ta && wave < kc) unrolled<WINDOW>([&](auto g) __attribute__((always_inline)) { load_step(B[g], wave, decltype(g)::value); });
#pragma unroll
        for (int r = 0; r < R; ++r) {
            load_tile(P[r], v0 + r, wave);
            const uint32_t at = v0 + r < tb_end ? ((uint32_t)(v0 + r) * kTileRows + j) * ROW_TABLE : kOob;
            if constexpr (BITS == 2) {
                const uint2v t = __builtin_amdgcn_raw_buffer_load_b64(rs_tb, at, 0, 0);
                tab[r] = RowTables{{t[0], 0u}, {t[1], 0u}};
            } else if constexpr (BITS == 3) {
                const uint4v t = __builtin_amdgcn_raw_buffer_load_b128(rs_tb, at, 0, 0);
                tab[r] = RowTables{{t[0], t[1]}, {t[2], t[3]}};
            } else {
                const uint4v t = __builtin_amdgcn_raw_buffer_load_b128(rs_tb, at, 0, 0), u = __builtin_amdgcn_raw_buffer_load_b128(rs_tb, at, 16, 0);
                tab[r] = RowTables4{{t[0], t[1], t[2], t[3]}, {u[0], u[1], u[2], u[3]}};
            }
#pragma unroll
            for (int t = 0; t < TB; ++t) acc[r][t] = float4v{0.f, 0.f, 0.f, 0.f};
        }
        // One chunk.  TAIL: the wave's last one of the pass (loads behind it would take the time of their addresses).
        auto chunk_products = [&](auto TAIL_, int c) __attribute__((always_inline)) {
            constexpr bool TAIL = decltype(TAIL_)::value;
            HighBits hb[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                hb[r] = HighBits{0u, 0u};
                if (BITS == 3) hb[r] = regroup_high(P[r].hi);
            }
            unrolled<4>([&](auto d_) __attribute__((always_inline)) {
                constexpr int d = decltype(d_)::value;
                uint4v(&b0)[TB] = B[(2 * d) % WINDOW], (&b1)[TB] = B[(2 * d + 1) % WINDOW];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r == 0 || r < n) {       // uniform
                        uint4v op0, op1;
                        if constexpr (BITS == 4) decode_word4(P[r].lo[d], P[r].hi4[d], tab[r], op0, op1);
                        else decode_word<BITS, d>(P[r].lo[d], hb[r], tab[r], op0, op1);
#pragma unroll
                        for (int t = 0; t < TB; ++t) acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(op0), as_half8(b0[t]), acc[r][t], 0, 0, 0);
#pragma unroll
                        for (int t = 0; t < TB; ++t) acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(op1), as_half8(b1[t]), acc[r][t], 0, 0, 0);
                    }
                    if constexpr (d == 3 && !TAIL) load_tile(P[r], v0 + r, c + kBW);
                }
                if constexpr (2 * d + WINDOW < 8) {
                    load_step(b0, c, 2 * d + WINDOW);
                    load_step(b1, c, 2 * d + 1 + WINDOW);
                } else if constexpr (!TAIL) {
                    load_step(b0, c + kBW, 2 * d + WINDOW - 8);
                    load_step(b1, c + kBW, 2 * d + 1 + WINDOW - 8);
                }
            });
        };
        int c = wave;
#pragma unroll 1
        for (; c + kBW < kc; c += kBW) chunk_products(std::false_type{}, c);
        if (c < kc) chunk_products(std::true_type{}, c);

        // ---- partial tiles to LDS, one barrier, sum over the waves in order, one rounding, store
        float *part = reinterpret_cast<float *>(smem) + wave * (R * TB * 256);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < TB; ++t) *reinterpret_cast<float4v *>(&part[(r * TB + t) * 256 + partial_quad(r, q, j)]) = acc[r][t];   // lane (q, j): rows 4q..4q+3 of token j
        __syncthreads();
        const int quads = n * 4;                 // row quads of one token
        for (int e = threadIdx.x; e < quads * M; e += kBW * 64) {
            const int m = e / quads, rest = e - m * quads, r = rest >> 2, rq = rest & 3;
            const float *src = reinterpret_cast<const float *>(smem) + (r * TB + (m >> 4)) * 256 + partial_quad(r, rq, m & 15);
            float4v sum = *reinterpret_cast<const float4v *>(src);
#pragma unroll
            for (int w = 1; w < kBW; ++w) sum += *reinterpret_cast<const float4v *>(src + w * (R * TB * 256));
            typedef _Float16 half4 __attribute__((ext_vector_type(4)));
            half4 o;
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = (_Float16)(sum[u] * out_scale);
            *reinterpret_cast<half4 *>(y + (size_t)m * N + (size_t)(v0 + r) * kTileRows + 4 * rq) = o;
        }
        if (v0 + R < tb_end) __syncthreads();    // the next partial tiles take the same places
    }
}

template <int BITS, int TB, int R>
static TokensVariant variant_of(int slot)
{
    return TokensVariant{(const void *)gemm_narrow_kernel<BITS, TB, R>, R, kBW, narrow_lds_bytes<TB, R>(), ((BITS - 2) * kNarrowBlocks + TB - 1) * 4 + slot};
}

// row tiles of the largest variant: what the registers hold next to the window, and LDS as partial tiles
template <int TB> constexpr int narrow_tiles() { return TB <= 3 ? 6 : TB == 4 ? 4 : 3; }

template <int BITS, int TB>
static TokensVariant pick_tiles(int tiles)
{
    if (tiles <= 1) return variant_of<BITS, TB, 1>(0);
    if (tiles <= 2) return variant_of<BITS, TB, 2>(1);
    if constexpr (narrow_tiles<TB>() > 3) if (tiles > 3) return variant_of<BITS, TB, narrow_tiles<TB>()>(3);
    return variant_of<BITS, TB, 3>(2);
}

template <int BITS>
static TokensVariant pick(int blocks, int tiles)
{
    switch (blocks) {
    case 1: case 2: return pick_tiles<BITS, 2>(tiles);
    case 3: return pick_tiles<BITS, 3>(tiles);
    case 4: return pick_tiles<BITS, 4>(tiles);
    case 5: return pick_tiles<BITS, 5>(tiles);
    default: return pick_tiles<BITS, 6>(tiles);
    }
}

TokensVariant narrow_variant(int bits, int tokens, int tiles)
{
    const int blocks = (tokens + kTokenBlock - 1) / kTokenBlock;
    return bits == 2 ? pick<2>(blocks, tiles) : bits == 3 ? pick<3>(blocks, tiles) : pick<4>(blocks, tiles);
}

}  // namespace lcd
