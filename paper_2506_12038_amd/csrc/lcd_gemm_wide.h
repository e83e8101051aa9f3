// The wide prefill kernel's workgroup (gfx950): prompts whose outputs fill the chip with large tiles.
//
// A dense contraction on v_mfma_f32_32x32x16_f16 with fp32 accumulators in fixed accumulation registers.  A wave owns 64 rows (two pairs of 32; 32
// rows in tiles of 128) and T blocks of 32 tokens.  Weights never pass through LDS: a lane loads its 16 bytes of the packed layout and dequantises them in
// registers into its A operand.  Activations (smoothed once per call, operand order) are shared by the workgroup's four row groups through a ring in
// LDS, filled by direct-to-LDS loads.  Two forms:
//   whole    4 waves, one per SIMD, T = 5..8 (4): 512 registers per lane hold 256 tokens' sums, an operand that was dequantised once meets 8
//            matrix instructions and an activation read from LDS two.  The least energy per product, which is what a full chip's rate hangs on.
//   halves   8 waves, two per SIMD, T = 1..4: each wave of a row group takes the 128-column halves of one parity; the two sums are added through
//            LDS at the end.  Two waves share a SIMD's issue (a wave alone issues one instruction per 8 cycles, which below T = 6 is less than the
//            dequantiser and the matrix pipe take), and smaller tiles fill the chip with fewer outputs.
// The order of the additions of an output depends on the form and K alone, not on T or the rows of a tile.
//
// Ring: 16 k-steps (two units of 8) of T KiB per half.  A quarter is 4 k-steps; while quarter i is multiplied, quarter i + 2 is copied into the
// place of quarter i - 2.  One barrier per quarter, AHEAD steps before its first read, so that no wave runs out of operands at it; copies have two quarters to
// land and the wait in front of the barrier leaves the newest T loads under way: the newer quarter's copies, or, at the second barrier of a unit, the next packed
// words' loads (1 to 4, asked for after those copies) and as many fewer of the copies.  (The copies are buffer loads: behind global loads to LDS
// the compiler waits for every load under way wherever packed words are used.)  Every matrix instruction is followed by a share of the next packed
// word's dequantisation.
//
// What bounds it: the power management.  8192 x 8192, 8192 tokens, T = 8: matrix pipe busy 85 % of the cycles, at 1.40 GHz (counter run, 878 us); with two wait states per
// matrix instruction and the dequantiser in one place per step less of them at a higher clock, the same time.  So fewer instructions per product count: 3 bits, 8192 tokens, tiles
// of 256 x 128 with two waves of 64 x 128 per SIMD as before 945 us, whole, T = 4, 6, 8 978, 930, 840 us (1.31 PFLOP/s); 2 bits 875 -> 800, 4 bits 1065 -> 868.
// Tiles of 128 x 256 in halves (same registers, twice the copies) 946 us.  Whole calls against the large-tile and the split kernel before it, 7B block in four
// calls, 2048 tokens, 3 bits 806 -> 746 us; 333 tokens of codes, 2 bits 193 -> 177 (both sides on one box); by layer: beside split_takes and in lcd_gemm_plan.h.
#pragma once
#include <type_traits>
#include "lcd_gemm_common.h"

namespace lcd {

// 1 KiB (16 bytes per lane) from byte lane_offset + offset of a buffer to LDS
__device__ __forceinline__ void copy_kib(__amdgpu_buffer_rsrc_t from, uint32_t to, uint32_t lane_offset, uint32_t offset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (lds_u32 *)(uintptr_t)to, 16, lane_offset, offset, 0, 0);
}

constexpr int kWideOutStride = 64 * 2 + 16;     // bytes of a token's 64 rows in the output stage (16-byte aligned, spreads the banks)
template <int T, int SPLIT, int PAIRS> constexpr size_t wide_lds_bytes()
{
    // whole: the output stage, two blocks per wave; halves: the sums that the waves of a row group hand over, which the output is staged in
    const size_t ring = (size_t)SPLIT * 16 * T * 1024, after = SPLIT == 1 ? (size_t)4 * 2 * 32 * kWideOutStride : (size_t)4 * 2 * (PAIRS == 2 ? T : (T + 1) / 2) * 4096;
    return ring > after ? ring : after;
}

// One output tile: tokens [32 tb0, 32 (tb0 + T)), rows [128 PAIRS bx, + 128 PAIRS).  SPLIT 2: K in halves.  The blocks all lie inside the padded tokens.
template <int BITS, int T, int SPLIT, int PAIRS>
__device__ __forceinline__ void wide_tile(const uint8_t *__restrict__ packed_, const uint8_t *__restrict__ lutB, const uint8_t *__restrict__ xs,
                                          uint16_t *__restrict__ y, int M, int mblk, int N, int K, int bx, int tb0, uint8_t *lds, float out_scale)
{
    constexpr uint32_t TB = kTileRows * kTileCols * BITS / 8;
    constexpr int WSTEPS = 2 * T;
    static_assert(PAIRS == 2 || SPLIT == 2, "tiles of 128 rows: in halves only");
    constexpr bool SHORT = T == 1 || SPLIT == 2;
    // operand window: reads AHEAD steps in front of their use (8 waves have registers for four)
    constexpr int WIN = SHORT ? 4 : 8, AHEAD = T * PAIRS == 1 ? 2 : SHORT ? 3 : T == 2 ? 5 : 6;
    constexpr int SPREAD = 2 * PAIRS;      // gaps from one copy to the next
    static_assert(4 * T - AHEAD > (SPREAD * (T - 1) + 1) / PAIRS, "every copy of a quarter is issued in front of the barrier of the next");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rgrp = wave & 3, kh = SPLIT == 2 ? wave >> 2 : 0;
    const int kc = K / kTileCols, nt = N / kTileRows;
    const int t0 = (bx * 4 + rgrp) * (2 * PAIRS);
    const __amdgpu_buffer_rsrc_t packed = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(packed_), 0, (uint32_t)nt * (uint32_t)kc * TB, 0x00020000);

    const size_t chunk_stride = (size_t)mblk * 16 * 1024;
    const uint8_t *const xs0 = xs + (size_t)tb0 * 16 * 1024;
    const uint32_t ring = lds_address(lds) + kh * (16 * T * 1024);
    // activations of chunk c: T blocks of 16 KiB
    auto chunk_at = [&](int c) __attribute__((always_inline)) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(xs0 + (size_t)c * chunk_stride), 0, T * 16 * 1024, 0x00020000); };
    // k-step `rgrp` of a quarter (4 k-steps of a unit): block b
    const uint32_t copy_to = ring + rgrp * (T * 1024), copy_from = lane * 16 + rgrp * 1024 + kh * 8192;
    auto copy_block = [&](__amdgpu_buffer_rsrc_t src, auto AT_, auto SLOT_, int b) __attribute__((always_inline)) {
        copy_kib(src, copy_to + decltype(SLOT_)::value * (4 * T * 1024) + b * 1024, copy_from, decltype(AT_)::value + b * (16 * 1024));
    };

    const GemmRows<PAIRS> rows = gemm_rows<BITS, PAIRS>(t0, nt, kc, lane);
    auto load_words = [&](GemmTileRegs<BITS, PAIRS> &r, int c, int h) __attribute__((always_inline)) { load_gemm_words<BITS>(r, packed, rows, (uint32_t)c, h); };
    using I0 = std::integral_constant<int, 0>; using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>; using I3 = std::integral_constant<int, 3>;

    GemmTileRegs<BITS, PAIRS> r0, r1;
    load_words(r0, 0, kh);
    load_words(r1, SPLIT == 2 ? min(1, kc - 1) : 0, SPLIT == 2 ? kh : 1);
    typename GemmTables<BITS>::type tb[PAIRS];
    load_gemm_tables<BITS>(tb, lutB, t0, nt, lane);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int b = 0; b < T; ++b) copy_block(chunk_at(0), I0{}, I0{}, b);
#pragma unroll
    for (int b = 0; b < T; ++b) copy_block(chunk_at(0), std::integral_constant<int, 4096>{}, I1{}, b);
    unrolled<PAIRS * T>([&](auto i) __attribute__((always_inline)) { zero_acc<decltype(i)::value>(); });

    struct Ops { uint4v op[PAIRS][2]; };
    Ops wa, wb;
    HighBits hb[PAIRS];
    auto high_bits = [&](const GemmTileRegs<BITS, PAIRS> &r) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            hb[p] = HighBits{0u, 0u};
            if (BITS == 3) hb[p] = regroup_high(r.hi[p]);
        }
    };
    high_bits(r0);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        if constexpr (BITS == 4) decode_word4(r0.lo[p][0], r0.hi4[p][0], tb[p], wa.op[p][0], wa.op[p][1]);
        else decode_word<BITS, 0>(r0.lo[p][0], hb[p], tb[p], wa.op[p][0], wa.op[p][1]);
    }
    vmem_wait<T>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    uint4v window[WIN];
    const uint32_t base[2] = {ring + lane * 16, ring + lane * 16 + 8 * T * 1024};
    unrolled<AHEAD>([&](auto i) __attribute__((always_inline)) { window[decltype(i)::value] = lds_read<decltype(i)::value * 1024>(base[0]); });

    // One packed word per pair: two k-steps.  U: parity of the unit (buffer half), D: word, DN: the word of rn decoded meanwhile.
    // The first and the third word copy the first and second half of the next unit's activations, which stand in chunk `src`.
    auto word = [&](auto U_, auto D_, auto DN_, const Ops &cur, Ops &nxt, const GemmTileRegs<BITS, PAIRS> &rn, __amdgpu_buffer_rsrc_t src) __attribute__((always_inline)) {
        constexpr int U = decltype(U_)::value, D = decltype(D_)::value, DN = decltype(DN_)::value;
        uint32_t sel[4 * PAIRS], pool[4 * PAIRS], lo[4 * PAIRS], hi[4 * PAIRS];
        // what stands behind matrix instruction G of the word: stages of the next word's dequantisation, a copy
        auto gap = [&](auto G_) __attribute__((always_inline)) {
            constexpr int G = decltype(G_)::value;
            if constexpr ((D & 1) == 0 && G % SPREAD == 1) {
                constexpr int at = (SPLIT == 2 ? 0 : (U ^ 1) * 8192) + (D >> 1) * 4096;
                copy_block(src, std::integral_constant<int, at>{}, std::integral_constant<int, 2 * (U ^ 1) + (D >> 1)>{}, G / SPREAD);
            }
            // stage i stands in gap i * GAPS / STAGES: never in a word's last, so that one matrix instruction at least lies between an operand and its reader
            constexpr int STAGES = 12 * PAIRS, GAPS = 2 * PAIRS * T - 1, i0 = (G * STAGES + GAPS - 1) / GAPS, i1 = ((G + 1) * STAGES + GAPS - 1) / GAPS;
            unrolled<(i1 < STAGES ? i1 : STAGES) - (i0 < STAGES ? i0 : STAGES)>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = i0 + decltype(i_)::value, q = i / 3, p = q >> 2, t = q & 3;
                {
                    if constexpr (i % 3 == 0) {
                        gemm_select<BITS, DN, t>(rn, p, hb[p], sel[q], pool[q]);
                    } else if constexpr (i % 3 == 1) {
                        gemm_lookup<BITS>(sel[q], pool[q], tb[p], lo[q], hi[q]);
                    } else {
                        uint32_t o0, o1;
                        decode_interleave(lo[q], hi[q], o0, o1);
                        asm volatile("" : "+v"(o0), "+v"(o1));     // here, and no later
                        nxt.op[p][0][t] = o0; nxt.op[p][1][t] = o1;
                    }
                }
            });
        };
        unrolled<WSTEPS>([&](auto st_) __attribute__((always_inline)) {
            constexpr int st = decltype(st_)::value, f = D * WSTEPS + st, j = f / T, blk = f % T, fa = f + AHEAD;
            if constexpr (fa == 4 * T || fa == 8 * T) {
                vmem_wait<T>();                  // this wave's copies of the next quarter have landed ...
                __builtin_amdgcn_s_barrier();      // ... and everybody else's
                asm volatile("" ::: "memory");
            }
            window[fa % WIN] = fa < 8 * T ? lds_read<(fa < 8 * T ? fa : 0) * 1024>(base[U]) : lds_read<(fa < 8 * T ? 0 : fa - 8 * T) * 1024>(base[U ^ 1]);
            lds_wait<AHEAD>();
            __builtin_amdgcn_sched_barrier(0);
            mfma_acc<blk, false>(cur.op[0][j & 1], window[f % WIN]);
            gap(std::integral_constant<int, PAIRS * st>{});
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (PAIRS == 2) {
                mfma_acc<T + blk, false>(cur.op[PAIRS - 1][j & 1], window[f % WIN]);
                gap(std::integral_constant<int, 2 * st + 1>{});
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // unit u from register set r; ro: the next unit's words.  src: chunk of the next unit; c2, h2: the unit after that
    auto unit = [&](auto U_, GemmTileRegs<BITS, PAIRS> &r, GemmTileRegs<BITS, PAIRS> &ro, __amdgpu_buffer_rsrc_t src, int c2, int h2) __attribute__((always_inline)) {
        word(U_, I0{}, I1{}, wa, wb, r, src);
        word(U_, I1{}, I2{}, wb, wa, r, src);
        word(U_, I2{}, I3{}, wa, wb, r, src);
        high_bits(ro);
        load_words(r, c2, h2);
        word(U_, I3{}, I0{}, wb, wa, ro, src);
    };
    if constexpr (SPLIT == 1) {
        for (int c = 0; c < kc; ++c) {
            const int cn = min(c + 1, kc - 1);
            unit(I0{}, r0, r1, chunk_at(c), cn, 0);
            unit(I1{}, r1, r0, chunk_at(cn), cn, 1);
        }
    } else {
        for (int c = 0; c < kc; c += 2) {
            const int c1 = min(c + 1, kc - 1), c2 = min(c + 2, kc - 1), c3 = min(c + 3, kc - 1);
            unit(I0{}, r0, r1, chunk_at(c1), c2, kh);
            if (c + 1 >= kc) break;
            unit(I1{}, r1, r0, chunk_at(c2), c3, kh);
        }
    }
    // The reads and copies issued past the end (of the last chunk again) are used by nobody: they must land before their registers and the ring are used for
    // something else.
    if constexpr (WIN == 8)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+v"(window[0]), "+v"(window[1]), "+v"(window[2]), "+v"(window[3]), "+v"(window[4]), "+v"(window[5]), "+v"(window[6]), "+v"(window[7]) : : "memory");
    else
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+v"(window[0]), "+v"(window[1]), "+v"(window[2]), "+v"(window[3]) : : "memory");
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");     // (a matrix instruction's registers are read by assembly text below)
    __syncthreads();

    // output: accumulator register 4 g + i of lane l: row 8 g + 4 (l / 32) + i of the pair, token l % 32
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    if constexpr (SPLIT == 1) {
        unrolled<T>([&](auto b_) __attribute__((always_inline)) {
            constexpr int b = decltype(b_)::value;
            uint8_t *const out = lds + (wave * 2 + (b & 1)) * (32 * kWideOutStride);
            unrolled<PAIRS>([&](auto p_) __attribute__((always_inline)) {
                constexpr int p = decltype(p_)::value;
                const float16v v = read_acc<p * T + b>();
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    half4 o;
#pragma unroll
                    for (int u = 0; u < 4; ++u) o[u] = (_Float16)(v[4 * g + u] * out_scale);
                    *reinterpret_cast<uint2v *>(out + (lane & 31) * kWideOutStride + (32 * p + 8 * g + 4 * (lane >> 5)) * 2) = __builtin_bit_cast(uint2v, o);
                }
            });
            asm volatile("" ::: "memory");      // LDS operations of one wave complete in order; keep the compiler's order too
            const int piece = lane & 7;
            const bool rows_ok = t0 + (piece >> 1) < nt;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int tk = it * 8 + (lane >> 3), m = (tb0 + b) * 32 + tk;
                const uint4v v = *reinterpret_cast<const uint4v *>(out + tk * kWideOutStride + piece * 16);
                if (m < M && rows_ok) *reinterpret_cast<uint4v *>(y + (size_t)m * N + (size_t)t0 * kTileRows + piece * 8) = v;
            }
        });
    } else {
        // Each wave of a row group keeps one pair (PAIRS 1: half of the blocks, the first of an odd number twice), and hands the other to its partner:
        // [row group][kh][block][register quad][lane] float4
        constexpr int KEPT = PAIRS == 2 ? T : (T + 1) / 2;
        float4v *const to = reinterpret_cast<float4v *>(lds) + (size_t)(rgrp * 2 + (kh ^ 1)) * (KEPT * 4 * 64);
        float4v *const from = reinterpret_cast<float4v *>(lds) + (size_t)(rgrp * 2 + kh) * (KEPT * 4 * 64);
        // accumulators of kh = 0: [0, KEPT), of kh = 1: the last KEPT
        constexpr int SECOND = PAIRS * T - KEPT;
        auto put = [&](const float16v &v, int b) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < 4; ++g) to[(b * 4 + g) * 64 + lane] = float4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        };
        if (kh == 0) unrolled<KEPT>([&](auto b) __attribute__((always_inline)) { put(read_acc<SECOND + decltype(b)::value>(), decltype(b)::value); });
        else unrolled<KEPT>([&](auto b) __attribute__((always_inline)) { put(read_acc<decltype(b)::value>(), decltype(b)::value); });
        __syncthreads();
        constexpr int kStride = 32 * 2 + 16;
        uint2v outv[KEPT][4];
        // the sum of a run is kh 0's plus kh 1's in either wave (the addition commutes)
        auto sum = [&](const float16v &own, int b) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4v other = from[(b * 4 + g) * 64 + lane];
                half4 o;
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = (_Float16)((own[4 * g + u] + other[u]) * out_scale);
                outv[b][g] = __builtin_bit_cast(uint2v, o);
            }
        };
        if (kh == 0) unrolled<KEPT>([&](auto b) __attribute__((always_inline)) { sum(read_acc<decltype(b)::value>(), decltype(b)::value); });
        else unrolled<KEPT>([&](auto b) __attribute__((always_inline)) { sum(read_acc<SECOND + decltype(b)::value>(), decltype(b)::value); });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the writes below reuse the bytes just read
        uint8_t *const out = reinterpret_cast<uint8_t *>(from);
#pragma unroll
        for (int b = 0; b < KEPT; ++b)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<uint2v *>(out + (b * 32 + (lane & 31)) * kStride + (8 * g + 4 * (lane >> 5)) * 2) = outv[b][g];
        asm volatile("" ::: "memory");
        const int piece = lane & 3, first = t0 + (PAIRS == 2 ? 2 * kh : 0), block = PAIRS == 2 ? 0 : kh * SECOND;
        const bool rows_ok = first + (piece >> 1) < nt;
#pragma unroll
        for (int it = 0; it < 2 * KEPT; ++it) {
            const int tk = it * 16 + (lane >> 2), m = (tb0 + block) * 32 + tk;
            const uint4v v = *reinterpret_cast<const uint4v *>(out + tk * kStride + piece * 16);
            if (m < M && rows_ok) *reinterpret_cast<uint4v *>(y + (size_t)m * N + (size_t)first * kTileRows + piece * 8) = v;
        }
    }
}

// The life of a workgroup of a launch whose columns have B blocks and B - 1.  The tile is found before either body begins: inside the loop over the layers
// the compiler moved what a lane's position gives in front of it and kept it through the products, up to 40 registers, in eight kernels some of them in accumulation
// registers.  Now none are, with 4 vector registers or more to spare; the same time.
template <int BITS, int B, int SPLIT, int PAIRS>
__device__ __forceinline__ void wide_workgroup(const GemmBatch &batch, uint32_t block, uint8_t *lds)   // lds: wide_lds_bytes of B blocks
{
    const WideTileAt at = wide_tile_of(batch, block);
    if (at.layer < 0) return;
    const GemmProblem &pb = batch.p[at.layer];
    const int bx = at.tile % pb.grid_rows, by = at.tile / pb.grid_rows;
    if (!at.second) wide_tile<BITS, B, SPLIT, PAIRS>(pb.packed, pb.lutB, pb.xs, pb.y, batch.M, batch.Mpad >> 5, pb.N, pb.K, bx, by * B, lds, pb.out_scale);
    else if constexpr (B > 1) wide_tile<BITS, B - 1, SPLIT, PAIRS>(pb.packed, pb.lutB, pb.xs, pb.y, batch.M, batch.Mpad >> 5, pb.N, pb.K, bx, batch.tiles.big * B + by * (B - 1), lds, pb.out_scale);
}

}  // namespace lcd
