// The large-tile prefill kernel's workgroup (gfx950).
//
// This path is a dense contraction, so it runs on v_mfma_f32_32x32x16_f16 with fp32
// accumulators (the 32x32 shape reaches the matrix peak from a single wave per SIMD; the 16x16
// shape does not).  Output tile per workgroup: 256 rows x 128 tokens, 8 waves: wave w owns rows
// [64*(w%4), +64) as two 32-row pairs, all 128 tokens as four 32-token blocks (8 accumulators of
// 16 registers, held in fixed accumulation registers) and the half w/4 of every 256-column
// chunk; the two waves of a row group add their accumulators through LDS at the end.  Two
// waves per SIMD keep the vector pipe (the dequantiser) near its full issue rate, which a single
// wave cannot reach.
//   * A operand = weights.  Lane L of the matrix instruction supplies row L%32 and 8 of the
//     step's 16 columns; it loads its own 16 bytes of the packed layout (row tile = pair's first
//     tile + (L>>4)&1) and dequantises them in registers (v_perm_b32 through the row's
//     byte-split codebook), so weights never pass through LDS.
//   * B operand = smoothed activations xs = x * rcp(s) (fp16), prepared once per call by a small
//     kernel in MFMA-operand order, so that the slice one workgroup needs per 256-column chunk
//     is one contiguous 64 KiB block.  It is copied global -> LDS with direct-to-LDS loads,
//     double buffered; every wave reads its B operands from LDS (16 bytes per lane,
//     conflict-free) through a 4-register rotating window.
// Each decoded A operand is used for 4 token blocks, each B operand for 2 row pairs.
// The last tiles of a launch may be cut in two of 128 rows (one pair per wave) so that they spread over more compute units;
// every output's additions keep their order.
#pragma once
#include "lcd_gemm_common.h"

namespace lcd {

constexpr int kGemmRowGroups = 4;   // 64-row groups per workgroup
constexpr int kGemmWaves = 2 * kGemmRowGroups;   // x the two halves of a chunk
constexpr int kGemmPairs = 2;        // 32-row pairs per wave
constexpr int kGemmTokBlks = 4;      // 32-token blocks per workgroup (shared by its waves)
constexpr int kGemmTokens = 32 * kGemmTokBlks;
constexpr int kStageBytes = kGemmTokBlks * 16 * 1024;  // 64 KiB: 4 token blocks x 16 k-steps x 1 KiB

__device__ __forceinline__ void zero_accs()
{
    zero_acc<0>(); zero_acc<1>(); zero_acc<2>(); zero_acc<3>(); zero_acc<4>(); zero_acc<5>(); zero_acc<6>(); zero_acc<7>();
}

// copy one 64 KiB stage: every wave copies 8 KiB as 8 wave-wide 1 KiB direct-to-LDS loads,
// blocks [first, first + count) of them per call (the copy is spread over a word's matrix steps)
__device__ __forceinline__ void stage_copy(const uint8_t *__restrict__ src, uint8_t *lds_dst, int wave, int lane, int first, int count)
{
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (u < first || u >= first + count) continue;
        const int blk = wave * 8 + u;  // 1 KiB block index inside the stage
        __builtin_amdgcn_global_load_lds((glb_u32 *)(src + (size_t)blk * 1024 + lane * 16),
                                         (lds_u32 *)(lds_dst + blk * 1024), 16, 0, 0);
    }
}

// B operands (16 bytes per lane) rotate through a window of four registers: the read for
// matrix step s+3 is issued while step s computes.  A stage holds blocks
// [token block 4][half 2][k-step 8] of 1 KiB.  The reads and the waits for them are written out
// (LDS reads of a wave return in order, so "at most n newer reads outstanding" is the exact
// condition for a window slot; left to itself the compiler waited for ALL outstanding reads at
// every fourth step, which emptied the window each time).
struct BWindow { uint4v w[4]; };

// `base` = 32-bit LDS address of (stage + half * 8 KiB + the lane's 16 bytes)
template <int G, int TBLK>
__device__ __forceinline__ uint4v read_b(uint32_t base)
{
    uint4v v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(base), "n"((TBLK * 16 + G) * 1024) : "memory");
    return v;
}
// Decoded A operands of one packed word: [pair][k-step of the word].
template <int PAIRS> struct WordOps { uint4v op[PAIRS][2]; };

// One packed word per pair (16 weights per lane) = two k-steps x 4 token blocks = 8 matrix steps
// of PAIRS MFMAs.  The word's operands `cur` were decoded during the previous word; each matrix step
// also decodes one eighth of the NEXT words (word DN of `rn`) into `nxt`, so that vector and
// matrix instructions alternate in every wave's stream instead of coming in bursts (two waves of
// a SIMD leave a barrier in phase; with bursts both would decode, then both would multiply).
// COPY: the step also issues its share of the next stage's global -> LDS copy.
// On entry the B window holds steps 0..2 of this word; on exit steps 0..2 of the next word of the
// chunk (the caller primes it again after the last word).
template <int BITS, int PAIRS, int D, int DN, bool COPY>
__device__ __forceinline__ void gemm_word(const WordOps<PAIRS> &cur, WordOps<PAIRS> &nxt, const GemmTileRegs<BITS, PAIRS> &rn,
                                          const HighBits (&hbn)[PAIRS], const typename GemmTables<BITS>::type (&tb)[PAIRS],
                                          uint32_t bbase, BWindow &bw,
                                          const uint8_t *copy_src, uint8_t *copy_dst, int wave, int lane)
{
#define LCD_GEMM_FENCE __builtin_amdgcn_sched_barrier(0);
    uint32_t sel = 0, pool = 0, lo = 0, hi = 0, o0, o1;
    /* quarter Q of the next words is decoded by matrix steps EACH * Q .. EACH * Q + EACH - 1 */
    constexpr int EACH = 2 / PAIRS;
#define LCD_GEMM_STEP(ST)                                                                                   \
    {                                                                                                       \
        constexpr int st = ST, a = st >> 2, blk = st & 3, nx = st + 3;                                      \
        constexpr int qt = st / EACH, qn = st == 7 ? 0 : (st + 1) / EACH;                                   \
        constexpr bool first = st % EACH == 0, last = (st + 1) % EACH == 0;                                 \
        /* prefetch step st+3 into the slot that step st-1 used */                                          \
        if (nx < 8) bw.w[nx & 3] = read_b<2 * D + (nx >> 2), (nx & 3)>(bbase);                              \
        else if (D < 3) bw.w[nx & 3] = read_b<(2 * D + 2) & 7, (nx - 8) & 3>(bbase);                        \
        if (st == 0) gemm_select<BITS, DN, 0>(rn, 0, hbn[0], sel, pool);                                    \
        /* reads newer than this step's operand: 3, fewer at the end of a chunk's last word */             \
        lds_wait<(D < 3 || st <= 4) ? 3 : 7 - st>();                                                        \
        mfma_acc<blk>(cur.op[0][a], bw.w[st & 3]);                                                          \
        /* the vector work of the step is split behind the two matrix instructions: the second one     */ \
        /* cannot issue before the first has left the pipe, and a wave issues in order.  Lookups of     */ \
        /* quarter st, then the selector of quarter st+1, then the interleave: dependent instructions   */ \
        /* stay a few issue slots apart.                                                                 */ \
        if (COPY && copy_src) stage_copy(copy_src, copy_dst, wave, lane, st, 1);                            \
        if (first) gemm_lookup<BITS>(sel, pool, tb[qt >> 2], lo, hi);                                       \
        LCD_GEMM_FENCE                                                                                      \
        if constexpr (PAIRS == 2) mfma_acc<4 + blk>(cur.op[PAIRS - 1][a], bw.w[st & 3]);                    \
        if (last) {                                                                                         \
            if (st < 7) gemm_select<BITS, DN, (qn & 3)>(rn, qn >> 2, hbn[qn >> 2], sel, pool);              \
            decode_interleave(lo, hi, o0, o1);                                                              \
            nxt.op[qt >> 2][0][qt & 3] = o0; nxt.op[qt >> 2][1][qt & 3] = o1;                               \
        }                                                                                                   \
        LCD_GEMM_FENCE                                                                                      \
    }
    LCD_GEMM_STEP(0) LCD_GEMM_STEP(1) LCD_GEMM_STEP(2) LCD_GEMM_STEP(3)
    LCD_GEMM_STEP(4) LCD_GEMM_STEP(5) LCD_GEMM_STEP(6) LCD_GEMM_STEP(7)
#undef LCD_GEMM_STEP
}


// One output tile (row block bx of 128 * PAIRS rows, token block by) of one layer: the whole life of a workgroup.
// PAIRS 1: half a tile, the same additions in the same order for every output.
template <int BITS, int PAIRS>
__device__ __forceinline__ void gemm_tile(const uint8_t *__restrict__ packed_, const uint8_t *__restrict__ lutB, const uint8_t *__restrict__ xs,
                                          uint16_t *__restrict__ y, int M, int Mpad, int N, int K, int bx, int by, uint8_t *lds,
                                          float out_scale)   // 1, or the quantisation step when xs holds INT8 codes (Eq. 11)
{
    constexpr uint32_t TB = kTileRows * kTileCols * BITS / 8;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keeps addresses scalar
    const int kc = K / kTileCols, nt = N / kTileRows;
    const int rgrp = wave & (kGemmRowGroups - 1), khalf = wave >> 2;     // row group and chunk half of this wave
    const int t0 = (bx * kGemmRowGroups + rgrp) * (2 * PAIRS);           // first row tile of this wave
    const int tb0 = by * kGemmTokBlks;                                   // first 32-token block of this workgroup
    const int boff = lane * 16;                                           // lane's 16 bytes inside a 1 KiB operand block
    const __amdgpu_buffer_rsrc_t packed = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(packed_), 0, (uint32_t)nt * (uint32_t)kc * TB, 0x00020000);

    // activations of chunk c for this workgroup's 128 tokens: one contiguous 64 KiB block
    const size_t chunk_stride = (size_t)(Mpad >> 5) * 16 * 1024;
    const uint8_t *xs_base = xs + (size_t)tb0 * 16 * 1024;

    typename GemmTables<BITS>::type tb[PAIRS];
    load_gemm_tables<BITS>(tb, lutB, t0, nt, lane);
    zero_accs();

    GemmTileRegs<BITS, PAIRS> r0, r1;
    load_gemm_tiles<BITS>(r0, packed, t0, nt, kc, 0, khalf, lane);
    stage_copy(xs_base, lds, wave, lane, 0, 8);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    auto high_bits = [&](const GemmTileRegs<BITS, PAIRS> &r, HighBits (&hb)[PAIRS]) {
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            hb[p] = HighBits{0u, 0u};
            if (BITS == 3) hb[p] = regroup_high(r.hi[p]);
        }
    };

    BWindow bw;
    WordOps<PAIRS> wa, wb;          // operands of the current / next word, swapping roles word by word
    HighBits hb[PAIRS], hbn[PAIRS];
    // Chunk c is computed from LDS stage c&1 and register set r; word D's matrix steps decode word
    // D+1, the last word's decode the first word of chunk c+1 (set rn, loaded at the top of chunk
    // c).  The copy of chunk c+1's stage is issued during word 0 (the other stage was released by
    // the barrier that ended chunk c-1) and has the whole chunk to land: one wait + one barrier
    // per chunk, after which the B window is primed from the new stage.
    auto compute = [&](const GemmTileRegs<BITS, PAIRS> &r, const GemmTileRegs<BITS, PAIRS> &rn, const uint8_t *stage,
                       uint8_t *other_stage, const uint8_t *copy_src) {
        const uint32_t bbase = lds_address(stage) + khalf * 8 * 1024 + boff;
        const uint32_t obase = lds_address(other_stage) + khalf * 8 * 1024 + boff;
        gemm_word<BITS, PAIRS, 0, 1, true>(wa, wb, r, hb, tb, bbase, bw, copy_src, other_stage, wave, lane);
        gemm_word<BITS, PAIRS, 1, 2, false>(wb, wa, r, hb, tb, bbase, bw, nullptr, nullptr, wave, lane);
        gemm_word<BITS, PAIRS, 2, 3, false>(wa, wb, r, hb, tb, bbase, bw, nullptr, nullptr, wave, lane);
        high_bits(rn, hbn);
        gemm_word<BITS, PAIRS, 3, 0, false>(wb, wa, rn, hbn, tb, bbase, bw, nullptr, nullptr, wave, lane);
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) hb[p] = hbn[p];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();   // the next stage has landed for every wave, and every wave is done with this one
        bw.w[0] = read_b<0, 0>(obase);
        bw.w[1] = read_b<0, 1>(obase);
        bw.w[2] = read_b<0, 2>(obase);
    };

    // prologue: B operands of the first three steps, operands of the first word
    {
        const uint32_t base0 = lds_address(lds) + khalf * 8 * 1024 + boff;
        bw.w[0] = read_b<0, 0>(base0);
        bw.w[1] = read_b<0, 1>(base0);
        bw.w[2] = read_b<0, 2>(base0);
    }
    high_bits(r0, hb);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p) {
        if constexpr (BITS == 4) decode_word4(r0.lo[p][0], r0.hi4[p][0], tb[p], wa.op[p][0], wa.op[p][1]);
        else decode_word<BITS, 0>(r0.lo[p][0], hb[p], tb[p], wa.op[p][0], wa.op[p][1]);
    }
    for (int c = 0; c < kc; c += 2) {
        // even chunk: compute from stage 0 / r0 while chunk c+1 lands in stage 1 / r1
        const bool more1 = c + 1 < kc;
        if (more1) load_gemm_tiles<BITS>(r1, packed, t0, nt, kc, c + 1, khalf, lane);
        compute(r0, r1, lds, lds + kStageBytes, more1 ? xs_base + (size_t)(c + 1) * chunk_stride : nullptr);
        if (!more1) break;
        const bool more2 = c + 2 < kc;
        if (more2) load_gemm_tiles<BITS>(r0, packed, t0, nt, kc, c + 2, khalf, lane);
        compute(r1, r0, lds + kStageBytes, lds, more2 ? xs_base + (size_t)(c + 2) * chunk_stride : nullptr);
    }

    // The two waves of a row group hold partial sums over the two halves of every chunk.  Each keeps
    // one 32-row pair (half a tile: two token blocks of the only pair) and hands the other accumulators to its partner
    // through LDS (the stages are free now): per row group two 16 KiB areas, area h read by the wave with khalf == h,
    // [accumulator 4][register quad 4][lane] float4.
    // The accumulator reads below are assembly text too: the distance the hardware requires between a
    // matrix instruction's register write and a vector instruction's read of it (19 wait states for
    // the 16-pass instruction) is kept here by hand, once per workgroup.
    // (The window reads issued after the last chunk's barrier are used by nobody: they must still land before their registers
    // are used for something else.)
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bw.w[0]), "+v"(bw.w[1]), "+v"(bw.w[2]) : : "memory");
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    float4v *area_in = reinterpret_cast<float4v *>(lds) + (size_t)(rgrp * 2 + khalf) * (4 * 4 * 64);
    float4v *area_out = reinterpret_cast<float4v *>(lds) + (size_t)(rgrp * 2 + (khalf ^ 1)) * (4 * 4 * 64);
    auto put_acc = [&](const float16v &v, int slot) {
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) area_out[(slot * 4 + rg) * 64 + lane] = float4v{v[4 * rg], v[4 * rg + 1], v[4 * rg + 2], v[4 * rg + 3]};
    };
    constexpr int KEPT = 2 * PAIRS;   // accumulators (token blocks) a wave keeps
    if constexpr (PAIRS == 2) {
        if (khalf == 0) { put_acc(read_acc<4>(), 0); put_acc(read_acc<5>(), 1); put_acc(read_acc<6>(), 2); put_acc(read_acc<7>(), 3); }
        else            { put_acc(read_acc<0>(), 0); put_acc(read_acc<1>(), 1); put_acc(read_acc<2>(), 2); put_acc(read_acc<3>(), 3); }
    } else {
        if (khalf == 0) { put_acc(read_acc<2>(), 0); put_acc(read_acc<3>(), 1); }
        else            { put_acc(read_acc<0>(), 0); put_acc(read_acc<1>(), 1); }
    }
    __syncthreads();

    // Sum of the two halves, rounded once to fp16.  Accumulator register r of lane l is row
    // 8*(r/4) + 4*(l/32) + r%4 of the pair, token l%32: four consecutive rows of one token per
    // register quad, i.e. 8-byte pieces of 32 different output rows per store instruction.  Stored
    // like that, every 128-byte line of y is written in 16 pieces and the end of the kernel waits
    // on the L2's request rate; so the wave first turns its 32 rows x 128 tokens into
    // [token][row] order through the area it has just read (nobody else touches it any more) and
    // then writes 64 contiguous bytes per token: 4 lanes x 16 bytes, the other half of the line
    // coming from its partner.
    const int tok = lane & 31, lh = lane >> 5;
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    constexpr int kOutStride = 32 * 2 + 16;   // bytes per token row of the tile (16-byte aligned, spreads the banks)
    uint8_t *tile_out = reinterpret_cast<uint8_t *>(area_in);
    uint2v outv[KEPT][4];
    auto sum_acc = [&](const float16v &own, int slot) {
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
            const float4v other = area_in[(slot * 4 + rg) * 64 + lane];
            half4 o;
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = (_Float16)((own[4 * rg + u] + other[u]) * out_scale);
            outv[slot][rg] = __builtin_bit_cast(uint2v, o);
        }
    };
    if constexpr (PAIRS == 2) {
        if (khalf == 0) { sum_acc(read_acc<0>(), 0); sum_acc(read_acc<1>(), 1); sum_acc(read_acc<2>(), 2); sum_acc(read_acc<3>(), 3); }
        else            { sum_acc(read_acc<4>(), 0); sum_acc(read_acc<5>(), 1); sum_acc(read_acc<6>(), 2); sum_acc(read_acc<7>(), 3); }
    } else {
        if (khalf == 0) { sum_acc(read_acc<0>(), 0); sum_acc(read_acc<1>(), 1); }
        else            { sum_acc(read_acc<2>(), 0); sum_acc(read_acc<3>(), 1); }
    }
    // every read above must precede the writes below, which reuse the same bytes: the wait orders
    // them for the compiler too (the two sides use different vector types)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int blk = 0; blk < KEPT; ++blk) {
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
            *reinterpret_cast<uint2v *>(tile_out + (blk * 32 + tok) * kOutStride + (8 * rg + 4 * lh) * 2) = outv[blk][rg];
    }
    asm volatile("" ::: "memory");               // LDS operations of one wave complete in order; keep the compiler's order too
    const int r4 = lane & 3;                       // which 8 rows of the pair's 32
    const int tile_first = t0 + (PAIRS == 2 ? 2 * khalf : 0);   // first 16-row tile of this wave's pair
    const bool rows_ok = tile_first + (r4 >> 1) < nt;   // N is a multiple of 16: 8 rows are all inside or all outside
#pragma unroll
    for (int it = 0; it < 2 * KEPT; ++it) {
        const int tk = it * 16 + (lane >> 2);
        const uint4v v = *reinterpret_cast<const uint4v *>(tile_out + tk * kOutStride + r4 * 16);
        const int m = tb0 * 32 + (PAIRS == 2 ? 0 : 64 * khalf) + tk;
        if (m < M && rows_ok) *reinterpret_cast<uint4v *>(y + (size_t)m * N + (size_t)tile_first * kTileRows + r4 * 8) = v;
    }
}

// XCD-aware tile order.  Workgroup ids go round-robin over the 8 XCDs, each with its own L2.
// Output tiles are numbered token-block-major and cut into 8 contiguous runs, one per XCD, so
// the workgroups that are resident on an XCD at the same time share one or two 128-token
// blocks of activations (1 MiB each at K = 4096), which then stay in that XCD's 4 MiB L2.
template <int BITS>
__device__ __forceinline__ void gemm_workgroup(const GemmBatch &batch, uint32_t block, uint8_t *lds)   // lds: 2 stages x 64 KiB
{
    const int xcd = (int)(block % kXcds);
    int pos = (int)(block / kXcds);
    const int past = pos - batch.tail_begin;       // from here on a place of the queue is two workgroups, half a tile each
    if (past >= 0) pos = batch.tail_begin + (past >> 1);
    int pi = 0;
    for (int i = 1; i < batch.count; ++i) pi += pos >= batch.p[i].queue_begin ? 1 : 0;   // queue_begin grows with i
    const GemmProblem pb = batch.p[pi];
    const int out_tile = xcd * pb.tiles_per_xcd + (pos - pb.queue_begin);
    if (out_tile >= pb.grid_rows * (batch.Mpad / kGemmTokens)) return;
    const int bx = out_tile % pb.grid_rows, by = out_tile / pb.grid_rows;
    if (past < 0) {
        gemm_tile<BITS, kGemmPairs>(pb.packed, pb.lutB, pb.xs, pb.y, batch.M, batch.Mpad, pb.N, pb.K, bx, by, lds, pb.out_scale);
        return;
    }
    const int half = 2 * bx + (past & 1);
    if (half * (kGemmRowGroups * 32) >= pb.N) return;   // uniform over the workgroup
    gemm_tile<BITS, 1>(pb.packed, pb.lutB, pb.xs, pb.y, batch.M, batch.Mpad, pb.N, pb.K, half, by, lds, pb.out_scale);
}

}  // namespace lcd
