// The split prefill kernel's workgroup (gfx950): layers of so few outputs that larger tiles would leave compute units idle.
//
// Output tile per workgroup: 32 or 64 rows x 32..128 tokens; its 8 waves all own the whole tile and
// split K: wave w takes the 128-column halves w, w + 8, ... of the chunks.  As in the wide kernel the
// packed words are dequantised in registers straight into A operands of v_mfma_f32_32x32x16_f16, but no
// B operand is shared between waves, so a wave streams its own through a private ring in LDS
// (direct-to-LDS loads, RING k-steps ahead, read back through a rotating window of four registers)
// and waits for nobody: no barrier inside K.  At the end the 8 partial tiles are added through
// LDS in the order of the waves, one 32-token block after the other.  The order of the additions of one output
// depends on K alone, so every tile shape gives the same bits.
//
// What bounds it: the activations' way from L2 into LDS (every wave reads its own: 2 bytes per token and
// column and workgroup, 75..98 GB/s per compute unit), with 32 tokens x 64 rows the dequantiser; around it about 2 us
// of start-up and epilogue per workgroup and about 4 us of smoothing launch per call.  That is why the tile is
// as small as fills the compute units.  Measured against tiles of 256 x 128 (16..86 workgroups on these; another kernel), per call: 11008 x 4096,
// 4 bits, 100 tokens 57 -> 22 us; 7B block (q, k, v | o | gate, up | down), 2 bits and INT8 codes, 333 tokens
// 298 -> 185 us.  Rings of 5 or 6 k-steps instead of 4 and tiles of 128 rows x 64..128 tokens whose activations all waves share gained nothing
// over the range (the latter 1.2 to 1.3 on some groups, 0.66 to 1 on the others and on single layers).
#pragma once
#include <type_traits>
#include "lcd_gemm_common.h"

namespace lcd {

constexpr int kSplitWaves = 8;

// k-steps (16 columns) a wave's ring holds
template <int PAIRS, int TBLK> constexpr int split_ring() { return TBLK >= 3 ? 4 : 8; }
// a partial block in LDS: [token 32][row], rows padded by 16 bytes (spreads the banks)
template <int PAIRS> constexpr int split_part_stride() { return 32 * PAIRS + 4; }
template <int PAIRS> constexpr int split_part_bytes() { return 32 * split_part_stride<PAIRS>() * 4; }
template <int PAIRS, int TBLK>
constexpr size_t split_lds_bytes()
{
    const size_t ring = (size_t)kSplitWaves * split_ring<PAIRS, TBLK>() * TBLK * 1024;
    const size_t parts = (size_t)2 * kSplitWaves * split_part_bytes<PAIRS>();
    return ring > parts ? ring : parts;
}

// 1 KiB (16 bytes per lane) from byte `offset` + OFFSET of a buffer to the LDS bytes at `to`.  The instruction adds its own
// offset (OFFSET) to the LDS address as well as to the buffer's.
template <int OFFSET>
__device__ __forceinline__ void copy_block(__amdgpu_buffer_rsrc_t from, uint32_t to, uint32_t lane_offset, uint32_t offset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (lds_u32 *)(uintptr_t)(to - OFFSET), 16, lane_offset, offset, OFFSET, 0);
}

template <int BITS, int PAIRS, int TBLK>
__device__ __forceinline__ void split_workgroup(const GemmBatch &batch, uint32_t block, uint8_t *lds)   // lds: split_lds_bytes
{
    constexpr uint32_t TB = kTileRows * kTileCols * BITS / 8;
    constexpr int RING = split_ring<PAIRS, TBLK>();
    constexpr int STEPS = 8 * TBLK;             // B blocks of a unit (128 columns): 8 k-steps x token blocks
    constexpr int WSTEPS = 2 * TBLK;            // ... of a packed word (two k-steps)

    // layer and output tile: every XCD has a queue of workgroups, each layer a run of places in it
    const int xcd = (int)(block % kXcds), pos = (int)(block / kXcds);
    int pi = 0;
    for (int i = 1; i < batch.count; ++i) pi += pos >= batch.p[i].queue_begin ? 1 : 0;   // queue_begin grows with i
    const GemmProblem pb = batch.p[pi];
    const int out_tile = xcd * pb.tiles_per_xcd + (pos - pb.queue_begin);
    const int M = batch.M, mblk = batch.Mpad >> 5;
    const int col_tiles = ((M + 31) / 32 + TBLK - 1) / TBLK;
    if (out_tile >= pb.grid_rows * col_tiles) return;
    const int bx = out_tile % pb.grid_rows, by = out_tile / pb.grid_rows;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keeps addresses scalar
    const int kc = pb.K / kTileCols, nt = pb.N / kTileRows, units = 2 * kc;
    const int t0 = bx * 2 * PAIRS;
    const __amdgpu_buffer_rsrc_t packed = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(pb.packed), 0, (uint32_t)nt * (uint32_t)kc * TB, 0x00020000);

    // Activations of unit u (chunk u / 2, half u % 2), token block b: 8 KiB, 1 KiB per k-step.  Blocks past the padded tokens
    // (the last tile of a layer, never stored) are read as the last block.  Everything but the lane's 16 bytes is wave-uniform
    // and travels as the scalar offset (the host takes this kernel only where xs is smaller than 4 GiB).
    uint32_t block_at[TBLK];
#pragma unroll
    for (int b = 0; b < TBLK; ++b) block_at[b] = (uint32_t)min(by * TBLK + b, mblk - 1) * (16 * 1024);
    auto unit_src = [&](int u) { return ((uint32_t)(u >> 1) * (uint32_t)mblk * 2 + (u & 1)) * (8 * 1024); };
    const __amdgpu_buffer_rsrc_t xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(pb.xs), 0, (uint32_t)kc * (uint32_t)mblk * (16 * 1024), 0x00020000);
    const uint32_t ring = lds_address(lds) + wave * (RING * TBLK * 1024);
    const uint32_t ring_base = ring + lane * 16;
    // k-step J of the unit at `src` into its slot
    auto copy_step = [&](uint32_t src, auto J) __attribute__((always_inline)) {
        constexpr int j = decltype(J)::value;
        uint32_t to = ring;
        asm volatile("" : "+s"(src), "+s"(to));   // one scalar addition per copy instead of an address kept for each
#pragma unroll
        for (int b = 0; b < TBLK; ++b)
            copy_block<(j & 3) * 1024>(xs, to + ((j % RING) * TBLK + b) * 1024, lane * 16, src + block_at[b] + (j & 4) * 1024);
    };

    const GemmRows<PAIRS> rows = gemm_rows<BITS, PAIRS>(t0, nt, kc, lane);
    auto load_words = [&](GemmTileRegs<BITS, PAIRS> &r, int u) __attribute__((always_inline)) { load_gemm_words<BITS>(r, packed, rows, (uint32_t)(u >> 1), u & 1); };

    // 4 bits, 64 rows: no registers for two units' words; words 0, 1 and words 2, 3 of the next unit are loaded when
    // the present unit's have been decoded
    constexpr bool HALVES = BITS == 4 && PAIRS == 2;
    auto load_half = [&](GemmTileRegs<BITS, PAIRS> &r, int u, auto H_) __attribute__((always_inline)) {
        constexpr int H = decltype(H_)::value;
        const uint32_t o = (uint32_t)(u >> 1) * TB + (u & 1) * 512 + 8 * H;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const uint2v a = __builtin_amdgcn_raw_buffer_load_b64(packed, rows.at[p], o, kGemmWeightPolicy);
            const uint2v b = __builtin_amdgcn_raw_buffer_load_b64(packed, rows.at[p], o + 1024, kGemmWeightPolicy);
            r.lo[p][2 * H] = a[0]; r.lo[p][2 * H + 1] = a[1];
            r.hi4[p][2 * H] = b[0]; r.hi4[p][2 * H + 1] = b[1];
        }
    };

    typename GemmTables<BITS>::type tb[PAIRS];
    load_gemm_tables<BITS>(tb, pb.lutB, t0, nt, lane);
    unrolled<PAIRS * TBLK>([&](auto i) __attribute__((always_inline)) { zero_acc<decltype(i)::value>(); });

    uint4v window[4];                    // B operands: the read of block f + 3 is issued while block f is multiplied
    struct Ops { uint4v op[PAIRS][2]; };  // A operands of one packed word: [pair][k-step of the word]
    Ops wa, wb;
    HighBits hb[PAIRS], hbn[PAIRS];
    auto high_bits = [&](const GemmTileRegs<BITS, PAIRS> &r, HighBits (&h)[PAIRS]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            h[p] = HighBits{0u, 0u};
            if (BITS == 3) h[p] = regroup_high(r.hi[p]);
        }
    };

    // One packed word per pair: WSTEPS steps of PAIRS matrix instructions; the steps also decode the next word (word DN of
    // `rn`), a share each.  LAST: the wave's last unit (no copies or reads beyond it).
    auto word = [&](auto D_, auto DN_, auto LAST_, const Ops &cur, Ops &nxt, const GemmTileRegs<BITS, PAIRS> &rn,
                    const HighBits (&hn)[PAIRS], uint32_t src, uint32_t src_next) __attribute__((always_inline)) {
        constexpr int D = decltype(D_)::value, DN = decltype(DN_)::value;
        constexpr bool LAST = decltype(LAST_)::value;
        unrolled<WSTEPS>([&](auto st_) __attribute__((always_inline)) {
            constexpr int st = decltype(st_)::value, f = D * WSTEPS + st, j = f / TBLK, blk = f % TBLK;
            constexpr int ahead = f + 3, ja = ahead / TBLK, issued = LAST && j - 1 + RING > 7 ? 7 : j - 1 + RING;
            if constexpr (ahead < STEPS || !LAST) {
                // the first read of k-step ja: its copy must have landed (copies land in order; loads of packed words that
                // were issued in between only make the wait stricter)
                if constexpr (ahead % TBLK == 0) vmem_wait<(issued - ja) * TBLK>();
                window[ahead & 3] = lds_read<((ja % RING) * TBLK + ahead % TBLK) * 1024>(ring_base);
            }
            lds_wait<(LAST && STEPS - 1 - f < 3) ? STEPS - 1 - f : 3>();
            __builtin_amdgcn_sched_barrier(0);
            mfma_acc<blk>(cur.op[0][j & 1], window[f & 3]);
            // this step's share of the next word's 4 * PAIRS quarters
            if constexpr (!(LAST && D == 3)) {
                constexpr int q0 = st * 4 * PAIRS / WSTEPS, q1 = (st + 1) * 4 * PAIRS / WSTEPS;
                unrolled<q1 - q0>([&](auto qi) __attribute__((always_inline)) {
                    constexpr int q = q0 + decltype(qi)::value, p = q >> 2, t = q & 3;
                    uint32_t sel = 0, pool = 0, lo, hi, o0, o1;
                    gemm_select<BITS, DN, t>(rn, p, hn[p], sel, pool);
                    gemm_lookup<BITS>(sel, pool, tb[p], lo, hi);
                    decode_interleave(lo, hi, o0, o1);
                    nxt.op[p][0][t] = o0; nxt.op[p][1][t] = o1;
                });
            }
            if constexpr (PAIRS == 2) {
                __builtin_amdgcn_sched_barrier(0);
                mfma_acc<TBLK + blk>(cur.op[PAIRS - 1][j & 1], window[f & 3]);
            }
            // every block of k-step j has arrived in registers: its slot takes k-step j + RING
            if constexpr (blk == TBLK - 1 && (j + RING < 8 || !LAST)) {
                constexpr int jc = j + RING;
                copy_step(jc < 8 ? src : src_next, std::integral_constant<int, jc>{});
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using W0 = std::integral_constant<int, 0>; using W1 = std::integral_constant<int, 1>;
    using W2 = std::integral_constant<int, 2>; using W3 = std::integral_constant<int, 3>;
    // one unit from register set r; rn receives the packed words of the wave's next unit (HALVES: the same set)
    auto unit = [&](auto LAST_, GemmTileRegs<BITS, PAIRS> &r, GemmTileRegs<BITS, PAIRS> &rn, int u) __attribute__((always_inline)) {
        constexpr bool LAST = decltype(LAST_)::value;
        const int un = u + kSplitWaves;
        if constexpr (!LAST && !HALVES) load_words(rn, un);
        const uint32_t src = unit_src(u), src_next = unit_src(un);
        word(W0{}, W1{}, LAST_, wa, wb, r, hb, src, src_next);
        if constexpr (!LAST && HALVES) load_half(rn, un, W0{});
        word(W1{}, W2{}, LAST_, wb, wa, r, hb, src, src_next);
        word(W2{}, W3{}, LAST_, wa, wb, r, hb, src, src_next);
        if constexpr (!LAST && HALVES) load_half(rn, un, W1{});
        if constexpr (!LAST) high_bits(rn, hbn);
        word(W3{}, W0{}, LAST_, wb, wa, rn, hbn, src, src_next);
        if constexpr (!LAST) {
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) hb[p] = hbn[p];
        }
    };

    if (wave < units) {
        GemmTileRegs<BITS, PAIRS> r0, r1;
        load_words(r0, wave);
        unrolled<RING>([&](auto j) __attribute__((always_inline)) { copy_step(unit_src(wave), j); });
        high_bits(r0, hb);
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            if constexpr (BITS == 4) decode_word4(r0.lo[p][0], r0.hi4[p][0], tb[p], wa.op[p][0], wa.op[p][1]);
            else decode_word<BITS, 0>(r0.lo[p][0], hb[p], tb[p], wa.op[p][0], wa.op[p][1]);
        }
        vmem_wait<(RING - 1 - 2 / TBLK) * TBLK>();
        window[0] = lds_read<0>(ring_base);
        window[1] = lds_read<1024>(ring_base);
        window[2] = lds_read<2048>(ring_base);
        int u = wave;
        if constexpr (HALVES) {
            for (; u + kSplitWaves < units; u += kSplitWaves) unit(std::false_type{}, r0, r0, u);
            unit(std::true_type{}, r0, r0, u);
        } else for (;;) {
            if (u + kSplitWaves >= units) { unit(std::true_type{}, r0, r1, u); break; }
            unit(std::false_type{}, r0, r1, u);
            u += kSplitWaves;
            if (u + kSplitWaves >= units) { unit(std::true_type{}, r1, r0, u); break; }
            unit(std::false_type{}, r1, r0, u);
            u += kSplitWaves;
        }
    }

    // ---- partial tiles through LDS, one 32-token block at a time (two buffers, one barrier each); accumulator
    // register 4 g + i of lane l: row 8 g + 4 (l / 32) + i of the pair, token l % 32.
    // The accumulator reads are assembly text: the distance to the last matrix instruction is kept by hand.
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
    __syncthreads();      // every wave has left its ring
    constexpr int STRIDE = split_part_stride<PAIRS>(), PART = split_part_bytes<PAIRS>();
    unrolled<TBLK>([&](auto b_) __attribute__((always_inline)) {
        constexpr int b = decltype(b_)::value;
        uint8_t *buffer = lds + (b & 1) * (kSplitWaves * PART);
        float *mine = reinterpret_cast<float *>(buffer + wave * PART) + (lane & 31) * STRIDE + 4 * (lane >> 5);
        unrolled<PAIRS>([&](auto p_) __attribute__((always_inline)) {
            constexpr int p = decltype(p_)::value;
            const float16v v = read_acc<p * TBLK + b>();
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4v *>(mine + 32 * p + 8 * g) = float4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        });
        __syncthreads();
        const int e = threadIdx.x, tok = e / (8 * PAIRS), rq = e % (8 * PAIRS);   // a quad of rows of one token
        const int m = (by * TBLK + b) * 32 + tok, row = t0 * kTileRows + 4 * rq;
        if (e < 256 * PAIRS && m < M && row < pb.N) {
            const float *src = reinterpret_cast<const float *>(buffer) + tok * STRIDE + 4 * rq;
            float4v sum = *reinterpret_cast<const float4v *>(src);
#pragma unroll
            for (int w = 1; w < kSplitWaves; ++w) sum += *reinterpret_cast<const float4v *>(src + w * (PART / 4));
            typedef _Float16 half4 __attribute__((ext_vector_type(4)));
            half4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (_Float16)(sum[i] * pb.out_scale);
            *reinterpret_cast<half4 *>(pb.y + (size_t)m * pb.N + row) = o;
        }
    });
}

}  // namespace lcd
