// Decode and short-prompt path (2 <= M <= 32 tokens; every M with 4 bits) of the smoothed
// table-lookup product, gfx950: the tokens kernel's workgroup.
//
// A batched product with few tokens: the packed indices are dequantised in registers (v_perm_b32
// through per-row byte-split codebook tables) into the A operand of v_mfma_f32_16x16x32_f16, blocks of
// 16 tokens are its columns, one dequantised operand serves every block.
//
// Work split.  A workgroup owns a contiguous run of row tiles (16 rows) of ONE layer and takes them
// R at a time; its waves (8 or 16) split K, wave w takes the 256-column chunks w, w + W, ...  Per chunk a wave stages
// the activations of its 256 columns once (smoothing, Sec. 3.4, and the turn into operand order through its own piece of
// LDS), then multiplies the chunk of every one of the R row tiles; the accumulators stay in registers over all of K.  No wave waits for another before the end: one
// barrier, then the partial tiles are added, rounded once and stored.  An output is the sum, in order, of 8 sums of two:
// chunks w, w + 16, ... and chunks w + 8, w + 24, ... -- two sets of accumulators of one wave, or one set of two waves.
// The order of the additions of one output depends on K alone -- not on the grouping of layers,
// on R or on the number of tokens -- so grouped, single and captured calls agree bit for bit.
//
// What bounds it: with many row tiles per workgroup the vector pipe (the dequantiser), 0.5 / 0.6 / 0.95 us (2 / 3 / 4 bits) per
// row tile and round of 8 chunks; with one row tile per workgroup the staging of the activations and the latencies in front.
// 16 waves hide one another's staging and latencies better where the registers are there for them: up to three row tiles, and any number
// up to K = 4096, where a wave has one chunk at most: its operands stay (RESIDENT) and row tiles stream past them.  Neither loads of
// tokens that are not there nor loads behind the last chunk are issued: a load out of range takes the time of its addresses.
// us a launch in a graph, every load issued whatever is valid and 8 waves beyond two row tiles / now: q, k, v of a 7B block (3 row tiles), 16 tokens, 2 / 3 / 4
// bits 10.1 / 12.3 / 14.5, 9.1 / 10.7 / 13.8; gate, up (5.4) 12.7 / 16.1 / 21.3, 11.7 / 14.1 / 18.7; o (1) 6.1 / 7.0 / 7.3, 5.5 / 5.8 / 6.8; three tokens, 3 bits:
// q, k, v 10.4, 8.5; gate, up 13.7, 11.3; o 6.0, 4.5; down (K = 11008) 9.9, 8.0.  Two resident chunks per wave (K = 5120, 8192) spill.
//
// Beyond K = 4096 a second pass over the activations costs 4 to 6 us, hence the variant of 14 row tiles (up to 57344 rows on 256 compute units
// in one pass): two layers of 28672 x 8192, 4 tokens, 3 / 4 bits 54.8 / 77.4 -> 44.1 / 64.6.  Its registers
// hold the packed words of a few tiles only, in a ring (2 / 3 / 4 bits: 4, 4, 3 tiles ahead, which is enough of them under way), and at 3 and 4 bits
// no row tables: those are read from LDS one tile ahead.  At 2 bits with 9 to 16 tokens made in the kernel 14 tiles and their tables spill: 12 tiles have
// room for both and serve where they need no more passes, 14 read the tables from LDS too (tables in registers / so: 7 tiles x K = 5120 15.3 / 14.7 us,
// 12 x 5120 21.1 / 20.6, 16 x 5120 30.0 / 28.8, 14 x 6400 31.3 / 29.7, 13 x 5120 21.6 / 21.8, 25 x 4352 39.4 / 39.9).
// Four and five tiles of these have forms of their own, short enough for a copy of the last chunk without loads, and six hold four tiles' words, not all
// (one form of six with all words / so, 16 tokens: 4 tiles x K = 5120 11.0 / 10.0 us, 5 tiles 12.2 / 11.2, 6 tiles 13.3 / 12.9; 6400 13.8 / 12.3, 15.3 / 14.2, 17.0 / 16.5; six
// with the copy spill, 14.6 and 18.2).
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include "lcd_decode.h"

namespace lcd {

constexpr int kStageStride = kTileCols + 8;   // halfs per token row of a wave's stage (+16 B: no bank conflicts)
constexpr int kStageBytes = kTokenBlock * kStageStride * 2;

// Row tiles a variant holds: one, two, as many as leave room for all their packed words of a chunk next to the B operands (32 registers
// per block), the staged activations and the tables, or kManyTiles.
template <int BITS, int TB> constexpr int whole_chunk_tiles() { return BITS == 4 ? (TB == 1 ? 4 : 3) : (TB == 1 ? 6 : 5); }
constexpr int kManyTiles = 14;
template <int BITS> constexpr int ring_tiles() { return BITS == 4 ? 3 : 4; }
constexpr bool ring_of_words(int tiles) { return tiles > 6; }      // (whole_chunk_tiles: up to 6)
template <int BITS, int R, int PAIRS, bool READY> constexpr bool tables_in_lds() { return R == kManyTiles && (BITS != 2 || (PAIRS == 8 && !READY)); }

template <int TB, int R>
constexpr int tokens_wave_bytes() { return R * TB * 1024 > kStageBytes ? R * TB * 1024 : kStageBytes; }
template <int BITS, int TB, int R, int WAVES, int PAIRS, bool READY>
constexpr size_t tokens_lds_bytes() { return (size_t)WAVES * tokens_wave_bytes<TB, R>() + (tables_in_lds<BITS, R, PAIRS, READY>() ? R * kTileRows * row_table_bytes<BITS>() : 0); }

// The life of a workgroup.  PAIRS: pairs of tokens the launch may have per block; smem: tokens_lds_bytes
template <int BITS, int TB, int R, int WAVES, int PAIRS, bool READY, bool RESIDENT>
__device__ __forceinline__ void tokens_workgroup(const uint32_t t0, const uint32_t t1, const uint32_t t2, const uint32_t t3,
                                                 const uint32_t t4, const uint32_t t5, const uint32_t t6, const uint32_t t7,
                                                 const uint16_t *head_x, const float *head_s, const uint32_t head_word, const BucketBatch &batch, uint8_t *smem)
{
    constexpr uint32_t TBYTES = kTileRows * kTileCols * BITS / 8;
    constexpr int NC = BITS == 2 ? 4 : 8;
    constexpr int RING = ring_of_words(R) || (R == 6 && BITS == 2 && PAIRS == 8 && !READY) ? ring_tiles<BITS>() : R;   // row tiles whose words of a chunk are held
    constexpr bool TABLES = tables_in_lds<BITS, R, PAIRS, READY>();
    constexpr bool STRAIGHT = TB == 1 && (R <= 3 || (BITS == 2 && R <= 5)) && !(BITS == 4 && R == 2 && PAIRS == 8);   // short code, and registers left: the last chunk has a copy of its own
    constexpr int SETS = 2 * kBW / WAVES;         // accumulator sets of a wave (see the order of the additions above)
    constexpr int kWaveBytes = tokens_wave_bytes<TB, R>();
    // smem: one piece per wave (its stage, in the end its partial tiles), then the row tables

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keeps addresses scalar
    const int q = lane >> 4, j = lane & 15;
    const int kg = lane & 31, th = lane >> 5;   // staging: 8 columns [8 kg, +8) of the chunk, tokens th, th + 2, ...

    int pi = (head_word & kHeadSingle) ? 0 : layer_of_workgroup(blockIdx.x, t0, t1, t2, t3, t4, t5, t6, t7);
    const uint16_t *x = head_x;
    const float *s = head_s;
    int kc;
    input_of(batch, pi, head_word, x, s, kc);
    const int M = head_tokens(head_word), K = kc * kTileCols;
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(x, (uint32_t)M * (uint32_t)K * 2);
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(s, (uint32_t)K * 4);
    _Float16 *stage = reinterpret_cast<_Float16 *>(smem + wave * kWaveBytes);

    // activations of one chunk as loaded: TB x 8 registers of 8 fp16 numbers.  READY: register g of a block is the B operand of
    // columns 64 q + 8 g .. of the lane's token.  Else: columns 8 kg .., tokens th + 2 mm.
    // The (token pair, chunk) part of the address is wave-uniform and travels as the scalar offset; lanes
    // of a token past the last one read zeros through an offset that is out of range.
    constexpr int XR = READY ? 8 : PAIRS;
    uint4v xr[TB][XR];
    const uint32_t row_bytes = (uint32_t)K * 2;
    const uint32_t x_lane = 16 * kg + th * row_bytes, x_last = th ? kOob : 16u * kg;
    auto load_x = [&](int chunk) __attribute__((always_inline)) {
        uint32_t o = __builtin_amdgcn_readfirstlane((uint32_t)chunk * (kTileCols * 2));
        const int left = __builtin_amdgcn_readfirstlane(chunk < kc ? M : 0);   // tokens of this chunk
        if constexpr (READY) {        // 16 bytes per token, the tokens of a (chunk, g, q) side by side
            o = __builtin_amdgcn_readfirstlane((uint32_t)chunk * (uint32_t)M * (kTileCols * 2));
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    xr[t][g] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, t * kTokenBlock + j < left ? (uint32_t)(q * M + t * kTokenBlock + j) * 16 : kOob,
                                                                     left ? o + (uint32_t)(4 * g * M) * 16 : 0u, 0);
            return;
        }
        asm volatile("" : "+s"(o));   // one addition per pair instead of 8 TB addresses kept in registers
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int mm = 0; mm < PAIRS; ++mm) {
                const int base = t * kTokenBlock + 2 * mm;
                const uint32_t v = left > base + 1 ? x_lane : left > base ? x_last : kOob;
                xr[t][mm] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, v, left > base ? o : 0u, 0);
                o += 2 * row_bytes;
            }
    };
    float4v sa, sb;
    auto load_s = [&](int chunk) __attribute__((always_inline)) {
        if constexpr (READY) return;
        const bool cv = chunk < kc;
        const uint32_t k0 = (uint32_t)chunk * kTileCols + 8 * kg;
        sa = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_s, cv ? k0 * 4 : kOob, 0, 0));
        sb = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_s, cv ? k0 * 4 + 16 : kOob, 0, 0));
    };
    load_s(wave);
    load_x(wave);     // the longest dependency chain: ahead of the packed words
    asm volatile("" ::: "memory");
    const LayerPart l = part_of(batch, pi, head_word, blockIdx.x, t0, t1, t2, t3, t4, t5, t6);
    const int ta = l.ta, tb_end = l.tb, N = l.nt * kTileRows;
    asm volatile("" : "+s"(pi) : : "memory");   // what is needed last is asked for last
    uint16_t *const y = batch.p[pi].y;
    const float act_scale = batch.p[pi].act_scale, out_scale = act_scale != 0.0f ? act_scale : 1.0f;
    const __amdgpu_buffer_rsrc_t rs_packed = make_rsrc(l.packed, (uint32_t)l.nt * (uint32_t)kc * TBYTES);
    // byte-split tables: behind the bucket multipliers (2 and 3 bits), the whole table (4 bits)
    const __amdgpu_buffer_rsrc_t rs_tb = make_rsrc(reinterpret_cast<const uint8_t *>(l.lut) + (BITS == 4 ? 0 : (size_t)N * NC * 4),
                                                   (uint32_t)N * row_table_bytes<BITS>());
    // packed words of the R row tiles from v0 (tiles past v1 and chunks past the layer's read zeros, no traffic)
    auto load_tile = [&](PackedTile<BITS> &p, int tile, int v1, int chunk) __attribute__((always_inline)) {
        const bool v = tile < v1 && chunk < kc;
        // the (tile, chunk) part of the address is wave-uniform and travels as the scalar offset
        const uint32_t o = v ? ((uint32_t)tile * (uint32_t)kc + (uint32_t)chunk) * TBYTES : 0u;
        p.lo = __builtin_amdgcn_raw_buffer_load_b128(rs_packed, v ? 16 * lane : kOob, o, kStreamPolicy);
        if (BITS == 3) p.hi = __builtin_amdgcn_raw_buffer_load_b64(rs_packed, v ? 8 * lane : kOob, o + 1024, kStreamPolicy);
        if (BITS == 4) p.hi4 = __builtin_amdgcn_raw_buffer_load_b128(rs_packed, v ? 16 * lane : kOob, o + 1024, kStreamPolicy);
    };

    uint4v B[TB][8];       // B operands of the current chunk: lane (q, token j) holds columns 64 q + 8 g .. of its token
    auto stage_x = [&]() __attribute__((always_inline)) {
        if constexpr (READY) {
#pragma unroll
            for (int t = 0; t < TB; ++t)
#pragma unroll
                for (int g = 0; g < 8; ++g) B[t][g] = xr[t][g];
            return;
        }
        const bool quantised = act_scale != 0.0f;   // wave-uniform
        float rs[8];                                // 1 / s, or the refined reciprocal of the quantiser's divisor
        auto step_of = [&](int e) { return e < 4 ? sa[e] : sb[e - 4]; };
#pragma unroll
        for (int e = 0; e < 8; ++e) rs[e] = quantised ? make_divisor(step_of(e), act_scale).y : __builtin_amdgcn_rcpf(step_of(e));
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            // operand slot order 0,4,1,5,2,6,3,7 (the dequantiser pairs weight v with weight 4 + v); rows past the last
            // token keep what the stage held: their columns of the product are never stored
#pragma unroll
            for (int mm = 0; mm < PAIRS; ++mm) {
                if (t * kTokenBlock + 2 * mm >= M) break;      // uniform
                const uint4v v = xr[t][mm];   // register i: columns 2i, 2i+1; result register i: columns i, 4+i
                uint4v o;
                if (!quantised) {
                    o[0] = smooth_pair<0, 0>(v[0], rs[0], v[2], rs[4]);
                    o[1] = smooth_pair<1, 1>(v[0], rs[1], v[2], rs[5]);
                    o[2] = smooth_pair<0, 0>(v[1], rs[2], v[3], rs[6]);
                    o[3] = smooth_pair<1, 1>(v[1], rs[3], v[3], rs[7]);
                } else {
                    half8 c;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const Divisor dv{-(step_of(e) * act_scale), rs[e]};
                        c[e < 4 ? 2 * e : 2 * (e - 4) + 1] = (e & 1) ? quantise_half<1>(v[e >> 1], dv) : quantise_half<0>(v[e >> 1], dv);
                    }
                    o = as_uint4(c);
                }
                *reinterpret_cast<uint4v *>(&stage[(2 * mm + th) * kStageStride + 8 * kg]) = o;
            }
            // written by this wave only: LDS operations of a wave stay in order
#pragma unroll
            for (int g = 0; g < 8; ++g)
                B[t][g] = *reinterpret_cast<const uint4v *>(&stage[j * kStageStride + 64 * q + 8 * g]);
        }
    };

    float4v acc[SETS][R][TB];
    typedef typename TablesOf<BITS>::type Tables;
    Tables tab[TABLES ? 2 : R];         // TABLES: of this tile and the next
    PackedTile<BITS> P[RING];
    // a row's table, 16 bytes (8 with 2 bits) at a time: piece i of it
    auto table_piece = [&](bool valid, uint32_t row, int i) __attribute__((always_inline)) {
        const uint32_t at = valid ? row * row_table_bytes<BITS>() + 16 * i : kOob;
        if constexpr (BITS == 2) {
            const uint2v t = __builtin_amdgcn_raw_buffer_load_b64(rs_tb, at, 0, 0);
            return uint4v{t[0], t[1], 0u, 0u};
        } else return __builtin_amdgcn_raw_buffer_load_b128(rs_tb, at, 0, 0);
    };
    auto make_tables = [](uint4v t, uint4v u) __attribute__((always_inline)) {
        if constexpr (BITS == 2) return RowTables{{t[0], 0u}, {t[1], 0u}};
        else if constexpr (BITS == 3) return RowTables{{t[0], t[1]}, {t[2], t[3]}};
        else return RowTables4{{t[0], t[1], t[2], t[3]}, {u[0], u[1], u[2], u[3]}};
    };
    uint8_t *const row_tables = smem + WAVES * kWaveBytes;
    auto table_of = [&](int r) __attribute__((always_inline)) {        // tile r of the pass, from LDS
        const uint8_t *at = row_tables + (r * kTileRows + j) * row_table_bytes<BITS>();
        if constexpr (BITS == 2) {
            const uint2v t = *reinterpret_cast<const uint2v *>(at);
            return make_tables(uint4v{t[0], t[1], 0u, 0u}, uint4v{});
        } else if constexpr (BITS == 3) return make_tables(*reinterpret_cast<const uint4v *>(at), uint4v{});
        else return make_tables(*reinterpret_cast<const uint4v *>(at), *reinterpret_cast<const uint4v *>(at + 16));
    };
    auto tile_product = [&](const PackedTile<BITS> &p, const typename TablesOf<BITS>::type &t, float4v (&a)[TB]) __attribute__((always_inline)) {
        uint4v op0, op1;
        auto multiply = [&](int d) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                a[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(op0), as_half8(B[b][2 * d]), a[b], 0, 0, 0);
                a[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_half8(op1), as_half8(B[b][2 * d + 1]), a[b], 0, 0, 0);
            }
        };
        if constexpr (BITS == 4) {
#pragma unroll
            for (int d = 0; d < 4; ++d) { decode_word4(p.lo[d], p.hi4[d], t, op0, op1); multiply(d); }
        } else {
            HighBits hb{0u, 0u};
            if (BITS == 3) hb = regroup_high(p.hi);
            decode_word<BITS, 0>(p.lo[0], hb, t, op0, op1); multiply(0);
            decode_word<BITS, 1>(p.lo[1], hb, t, op0, op1); multiply(1);
            decode_word<BITS, 2>(p.lo[2], hb, t, op0, op1); multiply(2);
            decode_word<BITS, 3>(p.lo[3], hb, t, op0, op1); multiply(3);
        }
    };

    float *part = reinterpret_cast<float *>(smem + wave * kWaveBytes);    // [tile][block][partial_quad]
    auto put_tile = [&](int slot, int b, float4v v) __attribute__((always_inline)) {
        *reinterpret_cast<float4v *>(&part[(slot * TB + b) * 256 + partial_quad(slot, q, j)]) = v;   // lane (q, j): rows 4q..4q+3 of token j
    };
    // the partial tiles of row tiles [first, end), in LDS from every wave's piece on: sum over the waves in order, one rounding, store
    auto store_tiles = [&](int first, int end) __attribute__((always_inline)) {
        __syncthreads();
        const int quads = (end - first) * 4;                 // row quads of one token
        for (int e = threadIdx.x; e < quads * M; e += WAVES * 64) {
            const int m = e / quads, rest = e - m * quads, r = rest >> 2, rq = rest & 3;
            const float *src = reinterpret_cast<const float *>(smem) + (r * TB + (m >> 4)) * 256 + partial_quad(r, rq, m & 15);
            auto pair_sum = [&](int w) __attribute__((always_inline)) {
                float4v v = *reinterpret_cast<const float4v *>(src + w * (kWaveBytes / 4));
                if (SETS == 1) v += *reinterpret_cast<const float4v *>(src + (w + kBW) * (kWaveBytes / 4));
                return v;
            };
            float4v sum = pair_sum(0);
#pragma unroll
            for (int w = 1; w < kBW; ++w) sum += pair_sum(w);
            typedef _Float16 half4 __attribute__((ext_vector_type(4)));
            half4 o;
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = (_Float16)(sum[u] * out_scale);
            *reinterpret_cast<half4 *>(y + (size_t)m * N + (size_t)(first + r) * kTileRows + 4 * rq) = o;
        }
    };

    if constexpr (RESIDENT) {
        // No wave has more than one chunk: its B operands are made once and stay, R row tiles after R row tiles go past, the next
        // ones' words and tables under way.  Partial tiles wait in the wave's piece of LDS (its stage is used up) until it is full.
        constexpr int VISIT = kWaveBytes / 1024 / R * R;
        auto load_both = [&](int r, int tile) __attribute__((always_inline)) {
            load_tile(P[r], tile, tb_end, wave);
            const uint32_t row = (uint32_t)tile * kTileRows + j;
            const uint4v t = table_piece(tile < tb_end, row, 0);
            tab[r] = make_tables(t, BITS == 4 ? table_piece(tile < tb_end, row, 1) : uint4v{});
        };
#pragma unroll
        for (int r = 0; r < R; ++r) load_both(r, ta + r);
        stage_x();
        int v0 = ta, visit = ta;
        auto pass = [&](auto TAIL_) __attribute__((always_inline)) {
            float4v a[R][TB];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                a[r][0] = float4v{0.f, 0.f, 0.f, 0.f};
                if (wave < kc && v0 + r < tb_end) tile_product(P[r], tab[r], a[r]);      // uniform
                if constexpr (!decltype(TAIL_)::value) load_both(r, v0 + R + r);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) put_tile(v0 + r - visit, 0, a[r][0]);
            v0 += R;
        };
        while (v0 + R < tb_end) {
            pass(std::false_type{});
            if (v0 - visit == VISIT) {
                store_tiles(visit, v0);
                visit = v0;
                __syncthreads();
            }
        }
        pass(std::true_type{});
        store_tiles(visit, tb_end);
        return;
    }

    int pass_tiles = R;
    if (ring_of_words(R) && tb_end - ta > R) {   // passes of one length: a last pass of few tiles would have few loads under way
        const int passes = (tb_end - ta + R - 1) / R;
        pass_tiles = (tb_end - ta + passes - 1) / passes;
    }
    for (int v0 = ta; v0 < tb_end; v0 += pass_tiles) {
        const int v1 = min(tb_end, v0 + pass_tiles);
        uint4v row_t = {0u, 0u, 0u, 0u}, row_u = {0u, 0u, 0u, 0u};   // TABLES: of the pass's rows, one row per thread
        if constexpr (TABLES) {
            const bool valid = (int)threadIdx.x < (v1 - v0) * kTileRows;
            const uint32_t row = (uint32_t)v0 * kTileRows + threadIdx.x;
            row_t = table_piece(valid, row, 0);
            if (BITS == 4) row_u = table_piece(valid, row, 1);
        }
#pragma unroll
        for (int r = 0; r < RING; ++r) load_tile(P[r], v0 + r, v1, wave);
        if constexpr (!TABLES) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint32_t row = (uint32_t)(v0 + r) * kTileRows + j;
                const uint4v t = table_piece(v0 + r < v1, row, 0);
                tab[r] = make_tables(t, BITS == 4 ? table_piece(v0 + r < v1, row, 1) : uint4v{});
            }
        } else {
            if (threadIdx.x < R * kTileRows) {
                uint8_t *to = row_tables + threadIdx.x * row_table_bytes<BITS>();
                if constexpr (BITS == 2) *reinterpret_cast<uint2v *>(to) = uint2v{row_t[0], row_t[1]};
                else *reinterpret_cast<uint4v *>(to) = row_t;
                if constexpr (BITS == 4) *reinterpret_cast<uint4v *>(to + 16) = row_u;
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int i = 0; i < SETS; ++i) acc[i][r][b] = float4v{0.f, 0.f, 0.f, 0.f};

        // One chunk of the pass's row tiles.  The loads of the wave's next chunk are issued whatever is valid (one that may or may not have
        // been issued makes the compiler wait for every load under way), but not behind the last chunk (TAIL): out of range they would
        // still take the time of their addresses.
        auto chunk_products = [&](auto TAIL_, float4v (&a)[R][TB], int chunk) __attribute__((always_inline)) {
            constexpr bool TAIL = decltype(TAIL_)::value;
            if constexpr (TABLES) tab[0] = table_of(0);
            stage_x();
            if constexpr (TB == 1 && !TAIL) { load_s(chunk + WAVES); load_x(chunk + WAVES); }   // room for the next chunk's activations while this one multiplies
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (STRAIGHT) {
                    if (r == 0 || v0 + r < v1) tile_product(P[r], tab[r], a[r]);     // uniform
                    if constexpr (!TAIL) load_tile(P[r], v0 + r, v1, chunk + WAVES);
                } else {
                    if (r > 0 && v0 + r >= v1) break;           // uniform
                    if constexpr (RING == R && !TABLES) {
                        tile_product(P[r], tab[r], a[r]);
                        load_tile(P[r], v0 + r, v1, chunk + WAVES);
                        continue;
                    }
                    if (TABLES && r + 1 < R) tab[(r + 1) & 1] = table_of(r + 1);
                    tile_product(P[r % RING], tab[TABLES ? r & 1 : r], a[r]);
                    // the slot's next tile: of this chunk, or the one it starts the next chunk with
                    const bool same = r + RING < R && v0 + r + RING < v1;
                    load_tile(P[r % RING], v0 + (same ? r + RING : r % RING), v1, same ? chunk : chunk + WAVES);
                }
            }
            if constexpr (TB > 1 && !TAIL) { load_s(chunk + WAVES); load_x(chunk + WAVES); }    // into the registers the B operands leave
        };
        if constexpr (!STRAIGHT) {
            for (int c = wave; c < kc; c += 2 * WAVES) {
                chunk_products(std::false_type{}, acc[0], c);
                if (c + WAVES >= kc) break;
                chunk_products(std::false_type{}, acc[SETS - 1], c + WAVES);
            }
        } else if constexpr (SETS == 1) {
            int c = wave;
#pragma unroll 1
            for (; c + WAVES < kc; c += WAVES) chunk_products(std::false_type{}, acc[0], c);
            if (c < kc) chunk_products(std::true_type{}, acc[0], c);
        } else {
            int c = wave;
#pragma unroll 1
            for (; c + WAVES < kc; c += 2 * WAVES) {
                chunk_products(std::false_type{}, acc[0], c);
                if (c + 2 * WAVES >= kc) { chunk_products(std::true_type{}, acc[SETS - 1], c + WAVES); c = kc; break; }
                chunk_products(std::false_type{}, acc[SETS - 1], c + WAVES);
            }
            if (c < kc) chunk_products(std::true_type{}, acc[0], c);
        }

        // ---- partial tiles to LDS, one barrier, sum over the waves in order, one rounding, store
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int b = 0; b < TB; ++b) put_tile(r, b, SETS == 2 ? acc[0][r][b] + acc[SETS - 1][r][b] : acc[0][r][b]);
        store_tiles(v0, v1);
        if (WAVES > kBW) break;             // (one pass: the host gives these variants no more row tiles than they hold)
        if (v1 < tb_end) {
            load_s(wave);
            load_x(wave);
            __syncthreads();                // the next tiles' stages overwrite the partial tiles
        }
    }
}

}  // namespace lcd
