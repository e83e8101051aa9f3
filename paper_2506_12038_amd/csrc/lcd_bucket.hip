// Single-token decode path of the smoothed table-lookup product, gfx950: the bucket kernel (with 2-bit indices also two
// tokens, and up to four on INT8 activation codes).
//
// The lookup + accumulation of paper Sec. 4.2 is done by the sparse matrix core:
// v_smfmac_f32_16x16x64_f16 multiplies, for each of 16 rows, 32 values of its A operand with rows of a dense
// B operand *selected by 2-bit indices held in a register*.  Feeding
//     A     = the smoothed activations xs[k]          (the same for all 16 output rows),
//     index = the packed 2-bit weight indices, as stored in memory (no decode instruction),
//     B     = a constant 0/1 matrix that routes "index == c" to accumulator column c,
// makes accumulator column c of row n the centroid bucket sum  S[n][c] = sum_{k: idx[n][k]==c} xs[k];
// the output is y[n] = sum_c C[n][c] * S[n][c], four multiplies per row at the very end.
// For 3-bit indices the third bit h flips the sign of the activation in a second pass that
// lands in columns 4..7:  C[n][4h+l] = P[n][l] + (1-2h) Q[n][l]  gives
//     y[n] = sum_l P[n][l] * (sum_{k: l_k==l} xs[k]) + Q[n][l] * (sum_{k: l_k==l} (-1)^{h_k} xs[k]).
// The sign flips cost one xor-and (v_bitop3_b32) per pair of weights plus one 64-bit shift per
// two pairs.
// Two tokens at 2 bits take the sign-flipped pass's place with the second token's activations.
// With the INT8 activation codes of Sec. 4.1 at 2 bits, A holds the codes as int8 numbers and the
// instruction is v_smfmac_i32_16x16x128_i8 (64 values per row and instruction): one to four tokens.
//
// Work split: a workgroup owns a contiguous run of row tiles (16 rows) of ONE layer and takes them R at a time; its waves (16, or 8)
// split K, wave w takes the 256-column chunks w, w + W, ...  A step is one chunk of R row tiles: the wave smooths the chunk's
// activations (4 columns per lane), hands them to the 16 lanes of a row with DPP broadcasts -- no LDS, no other wave to wait for -- and
// keeps them while the R tiles' packed words go through the matrix core.  The bucket sums stay in accumulators over all of the wave's
// chunks and go to LDS once per tile; behind one barrier the waves' sums are added in their order, multiplied, added over the buckets,
// rounded once and stored.  The order of the additions of one output depends on K alone.
//
// What bounds it: with few row tiles per workgroup the latencies in front (us from a launch's first wave, 4096 x 4096, 2 bits: waves start
// until 0.6, first words in use 0.5..1.6, barrier 1.8, end 2.2; 1.1 more between two launches of a graph); then, at 2 bits, HBM (5.9 TB/s
// over 3584 row tiles of K = 8192), at 3 bits the vector and matrix pipes, which sparse instructions hardly let work side by side: 48
// sign flips (192 cycles) and 16 sparse instructions (256) per tile and chunk.
// The kernel before it kept two chunks' operands per wave and walked all row tiles of a K segment before the next segment (a
// switch cost 1 us: activations fanned out through LDS), with a multiply and reduce per tile and segment.  7B block (q, k, v | o | gate, up |
// down), 3 bits, one token: 8.7, 5.3, 11.1, 9.9 -> 7.0, 4.2, 9.6, 6.6 us a launch in a graph; 70B MLP, 2 bits: gate, up 21.4 -> 21, down 17.2 ->
// 12.6; 7B block, 2 bits, four tokens of INT8 codes 7.3, 5.3, 9.2, 10.2 -> 6.6, 5.0, 8.3, 9.0; seven 7B layers in one launch, 3 bits 21.1 -> 19.4.
// Loads further ahead than the next step (5.5 instead of 3.9 us on 4096 x 4096, 3 bits: the addresses of loads that are out of range
// take their time too) and 8 waves for one token of fp16 activations (down, 3 bits 6.6 -> 7.6) were slower.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "lcd_decode.h"
#include "lcd_share.h"

namespace lcd {

// lane LANE of every row of 16 lanes to all lanes of that row
template <int LANE>
__device__ __forceinline__ uint32_t row_broadcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + LANE, 0xF, 0xF, true);
}

template <int BITS, int MT> constexpr int bucket_columns() { return (BITS == 2 ? 4 : 8) * MT; }
template <int R> constexpr int visit_tiles() { return 16 / R * R; }   // row tiles whose bucket sums fit LDS together
template <int BITS, int MT, int R, int W> constexpr size_t bucket_lds_bytes() { return (size_t)W * visit_tiles<R>() * bucket_columns<BITS, MT>() * 64; }

template <int BITS>
struct BucketWords {
    uint4v lo;   // the lane's 64 two-bit fields of a (tile, chunk)
    uint2v hi;   // 3 bits: its 64 third bits
};

// The most columns whose bucket sums are one run of additions: each may lose 2^-24 of the sum, and a wave of 16 makes 2^12 of them here.  (The int32 sums
// of a wave's codes hold 2^24 columns.)  Wider layers take the kernels that end a wave's run (WIDE) every kRunCols / W columns and add its
// sums to a total; layers up to kRunCols get the same bits from both.
constexpr int kRunCols = 1 << 21;

// R: row tiles of a pass, W: waves.  MT: token slots, NTOK: tokens the launch has (MT = 4 token slots also serve three tokens, which then leave the fourth pass out).
template <int BITS, int MT, bool I8, int NTOK, int R, int W, bool WIDE, class BATCH>
__global__ void __launch_bounds__(W * 64, 1) gemv_bucket_kernel(
    const uint32_t t0, const uint32_t t1, const uint32_t t2, const uint32_t t3, const uint32_t t4, const uint32_t t5, const uint32_t t6,
    const uint32_t t7, const uint16_t *head_x, const float *head_s, const uint32_t head_word, const BATCH batch)
{
    static_assert(MT == 1 || (MT == 2 && BITS == 2) || (MT == 4 && BITS == 2 && I8), "two tokens: 2-bit indices only; four: int8 operands only");
    typedef int int4v __attribute__((ext_vector_type(4)));
    typedef int int8v __attribute__((ext_vector_type(8)));
    constexpr bool kHalfOps = !I8 || BITS == 3;  // fp16 operands kept (3 bits with int8 codes: for the sign-flipped pass)
    constexpr int NA = kHalfOps ? 8 : 1;         // fp16 operands (4 registers) per chunk and token
    constexpr int NQ = I8 ? 4 : 1;               // int8 operands (4 registers) per chunk and token
    constexpr int NB = BITS == 2 ? 4 : 8;        // buckets per row
    constexpr int NC = bucket_columns<BITS, MT>();
    constexpr uint32_t TB = BITS == 2 ? 1024 : 1536;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];   // bucket sums [wave][tile][row quad 4][column NC][row 4]
    float *const sums = reinterpret_cast<float *>(smem);
    constexpr int kTileFloats = 16 * NC, kVisit = visit_tiles<R>(), kWaveFloats = kVisit * kTileFloats;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keeps addresses scalar
    const int q = lane >> 4, j = lane & 15;

    constexpr bool SINGLE = std::is_same<BATCH, SingleBatch>::value;
    const uint32_t word = SINGLE ? head_word | kHeadSingle | kHeadShared : head_word;
    int pi = SINGLE || (word & kHeadSingle) ? 0 : layer_of_workgroup(blockIdx.x, t0, t1, t2, t3, t4, t5, t6, t7);
    const uint16_t *x = head_x;
    const float *s = head_s;
    int kc;
    input_of(batch, pi, word, x, s, kc);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(x, (uint32_t)NTOK * (uint32_t)kc * kTileCols * 2);
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(s, (uint32_t)kc * kTileCols * 4);

    // Loads of a step: one chunk of up to R row tiles.  Activations: lane l takes columns [4 l, 4 l + 4) of the chunk.
    struct StepRegs {
        uint2v x[NTOK];
        float4v s;
        BucketWords<BITS> w[R];
    };
    StepRegs st;
    auto load_x = [&](int chunk, bool valid) {
        const uint32_t c = valid ? (uint32_t)chunk : 0u;
#pragma unroll
        for (int t = 0; t < NTOK; ++t)   // token t's row of x starts K fp16 numbers after token t - 1's
            st.x[t] = __builtin_amdgcn_raw_buffer_load_b64(rs_x, valid ? 8 * lane : kOob, (c + (uint32_t)t * (uint32_t)kc) * (kTileCols * 2), 0);
        st.s = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_s, valid ? 16 * lane : kOob, c * (kTileCols * 4), 0));
    };
    load_x(wave, wave < kc);
    asm volatile("" ::: "memory");   // these loads first: they start the longest dependency chain
    const LayerPart part_l = part_of(batch, pi, word, blockIdx.x, t0, t1, t2, t3, t4, t5, t6);
    const int nt = part_l.nt, ta = part_l.ta, tb = part_l.tb;
    const __amdgpu_buffer_rsrc_t rs_packed = make_rsrc(part_l.packed, (uint32_t)nt * (uint32_t)kc * TB);
    const __amdgpu_buffer_rsrc_t rs_lut = make_rsrc(part_l.lut, (uint32_t)nt * 16 * NB * 4);

    // the (tile, chunk) part of the address is wave-uniform and travels as the scalar offset; only the lane's part is
    // range-checked, so an invalid load swaps it for an offset that is out of range: zeros, no traffic
    auto load_words = [&](BucketWords<BITS> &p, int tile, int chunk, bool valid) {
        const uint32_t o = valid ? ((uint32_t)tile * (uint32_t)kc + (uint32_t)chunk) * TB : 0u;
        p.lo = __builtin_amdgcn_raw_buffer_load_b128(rs_packed, valid ? 16 * lane : kOob, o, kStreamPolicy);
        if (BITS == 3) p.hi = __builtin_amdgcn_raw_buffer_load_b64(rs_packed, valid ? 8 * lane : kOob, o + 1024, kStreamPolicy);
    };

    if (ta >= tb) return;            // (the host never launches such a workgroup)
    // the step whose loads are issued next: the wave's chunks of R row tiles one after the other, then the next R (a step past
    // the last one, and every step of a wave without chunks, loads nothing)
    int pf_tile = ta, pf_chunk = wave;
    auto load_step_words = [&](int r) { load_words(st.w[r], pf_tile + r, pf_chunk, pf_chunk < kc && pf_tile + r < tb); };
    auto advance = [&]() {
        pf_chunk += W;
        if (pf_chunk >= kc) { pf_chunk = wave; pf_tile += R; }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) load_step_words(r);
    advance();

    // per-bucket multipliers of the first visit: thread e holds those of item e (row quad and bucket) of it
    auto load_multipliers = [&](int first_tile, int items, int e) {
        const int i = e / NC, b = e % NB;
        return __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_lut, e < items ? (uint32_t)((first_tile * 4 + i) * NB + b) * 16 : kOob, 0, 0));
    };

    uint4v A[MT][NA];    // the chunk's smoothed activations, the same in the 16 lanes of a row
    uint4v Aq[MT][NQ];   // I8: the codes as int8 numbers
    half16 B1, B2;       // constant routing matrices: index c -> column c, column 4 + c
    int8v Bq[MT];        // I8: the same as int8 numbers; token t's sums go to columns 4t .. 4t+3
#pragma unroll
    for (int b = 0; b < 16; ++b) {
        B1[b] = ((b & 3) == j) ? (_Float16)1.0f : (_Float16)0.0f;
        B2[b] = ((b & 3) + 4 == j) ? (_Float16)1.0f : (_Float16)0.0f;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int b = 0; b < 8; ++b) Bq[t][b] = (j >> 2) == t ? 1 << (8 * (j & 3)) : 0;   // byte (b & 3) == j - 4t

    const float act_scale = I8 ? batch.p[pi].act_scale : 0.0f;
    auto make_operands = [&]() __attribute__((always_inline)) {
        if constexpr (I8) {
            Divisor dv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) dv[e] = make_divisor(st.s[e], act_scale);
#pragma unroll
            for (int t = 0; t < NTOK; ++t) {
                uint32_t halves[2];
                const uint32_t codes = quantise_four<kHalfOps>(st.x[t], dv, halves);
                unrolled<16>([&](auto r) __attribute__((always_inline)) {
                    constexpr int i = decltype(r)::value;
                    Aq[t][i / 4][i % 4] = row_broadcast<i>(codes);
                });
                if constexpr (kHalfOps) unrolled<32>([&](auto r) __attribute__((always_inline)) {
                    constexpr int i = decltype(r)::value;
                    A[t][i / 4][i % 4] = row_broadcast<i / 2>(halves[i % 2]);
                });
            }
        } else {
            float r[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = __builtin_amdgcn_rcpf(st.s[e]);
#pragma unroll
            for (int t = 0; t < NTOK; ++t) {
                const uint32_t halves[2] = {smooth_pair<0, 1>(st.x[t][0], r[0], st.x[t][0], r[1]), smooth_pair<0, 1>(st.x[t][1], r[2], st.x[t][1], r[3])};
                unrolled<32>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    A[t][i / 4][i % 4] = row_broadcast<i / 2>(halves[i % 2]);
                });
            }
        }
    };

    struct Sums { float4v f; int4v i; };   // fp16 operands: f; int8 operands: i; 3 bits with int8 codes: both
    auto tile_sums = [&](const BucketWords<BITS> &p, Sums &a) __attribute__((always_inline)) {
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const int idxreg = (int)p.lo[d];
            if constexpr (I8) {
#pragma unroll
                for (int t = 0; t < NTOK; ++t)
                    a.i = __builtin_amdgcn_smfmac_i32_16x16x128_i8(__builtin_bit_cast(int4v, Aq[t][d]), Bq[t], a.i, idxreg, 0, 0);
            }
            // half a = 0 of a word uses index bits [15:0], a = 1 bits [31:16]
            if constexpr (!I8) {
                a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(A[0][2 * d]), B1, a.f, idxreg, 0, 0);
                a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(A[0][2 * d + 1]), B1, a.f, idxreg, 0, 1);
                if constexpr (MT == 2) {
                    a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(A[1][2 * d]), B2, a.f, idxreg, 0, 0);
                    a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(A[1][2 * d + 1]), B2, a.f, idxreg, 0, 1);
                }
            }
            if constexpr (BITS == 3) {
                // sign-flipped operands: pair v of half a has its two third bits 16 apart in word a
                // of p.hi; one 64-bit shift moves them to bits 15 / 31 of both words, one
                // xor-and per word applies them
                const unsigned long long h64 = ((unsigned long long)p.hi[1] << 32) | p.hi[0];
                uint4v f0, f1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int sh = 15 - (8 * (v >> 1) + 2 * d + (v & 1));
                    unsigned long long t = h64;   // one full-rate v_lshlrev_b64 (the compiler would split it in two)
                    if (sh) asm("v_lshlrev_b64 %0, %1, %2" : "=v"(t) : "n"(sh), "v"(h64));
                    f0[v] = xor_and(A[0][2 * d][v], (uint32_t)t, 0x80008000u);
                    f1[v] = xor_and(A[0][2 * d + 1][v], (uint32_t)(t >> 32), 0x80008000u);
                }
                a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(f0), B2, a.f, idxreg, 0, 0);
                a.f = __builtin_amdgcn_smfmac_f32_16x16x64_f16(as_half8(f1), B2, a.f, idxreg, 0, 1);
            }
        }
    };

    const float4v cf_first = load_multipliers(ta, min(tb - ta, kVisit) * 4 * NC, threadIdx.x);
    Sums acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = Sums{{0.f, 0.f, 0.f, 0.f}, {0, 0, 0, 0}};
    auto value_of = [&](const Sums &a) __attribute__((always_inline)) {
        float4v v;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if constexpr (!I8) v[u] = a.f[u];
            else if constexpr (BITS == 2) v[u] = (float)a.i[u];   // (integers: exact up to 2^24)
            else v[u] = (float)a.i[u] + a.f[u];                   // columns 0..3 and 4..7: the other one is zero
        }
        return v;
    };
    float4v total[WIDE ? R : 1];
    int run = 0;                     // WIDE: chunks of the present run
#pragma unroll
    for (int r = 0; r < (WIDE ? R : 1); ++r) total[r] = float4v{0.f, 0.f, 0.f, 0.f};
    asm volatile("" : "+s"(pi) : : "memory");   // what is needed last is asked for last
    uint16_t *const y = batch.p[pi].y;
    const float out_scale = I8 ? act_scale : 1.0f;

    // The waves' bucket sums of row tiles [first, end) in a fixed order, multiplied, added over the buckets, rounded once, stored.
    // AHEAD: sums of a thread read together.
    auto store_visit = [&](auto AHEAD_, int first, int end) __attribute__((always_inline)) {
#pragma clang fp contract(off)
        constexpr int AHEAD = decltype(AHEAD_)::value;
        __syncthreads();
        const int items = (end - first) * 4 * NC;
        for (int e = threadIdx.x; e < items; e += W * 64) {
            const float4v cf = first == ta && e < W * 64 ? cf_first : load_multipliers(first, items, e);
            float4v sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < W; w += AHEAD) {
                float4v v[AHEAD];
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) v[i] = *reinterpret_cast<const float4v *>(&sums[(w + i) * kWaveFloats + e * 4]);
#pragma unroll
                for (int i = 0; i < AHEAD; ++i) sum += v[i];
                if (AHEAD < W) __builtin_amdgcn_sched_barrier(0);
            }
            typedef _Float16 half4 __attribute__((ext_vector_type(4)));
            half4 o;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float v = sum[u] * cf[u];
                v += dpp_f32<kDppQuadXor1>(v);
                v += dpp_f32<kDppQuadXor2>(v);
                if (NB == 8) v += dpp_f32<kDppRowHalfMirror>(v);
                o[u] = (_Float16)(v * out_scale);
            }
            if (e % NB == 0 && e % NC / NB < NTOK)
                *reinterpret_cast<half4 *>(&y[(size_t)(e % NC / NB) * nt * kTileRows + (size_t)first * kTileRows + (size_t)(e / NC) * 4]) = o;
        }
    };

    // One step.  It issues the loads of the next one into the registers it has used, all of
    // them whatever is valid: a load that may or may not have been issued makes the compiler wait for every one under way.
    // TAIL: there is no such step (loads out of range would still take the time of their addresses).
    int v0 = ta, visit = ta, c = wave;
    bool fresh = true;
    auto step = [&](auto TAIL_) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(TAIL_)::value;
        const int n = wave < kc ? min(R, tb - v0) : 0;
        if (fresh) make_operands();          // a wave's only chunk stays in registers
        fresh = kc > W;
        if constexpr (!TAIL) load_x(pf_chunk, fresh && pf_chunk < kc && pf_tile < tb);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r < n) tile_sums(st.w[r], acc[r]);
            if constexpr (!TAIL) load_step_words(r);
        }
        if constexpr (!TAIL) advance();
        c += W;
        if constexpr (WIDE) {
            if (c >= kc || ++run == kRunCols / kTileCols / W) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    total[r] += value_of(acc[r]);
                    acc[r] = Sums{{0.f, 0.f, 0.f, 0.f}, {0, 0, 0, 0}};
                }
                run = 0;
            }
        }
        if (c < kc) return;
        c = wave;
        // ---- all of K: the bucket sums to LDS
        if (j < NC) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                *reinterpret_cast<float4v *>(&sums[wave * kWaveFloats + (v0 + r - visit) * kTileFloats + (q * NC + j) * 4]) = WIDE ? total[WIDE ? r : 0] : value_of(acc[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (WIDE) total[r] = float4v{0.f, 0.f, 0.f, 0.f};
            else acc[r] = Sums{{0.f, 0.f, 0.f, 0.f}, {0, 0, 0, 0}};
        }
        v0 += R;
        if (v0 >= tb || v0 - visit < kVisit) return;
        store_visit(std::integral_constant<int, 2>{}, visit, v0);
        visit = v0;
        __syncthreads();             // the next visit's sums take the same places
    };
    int left = (tb - ta + R - 1) / R * (wave < kc ? (kc - wave + W - 1) / W : 1);   // steps of this wave
    for (; left > 1; --left) step(std::false_type{});
    step(std::true_type{});
    store_visit(std::integral_constant<int, W>{}, visit, tb);   // (nothing else lives here: registers for all reads at once)
}

template <int BITS, int MT, bool I8, int NTOK, int R, bool WIDE = false>
static BucketVariant variant_of(int id)
{
    constexpr int W = bucket_waves(MT, I8);
    const void *fn = (const void *)gemv_bucket_kernel<BITS, MT, I8, NTOK, R, W, WIDE, BucketBatch>;
    const void *single = fn;         // (the group's kernel takes one layer too)
    if constexpr (!WIDE) single = (const void *)gemv_bucket_kernel<BITS, MT, I8, NTOK, R, W, WIDE, SingleBatch>;
    return BucketVariant{fn, single, R, W, bucket_lds_bytes<BITS, MT, R, W>(), id};
}

template <int BITS, int MT, bool I8, int NTOK>
static BucketVariant pick(int pass, int tiles, int kc, int id)
{
    // (packed rows of kRunCols columns leave room for 512 row tiles: two for a workgroup)
    if (kc > kRunCols / kTileCols) return tiles == 1 ? variant_of<BITS, MT, I8, NTOK, 1, true>(9 * id + 7) : variant_of<BITS, MT, I8, NTOK, 2, true>(9 * id + 8);
    constexpr int lengths = bucket_rule(BITS, NTOK, I8).lengths;
    id = 9 * id + pass;
    if constexpr (lengths > 5) {
        if (pass == 5) return variant_of<BITS, MT, I8, NTOK, kBucketPass[5]>(id);
        if (pass == 6) return variant_of<BITS, MT, I8, NTOK, kBucketPass[6]>(id);
    }
    if constexpr (lengths > 3) {
        if (pass == 3) return variant_of<BITS, MT, I8, NTOK, kBucketPass[3]>(id);
        if (pass == 4) return variant_of<BITS, MT, I8, NTOK, kBucketPass[4]>(id);
    }
    if (pass == 0) return variant_of<BITS, MT, I8, NTOK, kBucketPass[0]>(id);
    return pass == 1 ? variant_of<BITS, MT, I8, NTOK, kBucketPass[1]>(id) : variant_of<BITS, MT, I8, NTOK, kBucketPass[2]>(id);
}

BucketVariant bucket_variant(int bits, int tokens, bool int8_codes, int pass, int tiles, int kc)
{
    if (bits == 3) return int8_codes ? pick<3, 1, true, 1>(pass, tiles, kc, 0) : pick<3, 1, false, 1>(pass, tiles, kc, 1);
    if (!int8_codes) return tokens == 1 ? pick<2, 1, false, 1>(pass, tiles, kc, 2) : pick<2, 2, false, 2>(pass, tiles, kc, 3);
    if (tokens <= 2) return tokens == 1 ? pick<2, 1, true, 1>(pass, tiles, kc, 4) : pick<2, 2, true, 2>(pass, tiles, kc, 5);
    return tokens == 3 ? pick<2, 4, true, 3>(pass, tiles, kc, 6) : pick<2, 4, true, 4>(pass, tiles, kc, 7);
}

}  // namespace lcd
