// Decode path (M <= 16) of the smoothed table-lookup product, gfx950: the launcher of the decode kernels (lcd_bucket.hip,
// lcd_tokens.hip) and the transformation of the activations ahead of the tokens kernel.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <mutex>
#include <climits>
#include "lcd_decode.h"
#include "lcd_launch.h"
#include "lcd_share.h"

namespace lcd {

// ---- activation transformation ahead of the tokens kernel (Sec. 4.1) -----------------------------
// On the tokens kernel's route (2..16 tokens, and 4 bits) every workgroup of a layer stages the whole activation matrix, so whatever is
// done to an activation is repeated by each of them.  This small kernel does it once per layer
// and leaves the result in the workspace, as fp16 numbers in the order of the matrix operands ([chunk][step 8][quarter 4]
// [token][8 columns, slots 0,4,1,5,2,6,3,7], so that the tokens kernel loads its B operands as they are: no smoothing, no
// turn through LDS): the INT8 codes of Eq. 10 or the smoothed activations x/s, where the saving exceeds the extra launch.
// One thread takes 8 columns of one token, or of four that share the divisor-only part of the division.
struct TransformItem {
    const uint16_t *x;
    const float *s;
    uint16_t *codes;
    int K;
    float s_q;
};
struct TransformBatch {
    TransformItem p[kMaxGroup];
};
constexpr int kQuantThreads = 64;
// Four tokens per thread only where one per thread is more than two waves per compute unit (kQuantWaves): the launch is a chain of
// latencies, which one token makes shorter.  A product of 8192 rows, 3 bits, behind it, four / one, us: 17 tokens, K = 2048 6.5 / 6.4 (INT8
// codes 6.7 / 6.3), 4096 8.8 / 8.5 (9.1 / 8.8), 11008 16.0 / 15.7 (16.3 / 15.8); 40 tokens, 4096 9.9 / 9.9 (10.4 / 9.9), 11008 20.0 / 20.4
// (20.4 / 20.4); 64 tokens, 4096 10.4 / 10.3 (10.9 / 10.3), 11008 24.7 / 25.2 (25.1 / 25.3); 80 tokens, 4096 12.3 / 12.6 (12.7 / 12.6).
constexpr int kQuantTokens = 4, kQuantWaves = 512;
constexpr long long kAheadCodes = 50000, kAheadSmoothed = 300000, kAheadTiles = 200000;   // activations per workgroup beyond which they are transformed ahead

template <int TOKENS>
__device__ __forceinline__ void transform_columns(const TransformItem &it, int M)
{
    const int k0 = ((int)blockIdx.x * kQuantThreads + (int)threadIdx.x) * 8;
    if (k0 >= it.K) return;   // K is a multiple of 256: a thread's 8 columns are all inside or all outside
    const float4v s0 = *reinterpret_cast<const float4v *>(it.s + k0), s1 = *reinterpret_cast<const float4v *>(it.s + k0 + 4);
    const bool quantised = it.s_q != 0.0f;   // uniform
    Divisor dv[8];
    float rs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        dv[e] = make_divisor(e < 4 ? s0[e] : s1[e - 4], quantised ? it.s_q : 1.0f);
        rs[e] = __builtin_amdgcn_rcpf(e < 4 ? s0[e] : s1[e - 4]);
    }
    // position of these 8 columns in operand order: chunk, then step g = (k % 64) / 8, then (k % 256) / 64
    const int group = (k0 / kTileCols) * 32 + ((k0 % 64) / 8) * 4 + (k0 % kTileCols) / 64;
    // blockIdx.z: a group of tokens (short dependent chains, all loads in flight together)
    const int m0 = (int)blockIdx.z * TOKENS;
    uint4v v[TOKENS];
#pragma unroll
    for (int i = 0; i < TOKENS; ++i)
        if (m0 + i < M) v[i] = *reinterpret_cast<const uint4v *>(it.x + (size_t)(m0 + i) * it.K + k0);
#pragma unroll
    for (int i = 0; i < TOKENS; ++i) {
        if (m0 + i < M) {
            // register i of the result: columns i, 4 + i
            uint4v o;
            if (quantised) {
                o[0] = quantise_pair<0, 0>(v[i][0], dv[0], v[i][2], dv[4]);
                o[1] = quantise_pair<1, 1>(v[i][0], dv[1], v[i][2], dv[5]);
                o[2] = quantise_pair<0, 0>(v[i][1], dv[2], v[i][3], dv[6]);
                o[3] = quantise_pair<1, 1>(v[i][1], dv[3], v[i][3], dv[7]);
            } else {                      // rounds as the fused path does
                o[0] = smooth_pair<0, 0>(v[i][0], rs[0], v[i][2], rs[4]);
                o[1] = smooth_pair<1, 1>(v[i][0], rs[1], v[i][2], rs[5]);
                o[2] = smooth_pair<0, 0>(v[i][1], rs[2], v[i][3], rs[6]);
                o[3] = smooth_pair<1, 1>(v[i][1], rs[3], v[i][3], rs[7]);
            }
            *reinterpret_cast<uint4v *>(it.codes + ((size_t)group * M + m0 + i) * 8) = o;
        }
    }
}

template <int TOKENS>
__global__ __launch_bounds__(kQuantThreads) void transform_kernel(const TransformBatch batch, int M) { transform_columns<TOKENS>(batch.p[blockIdx.y], M); }

// One input, the usual case: its arguments are in scalar registers when a wave starts, and the argument segment is 40 bytes
// (4096 x 4096, 3 bits: 20 tokens 9.0 -> 8.6 us, 48 tokens 10.5 -> 10.2).
template <int TOKENS>
__global__ __launch_bounds__(kQuantThreads) void transform_one_kernel(const uint16_t *x, const float *s, uint16_t *codes, int K, float s_q, int M)
{
    transform_columns<TOKENS>(TransformItem{x, s, codes, K, s_q}, M);
}

// Which kernel takes layers of a width.
// 4 bits: the register dequantiser serves one token too; 2 bits: the sparse-matrix-core kernel also takes
// two tokens (one sparse pass per token costs less than dequantising once)
// (with the INT8 codes of Sec. 4.1 as int8 operands the sparse-matrix-core kernel has room for four tokens)
// (dense: fp16 activations, because the routing matrix's zeros turn an infinite activation into a NaN of every bucket where
// the dequantised product gives the infinity that plain arithmetic gives; 3 bits, because the bucket kernel's multipliers are
// (C[j] +- C[4 + j]) / 2 in binary32, which loses the centroid next to a large entry that no index names)
static bool tokens_kernel_takes(int bits, int M, bool all_quantised, bool dense)
{
    const int sparse_tokens = bits != 2 ? 1 : all_quantised ? 4 : 2;   // most tokens the bucket kernel takes
    return bits == 4 || M > sparse_tokens || (dense && !(all_quantised && bits == 2));
}

// Several tokens: every workgroup transforms its layer's activations once per pass over its row tiles; ahead of the
// product they are transformed once, at the price of a launch (about 3 us in a graph).  The line lies where that much work is
// saved, counted in activations per workgroup (tokens x widest K x passes).  In the product / ahead, 2, 3, 4 bits, us a launch:
//   INT8 codes  4096 x 4096, 12 tokens (49 k) 6.5/6.7 6.8/7.0 7.4/7.5, 16 (66 k) 7.4/7.0 7.6/7.3 8.3/7.7; 4096 x 11008, 5 (55 k) 9.1/9.5 9.8/10.4 11.5/11.7,
//               8 (88 k) 10.2/9.5 10.8/10.5 12.4/11.9; 28672 x 8192, twice, 9 (74 k) 37.4/31.9 45.0/41.8 64.5/61.1
//   fp16        4096 x 13824, 16 (221 k) 12.2/12.6 13.5/14.3 15.9/15.9; 8192 x 28672, 8 (229 k) 22.1/22.0 28.2/26.1 36.4/34.0
// fp16 activations of 9 to 16 tokens: a workgroup of several row tiles has no registers left to load them early beyond K = 4096, so that from about
// two row tiles of K = 8192, or four of 6656 (2 bits: 7424), on they go ahead:
//               8192 x 8192, 9 tokens 9.8/9.7 11.0/11.1 15.1/13.9, 16 10.8/10.4 12.1/12.0 16.2/14.6; 16384 x 8192, 9 14.2/14.3 18.4/17.8 23.9/22.6, 16, 2 bits 15.7/15.0;
//               16384 x 6912, 9 11.9/12.9 16.2/15.9 21.2/20.0, 12288 x 6912, 9 10.4/11.2 12.0/12.6 15.9/16.1, 16384 x 5120, 9 9.6/10.6 12.9/12.7 15.8/16.4;
//               2 bits, 16 tokens, 16384, 20480 and 24576 x 7168 13.7/14.4 15.5/16.2 17.8/18.3, x 7424 15.5/14.8 17.6/17.1 19.6/19.3;
//               8192 x 13824, 9 14.2/13.5 16.9/16.1 22.8/20.0, 8 13.2/13.9 16.0/16.6 20.7/20.2; 28672 x 8192, twice, 16 39.6/36.6 47.8/45.8 65.6/64.6
// Layers of several widths, whose launches the transformation would set apart, stay with the higher line.
// Up to K = 4096 a workgroup makes its activations once whatever its row tiles are, but beyond 14 of them the line is as good as where they would be made again
// (INT8 codes, 2, 3, 4 bits): four layers of 16384 x 4096, 8 tokens 24.0/24.1 25.8/26.6 36.9/37.2, 12 tokens 23.4/22.9 26.7/27.2 37.6/37.7; five of 16384 x 2048, 13
// 19.4/19.0 22.5/22.9 30.3/29.9, 16 19.9/19.2 22.8/23.0 30.6/30.1.
static bool transforms_ahead(const GroupItem *items, int count, int M)
{
    int widest = 0;
    long long all_tiles = 0;
    bool mixed = false;
    for (int i = 0; i < count; ++i) {
        widest = std::max(widest, items[i].K);
        all_tiles += items[i].N / kTileRows;
        mixed = mixed || items[i].bits != items[0].bits;
    }
    const int held = tokens_variant(items[0].bits, M, INT_MAX, INT_MAX, false).tiles;   // row tiles of the longest pass beyond K = 4096
    const long long cus = num_cus(), per_pass = cus * held, passes = (all_tiles + per_pass - 1) / per_pass, activations = (long long)M * widest * passes;
    if (items[0].act_scale != 0.0f) return activations > kAheadCodes;
    if (mixed || M > kTokenBlock || all_tiles <= cus || widest <= 2 * kBW * kTileCols) return activations > kAheadSmoothed;
    return activations > kAheadTiles || (M > kTokenBlock / 2 && (widest >= 8192 || (widest >= (items[0].bits == 2 ? 7424 : 6656) && all_tiles > 3 * cus)));
}

// One launch (and transform_kernel's, where it pays) for layers that one kernel takes: of one width, or of several on the tokens kernel.
// narrow: prefill of few tokens (lcd_narrow.hip), always behind transform_kernel.
static int launch_decode_layers(const GroupItem *items, int count, int M, void *workspace, hipStream_t stream, bool dense, bool narrow = false)
{
    BucketBatch batch{};
    int tiles = 0;
    bool all_quantised = true, mixed = false;
    const int bits = items[0].bits;
    int width[kMaxGroup];
    for (int i = 0; i < count; ++i) {
        all_quantised = all_quantised && items[i].act_scale != 0.0f;
        mixed = mixed || items[i].bits != bits;
        width[i] = items[i].bits;
    }
    const bool tokens_path = narrow || tokens_kernel_takes(bits, M, all_quantised, dense);
    const uint16_t *codes[kMaxGroup] = {};
    int widest = 0;
    for (int i = 0; i < count; ++i) widest = std::max(widest, items[i].K);
    const int held = narrow ? narrow_variant(bits, M, INT_MAX).tiles : tokens_path ? tokens_variant(bits, M, INT_MAX, widest / kTileCols, false).tiles : 1;   // row tiles of a pass
    if (narrow || (tokens_path && transforms_ahead(items, count, M))) {
        // layers that read the same input (same x, s, K and quantisation step: q/k/v or gate/up of a decoder
        // block) share one transformed copy
        TransformBatch qb{};
        size_t offset = 0;
        int max_k = 0, distinct = 0;
        for (int i = 0; i < count; ++i) {
            for (int d = 0; d < distinct && !codes[i]; ++d)
                if (qb.p[d].x == items[i].x && qb.p[d].s == items[i].s && qb.p[d].K == items[i].K && qb.p[d].s_q == items[i].act_scale)
                    codes[i] = qb.p[d].codes;
            if (codes[i]) continue;
            uint16_t *dst = reinterpret_cast<uint16_t *>(static_cast<char *>(workspace) + offset);
            qb.p[distinct++] = TransformItem{items[i].x, items[i].s, dst, items[i].K, items[i].act_scale};
            codes[i] = dst;
            offset += decode_codes_bytes(M, items[i].K);
            if (items[i].K > max_k) max_k = items[i].K;
        }
        const int per_block = kQuantThreads * 8;
        TransformItem &one = qb.p[0];
        void *args[] = {&qb, &M}, *one_args[] = {&one.x, &one.s, &one.codes, &one.K, &one.s_q, &M};
        const int columns = (max_k + per_block - 1) / per_block, tokens = columns * distinct * M <= kQuantWaves ? 1 : kQuantTokens;
        const void *fn = distinct == 1 ? (tokens == 1 ? (const void *)transform_one_kernel<1> : (const void *)transform_one_kernel<kQuantTokens>)
                                       : (tokens == 1 ? (const void *)transform_kernel<1> : (const void *)transform_kernel<kQuantTokens>);
        if (hipError_t e = hipLaunchKernel(fn, dim3(columns, distinct, (M + tokens - 1) / tokens),
                                           dim3(kQuantThreads), distinct == 1 ? one_args : args, 0, stream)) return (int)e;
    }
    for (int i = 0; i < count; ++i) {
        BucketProblem &p = batch.p[i];
        p.packed = (const uint8_t *)items[i].packed;
        p.lutA = (const float *)items[i].lut;
        p.x = codes[i] ? codes[i] : items[i].x; p.s = items[i].s; p.y = items[i].y;
        p.nt = items[i].N / kTileRows; p.kc = items[i].K / kTileCols;
        p.act_scale = items[i].act_scale;
        tiles += p.nt;
    }
    // workgroups per layer
    int grid = num_cus();
    if (grid > tiles) grid = tiles;
    if (grid < count) grid = count;
    // 2 bits on the sparse matrix core with quantised activations: the codes go in as int8 numbers
    const bool int8_codes = !tokens_path && bits != 4 && all_quantised;   // (3 bits: one token, the plain pass only)
    const bool staged_ahead = tokens_path && codes[0] != nullptr;
    const DecodeCost cost = tokens_path ? tokens_cost(held, M, staged_ahead) : bucket_cost(bits, M, int8_codes);
    LayerShape shape[kMaxGroup];
    for (int i = 0; i < count; ++i) shape[i] = LayerShape{batch.p[i].nt, batch.p[i].kc, items[i].bits};
    // The split depends on the shapes only: the last few are kept (a block repeats a few groups; working one out takes 0.3 us of host time, 2 to 7 where the layers differ).
    static_assert(kBW == 8, "lcd_share.h counts rounds of 8 chunks");
    struct SplitMemo { int count, M, grid, ahead, route, pass, nwg[kMaxGroup]; LayerShape shape[kMaxGroup]; };
    constexpr int kMemos = 8;
    static thread_local SplitMemo memos[kMemos] = {};
    static thread_local int oldest = 0;
    const int route = narrow ? 3 : tokens_path ? 1 : int8_codes ? 2 : 0;   // the cost constants depend on it
    int nwg[kMaxGroup], pass = 0;      // pass: of the bucket kernel
    const SplitMemo *known = nullptr;
    for (int e = 0; e < kMemos && !known; ++e) {
        const SplitMemo &m = memos[e];
        bool same = m.count == count && m.M == M && m.grid == grid && m.ahead == (int)staged_ahead && m.route == route;
        for (int i = 0; same && i < count; ++i) same = m.shape[i] == shape[i];
        if (same) known = &m;
    }
    if (known) {
        for (int i = 0; i < count; ++i) nwg[i] = known->nwg[i];
        pass = known->pass;
    } else if (count == 1) {
        if (tokens_path) nwg[0] = grid;
        else pass = share_bucket(bits, M, int8_codes, shape, count, grid, nwg);
    } else {
        if (tokens_path) share_workgroups(cost, shape, count, grid, nwg);
        else pass = share_bucket(bits, M, int8_codes, shape, count, grid, nwg);
        SplitMemo &m = memos[oldest];
        oldest = (oldest + 1) % kMemos;
        m.count = count; m.M = M; m.grid = grid; m.ahead = (int)staged_ahead; m.route = route; m.pass = pass;
        for (int i = 0; i < count; ++i) { m.shape[i] = shape[i]; m.nwg[i] = nwg[i]; }
    }
    // Workgroups are dispatched in the order of their ids, the last of a full grid almost 1 us after the
    // first: the layers whose workgroups have the most to do take the lowest ids (of several widths: the widest first, which the kernel asks for).
    if (count > 1) {
        int order[kMaxGroup];
        double t[kMaxGroup];
        for (int i = 0; i < count; ++i) { order[i] = i; t[i] = cost.even_time(shape[i].bits, shape[i].kc, round_up_div(shape[i].tiles, nwg[i])); }
        std::stable_sort(order, order + count, [&](int a, int b) { return width[a] != width[b] ? width[a] > width[b] : t[a] > t[b]; });
        BucketProblem sorted_p[kMaxGroup];
        int sorted_n[kMaxGroup], sorted_w[kMaxGroup];
        for (int q = 0; q < count; ++q) { sorted_p[q] = batch.p[order[q]]; sorted_n[q] = nwg[order[q]]; sorted_w[q] = width[order[q]]; }
        for (int q = 0; q < count; ++q) { batch.p[q] = sorted_p[q]; nwg[q] = sorted_n[q]; width[q] = sorted_w[q]; }
    }
    grid = 0;
    for (int i = 0; i < count; ++i) grid += nwg[i];
    int acc = 0;
    int wg_begin[kMaxGroup + 1];   // first workgroup of every layer; entries past the last layer hold the total
    for (int i = 0; i < count; ++i) {
        wg_begin[i] = acc;
        acc += nwg[i];
        batch.p[i].tiles_base = batch.p[i].nt / nwg[i];
        batch.p[i].tiles_extra = batch.p[i].nt % nwg[i];
    }
    for (int i = count; i <= kMaxGroup; ++i) wg_begin[i] = acc;
    static_assert(kMaxGroup == 16, "eight leading kernel arguments hold wg_begin[1..16]");
    if (acc >= 0x7fff) return (int)hipErrorInvalidConfiguration;   // 16-bit table fields (acc <= max(CUs, count))
    WgTable table;
    for (int i = 0; i < kMaxGroup / 2; ++i) table.t[i] = (uint32_t)wg_begin[2 * i + 1] | (uint32_t)wg_begin[2 * i + 2] << 16;
    for (int i = 0; i < count; ++i) batch.p[i].wg_first = wg_begin[i];
    DecodeHead head{batch.p[0].x, batch.p[0].s, (uint32_t)batch.p[0].kc | (uint32_t)M << (narrow ? kNarrowTokensShift : 22)};
    bool shared = true;
    for (int i = 1; i < count; ++i) shared = shared && batch.p[i].x == head.x && batch.p[i].s == head.s && batch.p[i].kc == batch.p[0].kc;
    if (shared) head.word |= kHeadShared;
    if (count == 1) {
        const BucketProblem &p = batch.p[0];
        const uint64_t packed = (uint64_t)(uintptr_t)p.packed, lut = (uint64_t)(uintptr_t)p.lutA;
        const uint32_t layer[7] = {(uint32_t)packed, (uint32_t)(packed >> 32), (uint32_t)lut, (uint32_t)(lut >> 32), (uint32_t)p.nt, (uint32_t)p.tiles_base,
                                   (uint32_t)p.tiles_extra};
        for (int i = 0; i < 7; ++i) table.t[i] = layer[i];
        head.word |= kHeadSingle;
    }
    size_t lds;
    const void *fn;
    int variant, waves = kBW;
    int most = 1;          // row tiles of a workgroup
    for (int i = 0; i < count; ++i) most = std::max(most, (batch.p[i].nt + nwg[i] - 1) / nwg[i]);
    if (!tokens_path) {
        const BucketVariant v = bucket_variant(bits, M, int8_codes, pass, most, widest / kTileCols);
        lds = v.lds_bytes;
        fn = count == 1 ? v.single : v.fn;
        waves = v.waves;
        variant = 2 * v.id + (count == 1 ? 1 : 0);
    } else {
        const TokensVariant tv = narrow ? narrow_variant(bits, M, most) : mixed ? tokens_mixed_variant(M, most, widest / kTileCols) : tokens_variant(bits, M, most, widest / kTileCols, staged_ahead);
        lds = tv.lds_bytes;
        fn = tv.fn;
        waves = tv.waves;
        variant = 2 * kBucketVariants + (narrow ? kTokensVariants + kMixedTokensVariants : mixed ? kTokensVariants : 0) + tv.id;
    }
    uint32_t widths = 0;   // first workgroup of the 3-bit layers, and (upper half) of the 2-bit layers
    for (int i = 0; i < count; ++i) widths += width[i] == 4 ? nwg[i] * 0x10001u : width[i] == 3 ? nwg[i] * 0x10000u : 0u;
    static PerDeviceFlags<2 * kBucketVariants + kTokensVariants + kMixedTokensVariants + kNarrowVariants> lds_raised;
    if (hipError_t e = raise_lds_limit_once(lds_raised, variant, fn, lds)) return (int)e;
    void *args[] = {&table.t[0], &table.t[1], &table.t[2], &table.t[3], &table.t[4], &table.t[5], &table.t[6], &table.t[7],
                    &head.x, &head.s, &head.word, &batch};
    void *mixed_args[] = {&table.t[0], &table.t[1], &table.t[2], &table.t[3], &table.t[4], &table.t[5], &table.t[6], &table.t[7],
                          &head.x, &head.s, &head.word, &widths, &batch};
    if (hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(waves * 64), mixed ? mixed_args : args, lds, stream)) return (int)e;
    return (int)hipGetLastError();
}

// The kernels address a layer's activations with 32 bits.
static int tokens_that_fit(int M, int K) { return (int)std::min<long long>(M, ((1ll << 32) - 512) / (2ll * K)); }

// The launches of a group: one for layers of one width.  Layers of several widths that the tokens kernel takes go out together, unless their
// activations are transformed ahead (two launches already, and long ones); the bucket kernel's width by width.
int launch_decode_group(const GroupItem *items, int count, int M, int bits, void *workspace, void *stream_, bool dense)
{
    hipStream_t stream = (hipStream_t)stream_;
    bool all_quantised = true, mixed = false;
    for (int i = 0; i < count; ++i) {
        all_quantised = all_quantised && items[i].act_scale != 0.0f;
        mixed = mixed || items[i].bits != items[0].bits;
    }
    GroupItem sub[kMaxGroup];
    int n = 0;
    // layers of 4 GiB of activations and more: alone (a layer's launches must not depend on its neighbours), some tokens after the other
    for (int i = 0; i < count; ++i) {
        const int most = tokens_that_fit(M, items[i].K);
        if (most == M) { sub[n++] = items[i]; continue; }
        for (int m = 0; m < M; m += most) {
            GroupItem part = items[i];
            part.x += (size_t)m * part.K;
            part.y += (size_t)m * part.N;
            if (int e = launch_decode_layers(&part, 1, std::min(most, M - m), workspace, stream, dense)) return e;
        }
    }
    if (n == 0) return 0;
    if (n < count) return launch_decode_group(sub, n, M, bits, workspace, stream_, dense);
    if (bits != 0 || !mixed) return launch_decode_layers(items, count, M, workspace, stream, dense);
    n = 0;
    for (int i = 0; i < count; ++i)
        if (tokens_kernel_takes(items[i].bits, M, all_quantised, dense)) sub[n++] = items[i];
    const bool together = n > 0 && M <= kTokenBlock && !transforms_ahead(sub, n, M);
    if (together)
        if (int e = launch_decode_layers(sub, n, M, workspace, stream, dense)) return e;
    for (int b = 2; b <= 4; ++b) {
        if (together && tokens_kernel_takes(b, M, all_quantised, dense)) continue;
        n = 0;
        for (int i = 0; i < count; ++i)
            if (items[i].bits == b) sub[n++] = items[i];
        if (n > 0)
            if (int e = launch_decode_layers(sub, n, M, workspace, stream, dense)) return e;
    }
    return 0;
}

int launch_narrow_group(const GroupItem *items, int count, int M, void *workspace, void *stream)
{
    return launch_decode_layers(items, count, M, workspace, (hipStream_t)stream, true, true);
}

// ---- scratch for callers that cannot allocate ---------------------------------------------------
// lcd_lut_gemv_noalloc keeps the transformed activations (at most 16 tokens x kStaticScratchCols
// columns, fp16) in this file-scope device array instead of a workspace the caller brings.  Every GPU
// holds its own copy at its own address; the array's name is only a host-side handle, so the device
// address is asked for once per device and kernels are given that address.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static void *g_scratch_ptr[kMaxDevices] = {};
static std::mutex g_scratch_mutex;

// Device address of the current device's scratch array (hipError_t as int; 0 = success).
static int static_scratch(void **out)
{
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return 0;
}

int launch_gemv_noalloc(const void *packed, const void *lut, const uint16_t *x, const float *s, uint16_t *y,
                        int M, int N, int K, int bits, void *stream_)
{
    void *ws = nullptr;
    if (int e = static_scratch(&ws)) return e;
    GroupItem it{packed, lut, x, s, y, N, K, 0.0f, bits};
    return launch_decode_group(&it, 1, M, bits, ws, stream_);
}

int launch_gemv(const void *packed, const void *lut, const uint16_t *x, const float *s, uint16_t *y,
                int M, int N, int K, int bits, float act_scale, void *workspace, void *stream_)
{
    GroupItem it{packed, lut, x, s, y, N, K, act_scale, bits};
    return launch_decode_group(&it, 1, M, bits, workspace, stream_);
}

}  // namespace lcd
