// Prefill path (M >= 17; any M >= 1 accepted) of the smoothed table-lookup product, gfx950: the wide kernel
// (lcd_gemm_wide.h) and the launcher of all prefill kernels.
#include <hip/hip_runtime.h>
#include <algorithm>
#include "lcd_gemm_common.h"
#include "lcd_launch.h"

namespace lcd {

// Which kernel takes a layer.  The rules look at the layer and the number of tokens alone, never at the group it is
// called in: the kernels add in different orders, and a layer's result must not depend on its neighbours.
// Up to 16 tokens the decode kernels (the dequantising one, except for INT8 codes with 2-bit indices).  Up to 32 tokens the tokens kernel, which needs no smoothing launch,
// also keeps the small layers.  One call with 32 tokens, weights from memory, tokens kernel / split kernel, 2, 3 and 4 bits: 2048 x 2048
// 6.4/8.1 6.7/8.9 7.0/9.3 us, 2048 x 4096 8.3/10.6 8.7/11.4 9.3/11.9, 11008 x 1024 7.1/8.7 7.9/9.0 7.7/9.8, 28672 x 512 11.9/12.0 13.2/12.4 16.6/13.3;
// beyond the line 4096 x 4096 8.9/10.9 9.4/11.6 10.2/12.5, 6144 x 4096 11.6/11.0 12.5/11.8 15.1/13.0, 8192 x 4096 11.7/11.2 13.0/12.1 15.9/13.8.  A
// layer of 4096 x 4096 alone would gain from the tokens kernel too; three of them in one call, which must take the same kernel, are
// 12288 x 4096 to it and would lose.
static bool decode_takes(int M, int N, int K)
{
    return (M <= 16 || (M <= kDecodeTokens && (long long)N * K < (1ll << 24))) && (long long)M * K * 2 < (1ll << 32);
}
// The narrow kernel takes layers of few tokens: it reads every activation once per compute unit and pads tokens to 16 only, the split kernel
// reads a tile's activations once per 64 rows.  So the line lies where a compute unit has one row tile only (up to 4096 rows), which the
// activations of many tokens or columns do not pay for; beyond 64 tokens it holds three row tiles at a time, so that a fourth costs a second
// pass.  One call, weights from memory, split (up to 32 tokens and beyond 128 large tiles: as before it) / narrow, 2, 3 and 4 bits, us:
//   32 tokens   4096 x 4096  9.9/9.5 10.4/10.0 11.9/10.4     4096 x 11008 16.9/15.8 19.9/16.5 22.5/17.9     28672 x 8192, twice 62.6/55.7 81.4/70.5 92.5/94.0
//   40          4096 x 4096 10.6/10.5 11.1/10.8 12.8/11.4    4096 x 11008 18.3/18.1 20.3/19.4 23.4/20.4     11008 x 4096, twice 27.9/18.2 30.8/20.9 35.4/26.9
//   48          4096 x 11008 17.9/19.4 20.3/20.5 23.2/21.3   8192 x 8192 20.0/17.8 24.2/19.5 26.1/22.4      28672 x 8192, twice 89.1/67.9 101.6/82.0 121.3/105.7
//   64          4096 x 4096 10.7/11.8 11.2/12.2 12.8/12.5    8192 x 8192 20.2/20.0 24.4/21.9 26.0/24.5      11008 x 4096, twice 29.5/25.0 31.8/28.0 37.1/32.2
//   80          4096 x 4096 12.7/13.6 14.5/14.0 15.9/14.5    8192 x 8192 27.7/23.5 30.0/25.1 35.4/27.5      11008 x 4096, twice 36.0/27.9 39.3/30.8 43.5/34.9
//   old time / new, over all widths   48 tokens, 1024..4096 rows: K = 2048 1.02..1.14, 4096 0.94..1.11, 8192 0.82..1.09     64 tokens: K = 2048 0.95..1.11, 4096 0.87..1.04
//                                     80 tokens: 5120 rows 0.84..1.25, 6144..11008 1.05..1.33, 16384 0.83..0.94             96 tokens: 6144..11008 rows 0.94..1.23
static bool narrow_takes(int M, int N, int K, int bits)
{
    if (M <= 16 || M > kNarrowTokens || (long long)M * K * 2 >= (1ll << 32)) return false;
    if (N > 4096) return M <= 64 || (N >= 6144 && N <= 12288);
    if (M <= 32) return true;
    if (M <= 48) return K <= 2048 || (N > 2048 && (K <= 4096 || bits > 2));
    return M <= 64 && N >= 2048 && K <= 2048;
}
// The split kernel takes layers of few output tiles: those that fit one round of its largest tile (64 x 128) on the 256 compute units (the whole
// chip, whatever part of it a process sees: a layer's bits must not depend on that).  Beyond that the wide kernel's tiles, which share the activations among
// four or eight waves, win.  A call without its smoothing, split / wide, 2, 3 and 4 bits, us:
//   one round         4096 x 4096, 333 tokens 17.3/20.7 19.3/24.4 21.2/29.3, 450 (256 tiles) 22.5/22.7 24.0/26.4 25.7/30.8; 4096 x 11008, 333 39.9/47.9 41.4/54.9 47.4/67.7;
//                     8192 x 8192, 224 tokens 37.8/39.0 37.7/45.7 41.9/54.0; 11008 x 4096, 100 tokens 15.5/18.5 16.2/24.0 19.5/28.6
//   beyond            4096 x 4096, 640 tokens (large tiles of 256 x 128 as before / wide) 30.8/26.4 32.8/29.0 36.3/32.9; 11008 x 4096, 160 tokens 25.2/22.5 28.8/26.3 31.7/30.4;
//                     8192 x 8192, 333 tokens 54.2/49.2 57.7/54.4 68.6/62.5; two of 11008 x 4096, 333 tokens 84.8/69.8 94.5/77.1 103.8/89.5
//   several layers    three of 4096 x 4096, 333 tokens 45.5/39.8 49.7/42.9 58.9/50.8, 450 58.8/45.7 63.0/49.6 68.8/58.1: hence the lower line at 2 bits, where a
//                     single layer of a nearly full round is as fast either way
// (The split kernel addresses the activations with 32 bits.)
static bool split_takes(int M, int N, int K, int bits)
{
    const long long blocks = (M + 127) / 128, rows64 = (N + 63) / 64;
    return rows64 * blocks <= (bits == 2 ? 224 : 256) && (long long)plan_gemm(M, N, K, 2).m_pad * K * 2 < (1ll << 32);
}

// Tile of a launch of the split kernel: rounds of workgroups over the compute units times the time of one workgroup.  Measured
// in single rounds (K = 4096 and 11008): a fixed part, and a part per column that is bound by the activations' way into LDS
// (75..98 GB/s per compute unit; 32 tokens x 64 rows: by the dequantiser).  In launches of several rounds every tile takes longer
// than that (the rounds share the L2), but their order holds: 177 launches timed with each of the six tiles (1 to 3 layers of 1024..13824
// rows, K = 2048..11008, 33..512 tokens, 2, 3 and 4 bits) took 1.002 times the best tile's time in the mean, 1.03 at the ninth decile,
// 1.14 at most (three layers of 2048 x 2048, 512 tokens, 3 bits: 32.8 against 28.9 us).
struct SplitTile { int pairs, blocks; double fixed_us, column_ns[3]; };   // column_ns: 2, 3, 4 bits
static const SplitTile kSplitTiles[] = {
    {2, 4, 3.0, {2.58, 2.70, 3.13}}, {2, 3, 2.5, {2.13, 2.40, 3.05}}, {2, 2, 2.0, {1.56, 1.74, 2.33}},
    {2, 1, 1.5, {1.34, 1.66, 2.58}}, {1, 2, 1.5, {1.48, 1.60, 1.69}}, {1, 1, 1.3, {0.79, 0.88, 1.17}},
};
// time of all workgroups of a tile's launch one after the other, and their number
static double split_work(const GemmBatch &bt, const SplitTile &t, int M, int bits, double &wgs)
{
    double work = 0.0;
    wgs = 0.0;
    for (int q = 0; q < bt.count; ++q) {
        const double n = (double)((bt.p[q].N + 32 * t.pairs - 1) / (32 * t.pairs)) * ((M + 32 * t.blocks - 1) / (32 * t.blocks));
        wgs += n;
        work += n * (t.fixed_us + 1e-3 * t.column_ns[bits - 2] * bt.p[q].K);
    }
    return work;
}
static const SplitTile &choose_split_tile(const GemmBatch &bt, int M, int bits)
{
    const SplitTile *best = nullptr;
    double best_time = 0.0;
    for (const SplitTile &t : kSplitTiles) {
        double wgs;
        const double work = split_work(bt, t, M, bits, wgs), time = __builtin_ceil(wgs / num_cus()) * work / wgs;
        if (!best || time < best_time) { best = &t; best_time = time; }
    }
    return *best;
}
// Next to wide tiles there are no rounds of their own to fill: the tile with the least work of the two that cost least per output.
static const SplitTile &choose_mixed_tile(const GemmBatch &bt, int M, int bits)
{
    double wgs;
    return split_work(bt, kSplitTiles[0], M, bits, wgs) <= split_work(bt, kSplitTiles[1], M, bits, wgs) ? kSplitTiles[0] : kSplitTiles[1];
}

// Whether the wide kernel takes a layer whole (lcd_gemm_plan.h); the last few answers are kept (working one out takes 2 us of host time).
static bool wide_whole(int M, int N, int K, int bits)
{
    struct Memo { int M, N, K, bits; bool whole; };
    constexpr int kMemos = 8;
    static thread_local Memo memos[kMemos] = {};
    static thread_local int oldest = 0;
    for (const Memo &m : memos)
        if (m.M == M && m.N == N && m.K == K && m.bits == bits) return m.whole;
    const bool whole = whole_takes(M, N, K, bits);
    memos[oldest] = Memo{M, N, K, bits, whole};
    oldest = (oldest + 1) % kMemos;
    return whole;
}

int launch_gemm(const void *packed, const void *lut, const uint16_t *x, const float *s, uint16_t *y,
                int M, int N, int K, int bits, float act_scale, void *workspace, const GemmPlan &, void *stream)
{
    GroupItem it{packed, lut, x, s, y, N, K, act_scale, bits};
    return launch_gemm_group(&it, 1, M, bits, workspace, stream);
}

int launch_gemm_group(const GroupItem *items, int count, int M, int bits, void *workspace, void *stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    const int Mpad = plan_gemm(M, items[0].N, items[0].K, bits).m_pad;
    // layers with the longest tiles (largest K) first in every XCD's queue
    int order[kMaxGroup];
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order, order + count, [&](int a, int b) { return items[a].K > items[b].K; });
    // Layers that read the same input (same x, s, K and quantisation step: q/k/v, gate/up of a decoder
    // block) share one transformed copy of it: the activations are smoothed once per distinct input.
    SmoothItem sm[kMaxGroup];
    int distinct = 0;
    GemmBatch batch[3] = {};   // the wide kernel's layers in halves, the split kernel's, the wide kernel's whole ones
    GroupItem small[kMaxGroup], narrow[kMaxGroup];
    int small_count = 0, narrow_count = 0;       // the decode kernels' layers, the narrow kernel's
    size_t offset = 0;
    for (int q = 0; q < count; ++q) {
        const GroupItem &it = items[order[q]];
        if (decode_takes(M, it.N, it.K)) { small[small_count++] = it; continue; }
        if (narrow_takes(M, it.N, it.K, bits)) { narrow[narrow_count++] = it; continue; }
        uint8_t *xs = nullptr;
        for (int d = 0; d < distinct && !xs; ++d)
            if (sm[d].x == it.x && sm[d].s == it.s && sm[d].K == it.K && sm[d].s_q == it.act_scale) xs = static_cast<uint8_t *>(sm[d].xs);
        if (!xs) {
            xs = static_cast<uint8_t *>(workspace) + offset;
            offset += plan_gemm(M, it.N, it.K, bits).xs_bytes;
            sm[distinct++] = SmoothItem{it.x, it.s, xs, it.K, it.act_scale};
        }
        GemmBatch &bt = batch[split_takes(M, it.N, it.K, bits) ? 1 : wide_whole(M, it.N, it.K, bits) ? 2 : 0];
        GemmProblem &p = bt.p[bt.count++];
        p.packed = static_cast<const uint8_t *>(it.packed);
        // byte-split tables: behind the bucket multipliers (2 and 3 bits), the whole table (4 bits)
        p.lutB = static_cast<const uint8_t *>(it.lut) + (bits == 4 ? 0 : (size_t)it.N * (bits == 2 ? 4 : 8) * 4);
        p.xs = xs;
        p.y = it.y;
        p.N = it.N; p.K = it.K;
        p.out_scale = it.act_scale != 0.0f ? it.act_scale : 1.0f;
    }
    // the decode kernels' scratch lies behind the smoothed activations (it takes less than a layer's share of those)
    if (small_count > 0)
        if (int e = launch_decode_group(small, small_count, M, bits, static_cast<char *>(workspace) + offset, stream, true)) return e;
    if (narrow_count > 0) {
        for (int i = 0; i < small_count; ++i) offset += decode_codes_bytes(M, small[i].K);
        if (int e = launch_narrow_group(narrow, narrow_count, M, static_cast<char *>(workspace) + offset, stream)) return e;
    }
    if (distinct == 0) return 0;
    for (GemmBatch &bt : batch) { bt.M = M; bt.Mpad = Mpad; }
    // places of the split kernel's tiles (rows x tokens each) in the XCDs' queues; returns the queue's length
    auto queue_split = [&](GemmBatch &bt, int rows, int tokens) {
        int queue = 0;
        for (int q = 0; q < bt.count; ++q) {
            GemmProblem &p = bt.p[q];
            p.grid_rows = (p.N + rows - 1) / rows;
            p.tiles_per_xcd = (p.grid_rows * ((M + tokens - 1) / tokens) + kXcds - 1) / kXcds;
            p.queue_begin = queue;
            queue += p.tiles_per_xcd;
        }
        return queue;
    };
    auto queue_wide = [&](GemmBatch &bt, bool whole) {
        WideLayer layers[kMaxGroup];
        for (int q = 0; q < bt.count; ++q) layers[q] = WideLayer{bt.p[q].N, bt.p[q].K};
        double wgs, more_us = 0.0;      // (split tiles next to others take 1.5 times what they take in a round of their own)
        if (!whole && batch[1].count > 0) more_us = 1.5 * split_work(batch[1], choose_mixed_tile(batch[1], M, bits), M, bits, wgs) / num_cus();
        const WideTiles t = choose_wide(whole, layers, bt.count, (M + 31) / 32, bits, num_cus(), nullptr, more_us);
        long long tiles = 0;
        for (int q = 0; q < bt.count; ++q) {
            GemmProblem &p = bt.p[q];
            p.grid_rows = (p.N + wide_rows(t.form) - 1) / wide_rows(t.form);
            p.tiles[0] = (uint32_t)p.grid_rows * t.big;
            p.tiles[1] = (uint32_t)p.grid_rows * (t.columns - t.big);
            tiles += (long long)p.grid_rows * t.columns;
        }
        bt.tiles = t;
        return (int)((tiles + kXcds - 1) / kXcds);
    };
    if (int e = launch_smooth_group(sm, distinct, M, Mpad, stream)) return e;
    static PerDeviceFlags<kWideVariants + kSplitVariants + kMixedVariants> lds_raised;
    auto launch = [&](int queue, const void *fn, int flag, int threads, size_t lds_bytes, void **args) -> int {
        if (hipError_t e = raise_lds_limit_once(lds_raised, flag, fn, lds_bytes)) return (int)e;
        if (hipError_t e = hipLaunchKernel(fn, dim3((unsigned)queue * kXcds), dim3(threads), args, lds_bytes, stream)) return (int)e;
        return (int)hipGetLastError();
    };
    auto launch_wide = [&](GemmBatch &bt, int queue) -> int {
        const WideVariant v = bits == 2 ? wide_variant<2>(bt.tiles) : bits == 3 ? wide_variant<3>(bt.tiles) : wide_variant<4>(bt.tiles);
        void *args[] = {&bt};
        return launch(queue, v.fn, v.id, v.threads, v.lds_bytes, args);
    };
    if (batch[2].count > 0)
        if (int e = launch_wide(batch[2], queue_wide(batch[2], true))) return e;
    const int wide = batch[0].count > 0 ? queue_wide(batch[0], false) : 0;
    // wide tiles of 3 or 4 blocks go out with the split tiles
    const WideTiles &tiles = batch[0].tiles;
    const bool together = wide > 0 && batch[1].count > 0 && (tiles.blocks == 4 || (tiles.blocks == 3 && tiles.big == tiles.columns));
    if (wide > 0 && !together)
        if (int e = launch_wide(batch[0], wide)) return e;
    if (batch[1].count == 0) return 0;
    const SplitTile &t = together ? choose_mixed_tile(batch[1], M, bits) : choose_split_tile(batch[1], M, bits);
    const int split = queue_split(batch[1], 32 * t.pairs, 32 * t.blocks);
    if (!together) {
        const SplitVariant sv = split_variant(bits, t.pairs, t.blocks);
        void *args[] = {&batch[1]};
        return launch(split, sv.fn, kWideVariants + sv.id, 512, sv.lds_bytes, args);
    }
    const WideVariant v = bits == 2 ? mixed_variant<2>(tiles, t.blocks) : bits == 3 ? mixed_variant<3>(tiles, t.blocks) : mixed_variant<4>(tiles, t.blocks);
    uint32_t wide_blocks = (uint32_t)wide * kXcds;
    void *args[] = {&batch[0], &batch[1], &wide_blocks};
    return launch(wide + split, v.fn, kWideVariants + kSplitVariants + v.id, v.threads, v.lds_bytes, args);
}

}  // namespace lcd
