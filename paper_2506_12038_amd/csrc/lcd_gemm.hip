// Prefill path (M >= 17; any M >= 1 accepted) of the smoothed table-lookup product, gfx950: the large-tile kernel
// (lcd_gemm_large.h) and the launcher of all prefill kernels.
#include <hip/hip_runtime.h>
#include <algorithm>
#include "lcd_gemm_large.h"
#include "lcd_launch.h"

namespace lcd {

template <int BITS>
__global__ void __launch_bounds__(kGemmWaves * 64, 1) gemm_group_kernel(const GemmBatch batch)
{
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    gemm_workgroup<BITS>(batch, blockIdx.x, lds);
}

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
// The split kernel takes layers of few output tiles.  Its advantage lies in rounds of workgroups over the 256 compute units (the whole
// chip, whatever part of it a process sees: a layer's bits must not depend on that) and in tiles as narrow as the tokens: 256 x 128 tiles
// spend the same time on 33 tokens as on 128.  It takes what fits
//   - one round of any of its tiles (64 x 128 being the largest);
//   - two rounds of 64 x 64;
//   - two rounds of 64 x 96 where K >= 8192, or where K >= 4096 and a quarter or more of the large tiles' work would be padding;
//   - just above 128 large tiles, which no longer fit one round when cut in two (K >= 4096).
// Time of a call, large tiles / split tiles, 2, 3 and 4 bits:
//   one round         4096 rows, 512 tokens    K = 2048 22.0/19.9 23.1/20.2 25.6/21.1   K = 4096 35.3/28.4 37.8/29.9 41.4/31.3   K = 11008 79.7/59.3 84.5/61.6 95.7/66.7
//   two of 64 x 64    28672 rows, 40 tokens    K = 2048 19.7/17.6 21.1/18.8 24.0/21.8   K = 4096 31.6/25.3 33.7/27.7 39.0/32.7   K = 8192 54.1/40.8 58.4/44.4 67.6/53.3
//                     8448 rows, 192 tokens    K = 2048 20.4/18.5 21.2/19.3 23.9/22.3   K = 4096 33.3/27.0 35.1/29.6 39.5/34.4   K = 8192 56.3/42.8 60.2/47.3 70.0/56.8
//   two of 64 x 96    11008 rows, 160 tokens   K = 2048 20.8/21.5 21.7/22.0 24.5/24.9   K = 4096 33.9/30.8 35.8/33.6 40.0/39.3   K = 8192 56.7/51.0 61.1/55.2 68.7/66.2
//                     4096 rows, 545 tokens    K = 2048 22.0/23.2 23.0/23.9 25.9/26.8   K = 4096 35.7/34.6 37.4/37.1 42.1/42.7   K = 8192 59.8/56.4 64.7/60.7 75.8/72.3
//   two of 64 x 128   11008 rows, 224 tokens   K = 2048 21.6/25.5 22.2/27.9 25.7/29.5   K = 4096 35.3/38.2 37.4/41.6 43.7/46.4   K = 8192 58.9/62.3 62.9/67.5 74.3/76.7
//                     28672 rows, 128 tokens   K = 2048 22.9/28.2 23.8/29.4 26.6/32.0   K = 4096 38.0/44.1 39.7/46.0 45.1/50.7   K = 8192 65.7/72.3 68.5/74.4 78.2/83.9
//   129 large tiles   11008 rows, 333 tokens   K = 2048 32.4/34.3 34.1/36.2 40.3/40.6   K = 4096 53.9/51.6 58.2/56.5 67.8/64.6   K = 11008 121.6/114.0 131.1/119.2 161.3/144.5
// Several layers of a size in one launch fill large tiles' rounds better.  K = 4096, 3 bits: two layers of 11008 rows, 160 tokens 58.7/52.3, 256 tokens 60.5/68.0;
// three of 4096 rows, 576 tokens 67.1/88.4, 1024 tokens 109/139: hence the padding's share, which leaves those to the large tiles.
// (The split kernel addresses the activations with 32 bits.)
static bool split_takes(int M, int N, int K)
{
    constexpr long long kChip = 256;
    const long long blocks = (M + kGemmTokens - 1) / kGemmTokens, tiles = (N + 255) / 256 * blocks, rows64 = (N + 63) / 64;
    const bool padding = 3 * blocks * kGemmTokens >= 4ll * M;
    const bool one_round = rows64 * blocks <= kChip, narrow = rows64 * ((M + 63) / 64) <= 2 * kChip;
    const bool medium = rows64 * ((M + 95) / 96) <= 2 * kChip && (K >= 8192 || (K >= 4096 && padding));
    const bool idle = one_round || narrow || medium || (tiles > 128 && tiles <= 136 && K >= 4096);
    return idle && (long long)plan_gemm(M, N, K, 2).m_pad * K * 2 < (1ll << 32);
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
// Next to large tiles there are no rounds of their own to fill: the tile with the least work of the two that cost least per output.
static const SplitTile &choose_mixed_tile(const GemmBatch &bt, int M, int bits)
{
    double wgs;
    return split_work(bt, kSplitTiles[0], M, bits, wgs) <= split_work(bt, kSplitTiles[1], M, bits, wgs) ? kSplitTiles[0] : kSplitTiles[1];
}

// Last tiles of an XCD's queue that are cut in two (128 rows each): those of a last round that would leave half of the compute units
// or more idle, so that the halves still fit one round.
// 7B block, 3 bits, 2048 tokens (gate and up: 172 tiles per queue, the last 12 of them in a sixth round of 32): 793 -> 780 us.  With
// more than half a round left the halves would need two rounds of about 0.6 of a whole tile's time each.
static int half_tiles(int queue)
{
    const int cus = num_cus() / kXcds, rest = cus > 0 ? queue % cus : 0;
    return 2 * rest <= cus ? rest : 0;
}

// The same cut where split tiles follow in the queue: they can fill the idle compute units as well, so both ways are played
// through on an XCD's compute units (each takes the next workgroup of the queue), with the times of workgroups on a full chip:
// a whole large tile 3 us + 10.5 ns per column (4 bits: 13.7), half a tile 0.65 of it, a split tile 1.5 times what it takes in a
// round of its own.  3 bits, no cut / cut: q 8192, k, v 1024 rows, K = 8192, 333 tokens 101 / 78 us, 1500 tokens 255 / 271; 8192 x 2048
// with 2048 x 8192, 333 tokens 45 / 60.
class CuTimes {
public:
    explicit CuTimes(int cus) { t_[0] = 0.0; n_[0] = cus; }
    void add(int wgs, double us)      // the next `wgs` workgroups of the queue
    {
        while (wgs > 0) {
            const int take = std::min(wgs, n_[0]);
            const double end = t_[0] + us;
            wgs -= take;
            n_[0] -= take;
            if (n_[0] == 0) {
                --count_;
                for (int i = 0; i < count_; ++i) { t_[i] = t_[i + 1]; n_[i] = n_[i + 1]; }
            }
            int at = count_;
            for (; at > 0 && t_[at - 1] > end; --at) { t_[at] = t_[at - 1]; n_[at] = n_[at - 1]; }
            t_[at] = end;
            n_[at] = take;
            ++count_;
        }
    }
    double end() const { return t_[count_ - 1]; }

private:
    // ascending: n_[i] compute units are free at t_[i].  A call adds one entry at most (its last workgroups may take a part
    // of one), and a launch makes fewer than three calls per layer.
    double t_[3 * kMaxGroup + 1];
    int n_[3 * kMaxGroup + 1], count_ = 1;
};
static int mixed_half_tiles(const GemmBatch &large, int queue, const GemmBatch &split, const SplitTile &t, int M, int bits)
{
    const int cut = half_tiles(queue), cus = num_cus() / kXcds;
    if (cut == 0 || cus <= 0) return 0;
    double time[2];
    for (int c = 0; c < 2; ++c) {
        CuTimes cu(cus);
        for (int q = 0; q < large.count; ++q) {
            const int end = q + 1 < large.count ? large.p[q + 1].queue_begin : queue;
            const int whole = std::max(0, std::min(end, c ? queue - cut : queue) - large.p[q].queue_begin);
            const double us = 3.0 + 1e-3 * (bits == 4 ? 13.7 : 10.5) * large.p[q].K;
            cu.add(whole, us);
            cu.add(2 * (end - large.p[q].queue_begin - whole), 0.65 * us);
        }
        for (int q = 0; q < split.count; ++q) {
            const int wgs = (split.p[q].N + 32 * t.pairs - 1) / (32 * t.pairs) * ((M + 32 * t.blocks - 1) / (32 * t.blocks));
            cu.add((wgs + kXcds - 1) / kXcds, 1.5 * (t.fixed_us + 1e-3 * t.column_ns[bits - 2] * split.p[q].K));
        }
        time[c] = cu.end();
    }
    return time[1] < 1.08 * time[0] ? cut : 0;   // (the cut where they are near one another: shorter workgroups even out)
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
    GemmBatch batch[2] = {};   // [0] the large-tile kernel's layers, [1] the split kernel's
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
        GemmBatch &bt = batch[split_takes(M, it.N, it.K)];
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
    // places of the layers' tiles (rows x tokens each) in the XCDs' queues; returns the queue's length
    auto queue_tiles = [&](GemmBatch &bt, int rows, int tokens) {
        int queue = 0;
        for (int q = 0; q < bt.count; ++q) {
            GemmProblem &p = bt.p[q];
            p.grid_rows = (p.N + rows - 1) / rows;
            p.tiles_per_xcd = (p.grid_rows * ((M + tokens - 1) / tokens) + kXcds - 1) / kXcds;
            p.queue_begin = queue;
            queue += p.tiles_per_xcd;
        }
        bt.M = M; bt.Mpad = Mpad;
        return queue;
    };
    if (int e = launch_smooth_group(sm, distinct, M, Mpad, stream)) return e;
    static PerDeviceFlags<3 + kSplitVariants + kMixedVariants> lds_raised;
    auto launch = [&](int queue, const void *fn, int flag, size_t lds_bytes, void **args) -> int {
        if (hipError_t e = raise_lds_limit_once(lds_raised, flag, fn, lds_bytes)) return (int)e;
        if (hipError_t e = hipLaunchKernel(fn, dim3((unsigned)queue * kXcds), dim3(kGemmWaves * 64), args, lds_bytes, stream)) return (int)e;
        return (int)hipGetLastError();
    };
    const int large = batch[0].count > 0 ? queue_tiles(batch[0], kGemmRowGroups * 32 * kGemmPairs, kGemmTokens) : 0;
    if (batch[1].count == 0) {
        const void *fn = bits == 2 ? (const void *)gemm_group_kernel<2> : bits == 3 ? (const void *)gemm_group_kernel<3> : (const void *)gemm_group_kernel<4>;
        const int tail = half_tiles(large);
        batch[0].tail_begin = large - tail;
        void *args[] = {&batch[0]};
        return launch(large + tail, fn, bits - 2, 2 * kStageBytes, args);
    }
    if (batch[0].count == 0) {
        const SplitTile &t = choose_split_tile(batch[1], M, bits);
        const SplitVariant sv = split_variant(bits, t.pairs, t.blocks);
        void *args[] = {&batch[1]};
        return launch(queue_tiles(batch[1], 32 * t.pairs, 32 * t.blocks), sv.fn, 3 + sv.id, sv.lds_bytes, args);
    }
    const SplitTile &t = choose_mixed_tile(batch[1], M, bits);
    const SplitVariant sv = mixed_variant(bits, t.blocks);
    const int split = queue_tiles(batch[1], 32 * t.pairs, 32 * t.blocks), tail = mixed_half_tiles(batch[0], large, batch[1], t, M, bits);
    batch[0].tail_begin = large - tail;
    uint32_t large_blocks = (uint32_t)(large + tail) * kXcds;
    void *args[] = {&batch[0], &batch[1], &large_blocks};
    return launch(large + tail + split, sv.fn, 3 + kSplitVariants + sv.id, sv.lds_bytes, args);
}

}  // namespace lcd
